"""Dense products on the bf16 matrix cores (three bf16 parts per float32) where the split could go wrong: against 64 bits
at tile edges, and where the float32 instructions have to take over (infinities, NaN, overflow, tiny values)."""
import numpy as np
import pytest
import torch

from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("transform_family")]

# Sums of K terms in float32, each operand within 2^-25 of its value after the split: K roundings of the running sum at
# worst, sqrt(K) as they fall.  The row's largest element is about sqrt(K) |h| |w|, so 1e-5 of it leaves a factor of five
# at K = 2900; the 2-norm of the error is held to eight roundings of size 2^-24 (measured: 2 to 14 e-8 * sqrt(K / 16)).
def norm_error(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


@pytest.mark.parametrize("n,d_in,d_out", [
    (127, 15, 31), (128, 16, 32), (129, 17, 33),            # one tile and its neighbours, one K tile
    (257, 31, 63), (257, 33, 65), (300, 47, 129), (300, 8, 192), (300, 7, 193),
    (1000, 1, 256), (1000, 2900, 255), (385, 64, 257), (130, 100, 513),
])
@pytest.mark.parametrize("pitch", [0, 3])                   # rows 16-byte aligned or not
def test_forward_and_weight_gradient_against_64_bits(n, d_in, d_out, pitch):
    ldh = wl.pad_ld(d_in, 4) + pitch
    H = wl.random_matrix(n, d_in, n + d_in, ld=ldh)
    H[:, d_in:] = np.nan
    W = wl.random_matrix(d_in, d_out, d_out)
    G = wl.random_matrix(n, d_out, 5)
    Z = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), None, False).cpu().numpy()[:, :d_out].astype(np.float64)
    H64 = H[:, :d_in].astype(np.float64)
    want = H64 @ W.astype(np.float64)
    assert_close(Z, want, what="forward")
    assert norm_error(Z, want) <= 2.0 ** -24 * 8 * max(1.0, np.sqrt(d_in / 16.0))
    gW, gb = Hn.transform_backward(Hn.dev(H), d_in, Hn.dev(G), d_out)
    want = H64.T @ G.astype(np.float64)
    assert_close(gW.cpu().numpy(), want, what="weight gradient")
    assert norm_error(gW.cpu().numpy().astype(np.float64), want) <= 2.0 ** -24 * 8 * max(1.0, np.sqrt(n / 16.0))


@pytest.mark.parametrize("k", [2, 14, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97, 112, 127])
@pytest.mark.parametrize("width", [5, 40, 100, 190, 256])
def test_every_number_of_tiles_along_k(k, width):
    # whole and partial last tiles behind none to eight others: the steady loop, its end and the tiles fetched ahead; the
    # same number of nodes behind a weight gradient
    H, W = wl.random_matrix(260, k, k + width, ld=k + 1), wl.random_matrix(k, width, width)
    H[:, k:] = np.nan
    Z = Hn.transform(Hn.dev(H), k, Hn.dev(W), None, False).cpu().numpy()[:, :width].astype(np.float64)
    want = H[:, :k].astype(np.float64) @ W.astype(np.float64)
    assert norm_error(Z, want) <= 2.0 ** -24 * 8 * max(1.0, np.sqrt(k / 16.0))
    P, G = wl.random_matrix(k, 150, 3, ld=151), wl.random_matrix(k, width, 5)
    gW = Hn.transform_backward(Hn.dev(P), 150, Hn.dev(G), width)[0].cpu().numpy().astype(np.float64)
    want = P[:, :150].astype(np.float64).T @ G.astype(np.float64)
    assert norm_error(gW, want) <= 2.0 ** -24 * 8 * max(1.0, np.sqrt(k / 16.0))


def test_infinities_nan_and_overflow_come_out_as_float32_sums_give_them():
    n, d_in, d_out = 300, 40, 70
    H = wl.random_matrix(n, d_in, 3)
    W = wl.random_matrix(d_in, d_out, 4)
    W[7] = 0.0                                 # inf * 0 is NaN
    H[5, 3] = np.inf
    H[130, 0] = -np.inf
    H[131, 7] = np.inf
    H[200, 39] = np.nan
    H[250, 10], H[250, 11] = 3.4e38, 3.4e38    # rounds to infinity in bf16; the sums overflow where W adds up past one
    H[260, 12] = 3.3999e38                     # rounds to infinity in bf16; times a weight below one it is a number
    Z = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), None, False).cpu().numpy()[:, :d_out]
    with np.errstate(all="ignore"):
        want = H.astype(np.float64) @ W.astype(np.float64)
        w32 = want.astype(np.float32)
    for r in (5, 130, 131, 200):
        assert np.array_equal(np.isnan(Z[r]), np.isnan(want[r])) and np.array_equal(Z[r][np.isinf(want[r])], w32[r][np.isinf(want[r])])
    sure = np.abs(want[250]) > 6e38
    assert np.array_equal(Z[250][sure], np.sign(want[250][sure]) * np.float32(np.inf))
    keep = np.abs(want[260]) < 3e38
    assert keep.any() and np.abs(Z[260][keep] / want[260][keep] - 1).max() < 1e-5
    rest = np.setdiff1d(np.arange(n), (5, 130, 131, 200, 250, 260))
    assert_close(Z[rest], want[rest], what="rows of the same tiles")
    # the weight gradient sums over the rows: a bad row reaches every output of its column
    G = wl.random_matrix(n, d_out, 6)
    gW, _ = Hn.transform_backward(Hn.dev(H[:, :3]), 3, Hn.dev(G), d_out)
    with np.errstate(all="ignore"):
        want = H[:, :3].astype(np.float64).T @ G.astype(np.float64)
    got = gW.cpu().numpy()
    assert np.array_equal(got[0], want[0].astype(np.float32)) and np.all(np.isinf(got[0]))
    assert_close(got[1:], want[1:], what="columns without a bad value")


@pytest.mark.parametrize("scale_h,scale_w", [(-118, 0), (-60, -60), (0, -122), (-126, 20), (100, 20), (-100, 110)])
def test_scales_at_the_ends_of_the_range(scale_h, scale_w):
    # operands and results towards the ends of float32's range: float32 holds 24 bits of them (results of 2^-120 and more
    # here), so the bound stays the one of ordinary rows
    n, d_in, d_out = 200, 50, 40
    H = np.ldexp(wl.random_matrix(n, d_in, 8), scale_h)
    W = np.ldexp(wl.random_matrix(d_in, d_out, 9), scale_w)
    Z = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), None, False).cpu().numpy()[:, :d_out].astype(np.float64)
    want = H.astype(np.float64) @ W.astype(np.float64)
    s = np.ldexp(1.0, -(scale_h + scale_w))
    assert_close(Z * s, want * s, what="scales 2^%d, 2^%d" % (scale_h, scale_w))


@pytest.mark.parametrize("scale_h,scale_w", [(-118, 40), (-120, 30), (-124, 40), (-126, 60), (-130, 100), (-143, 100),
                                             (40, -124), (30, -120), (100, -140)])
def test_small_operands_beside_large_ones_keep_all_their_bits(scale_h, scale_w):
    # an operand far below the range in which bf16 keeps three parts, lifted by its partner to an ordinary sum (smaller
    # than float32's normal range at (-130, 100), (-143, 100): the operand then has fewer bits, and these count)
    n, d_in, d_out = 200, 50, 40
    H = np.ldexp(wl.random_matrix(n, d_in, 8), scale_h)
    W = np.ldexp(wl.random_matrix(d_in, d_out, 9), scale_w)
    H64, s = H.astype(np.float64), np.ldexp(1.0, -(scale_h + scale_w))
    Z = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), None, False).cpu().numpy()[:, :d_out].astype(np.float64)
    want = H64 @ W.astype(np.float64)
    assert_close(Z * s, want * s, what="forward, scales 2^%d, 2^%d" % (scale_h, scale_w))
    assert norm_error(Z * s, want * s) <= 2.0 ** -24 * 8 * np.sqrt(d_in / 16.0)
    G = np.ldexp(wl.random_matrix(n, d_out, 5), scale_w)
    gW = Hn.transform_backward(Hn.dev(H), d_in, Hn.dev(G), d_out)[0].cpu().numpy().astype(np.float64)
    want = H64.T @ G.astype(np.float64)
    assert_close(gW * s, want * s, what="weight gradient, scales 2^%d, 2^%d" % (scale_h, scale_w))
    assert norm_error(gW * s, want * s) <= 2.0 ** -24 * 8 * np.sqrt(n / 16.0)


@pytest.mark.parametrize("n,d_out", [(1, 1), (130, 33), (300, 257)])
def test_single_products_are_rounded_once(n, d_out):
    # one input column, and the gradient of one node: float32 products, each correctly rounded
    H, W = wl.random_matrix(n, 1, 21), wl.random_matrix(1, d_out, 22)
    Z = Hn.transform(Hn.dev(H), 1, Hn.dev(W), None, False).cpu().numpy()[:, :d_out]
    assert np.array_equal(Z, H[:, :1] * W)
    x, g = wl.random_matrix(1, 300, 23, ld=300), wl.random_matrix(1, d_out, 24)
    gW = Hn.transform_backward(Hn.dev(x), 300, Hn.dev(g), d_out)[0].cpu().numpy()
    assert np.array_equal(gW, x.T * g)


def test_zero_rows_stay_zero_and_small_terms_do_not_disturb():
    n, d_in, d_out = 260, 48, 33
    H = wl.random_matrix(n, d_in, 10)
    H[3] = 0.0
    H[140:150] = 0.0
    H[200, ::2] = 1e-38                        # terms far below the others of their row
    W = wl.random_matrix(d_in, d_out, 11)
    Z = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), None, False).cpu().numpy()[:, :d_out]
    assert np.all(Z[3] == 0) and np.all(Z[140:150] == 0)
    assert_close(Z, H.astype(np.float64) @ W.astype(np.float64), what="small terms")


def test_weight_gradient_over_many_chunks_does_not_drift():
    # thousands of row chunks with partial sums of one sign: what each chunk's rounding leans to must not add up
    n = 400_000
    g = torch.Generator(device="cuda").manual_seed(3)
    H = torch.rand((n, 32), generator=g, device="cuda") + 0.5
    G = torch.rand((n, 16), generator=g, device="cuda") + 0.5
    gW, gb = Hn.transform_backward(H, 32, G, 16)
    want = (H.double().T @ G.double()).cpu().numpy()
    # one rounding per addition and chunk at worst: 2^-24 of a sum that the next chunk carries on
    assert np.abs(gW.cpu().numpy() / want - 1).max() < 2e-6
    assert np.abs(gb.cpu().numpy() / G.double().sum(0).cpu().numpy() - 1).max() < 2e-6
    assert B.retexo_transform_backward_workspace_bytes(n, 32, 16) > 0


def test_training_decides_units_near_zero_by_the_float32_sum():
    # half the rows cancel to within rounding of zero in every unit; which units are on is the float32 sum's decision, k
    # ascending, and a wrong one moves a whole unit of a node
    n, d_in, hid, cls = 300, 50, 64, 5
    B.check(B.retexo_set_option("transform_few_blocks", 0), "set_option")
    rng = np.random.Generator(np.random.Philox(key=17))
    X = rng.standard_normal((n, d_in), dtype=np.float32)
    W1 = (rng.standard_normal((d_in, hid), dtype=np.float32) / 8).astype(np.float32)
    W1[d_in // 2:] = -W1[:d_in // 2]
    X[::2, d_in // 2:] = X[::2, :d_in // 2] * (1 + rng.integers(-1, 2, (n // 2, d_in // 2)) * np.float32(2.0 ** -23)).astype(np.float32)
    b1 = np.zeros(hid, np.float32)
    Wc = rng.standard_normal((hid, cls), dtype=np.float32)
    bc = np.zeros(cls, np.float32)
    y = rng.integers(0, cls, n).astype(np.int32)
    acc = np.zeros((n, hid), np.float32)
    for k in range(d_in):                      # a product of two float32 is exact in 64 bits: one rounding per step
        acc = (acc.astype(np.float64) + X[:, k:k + 1].astype(np.float64) * W1[k].astype(np.float64)).astype(np.float32)
    on = acc > 0
    exact = X.astype(np.float64) @ W1.astype(np.float64)
    assert 0.02 < np.mean(on != (exact > 0)) < 0.4         # the decisions differ from the exact sums' in many units
    A = np.where(on, exact, 0.0)
    L = A @ Wc.astype(np.float64)
    P = np.exp(L - L.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    P[np.arange(n), y] -= 1.0
    dA = np.where(on, (P / n) @ Wc.astype(np.float64).T, 0.0)
    d = Hn.dev
    _, gW1, gb1, _, _ = Hn.layer_grad(d(X), d_in, d(y), d(W1), d(b1), d(Wc), d(bc))
    assert_close(gW1.cpu().numpy(), X.astype(np.float64).T @ dA, what="gW1")
    assert_close(gb1.cpu().numpy()[None, :], dA.sum(0)[None, :], what="gb1")


def test_weight_gradient_of_a_large_first_layer_against_64_bits():
    # 1204 x 256 outputs over 232,965 nodes, a thousand chunks' partial sums: the measured training step's first gradient,
    # without the unit decisions that keep that one from having a value in 64 bits
    n, d_in, d_out = 232965, 1204, 256
    g = torch.Generator(device="cuda").manual_seed(11)
    X = torch.empty((n, 1216), device="cuda").normal_(generator=g)
    G = torch.empty((n, d_out), device="cuda").normal_(generator=g) * 1e-3
    gW, gb = Hn.transform_backward(X, d_in, G, d_out)
    want = torch.zeros((d_in, d_out), dtype=torch.float64, device="cuda")
    for i in range(0, n, 20000):
        want += X[i:i + 20000, :d_in].double().T @ G[i:i + 20000].double()
    # a chunk's float32 sum of 2,300 products and the sum of a hundred chunks: about sqrt(2,300) roundings of 2^-25 each
    assert float((gW.double() - want).norm() / want.norm()) <= 48 * 2.0 ** -25
    assert float((gW.double() - want).abs().max() / want.pow(2).mean().sqrt()) <= 6 * 48 * 2.0 ** -25
    assert float((gb.double() - G.double().sum(0)).norm() / G.double().sum(0).norm()) <= 48 * 2.0 ** -25
