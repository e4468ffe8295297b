"""Training steps in which many hidden units lie near zero, or some are not finite: which units are on is the float32
sum's decision, and forming those sums again stays a small part of the step."""
import numpy as np
import pytest
import torch

from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close

pytestmark = pytest.mark.gpu

N, D_IN, HIDDEN, CLASSES = 16384, 512, 64, 5          # 128 blocks of 128 rows: the block kernel's


def step(change=lambda X, W1: None):
    """A step's inputs, with `change` made to them -> a call that takes the step."""
    rng = np.random.Generator(np.random.Philox(key=5))
    X = wl.random_matrix(N, D_IN, 31)
    W1 = wl.glorot(rng, D_IN, HIDDEN, (D_IN, HIDDEN))
    Wc = wl.glorot(rng, HIDDEN, CLASSES, (HIDDEN, CLASSES))
    y = rng.integers(0, CLASSES, N).astype(np.int32)
    change(X, W1)
    d = Hn.dev
    X, y, W1, Wc = d(X), d(y), d(W1), d(Wc)
    b1, bc = torch.zeros(HIDDEN, device="cuda"), torch.zeros(CLASSES, device="cuda")
    return lambda: Hn.layer_grad(X, D_IN, y, W1, b1, Wc, bc)


def best_time(call):
    call()
    times = []
    for _ in range(9):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        call()
        stop.record()
        stop.synchronize()
        times.append(start.elapsed_time(stop))
    return min(times)


@pytest.fixture(scope="module")
def ordinary():
    return best_time(step())


def infinite_input(X, W1):
    X[100, 3] = np.inf


def overflowing_row(X, W1):
    X[100] = np.where(X[100] > 0, 3e38, -3e38)          # finite inputs whose sums are not


@pytest.mark.parametrize("change", [infinite_input, overflowing_row])
def test_a_sum_that_is_not_finite_costs_no_other_its_time(ordinary, change):
    # a wave's 1,024 or more sums formed again one at a time take milliseconds; the step takes about a tenth of one
    assert best_time(step(change)) < 4 * ordinary


def weak_units(X, W1):
    W1[:, ::2] *= np.float32(1e-6)


def rows_of_all_sizes(X, W1):
    X *= (10.0 ** np.linspace(-6, 6, N)[np.random.Generator(np.random.Philox(key=8)).permutation(N)]).astype(np.float32)[:, None]


@pytest.mark.parametrize("change", [weak_units, rows_of_all_sizes])
def test_units_and_rows_small_beside_the_others_are_not_all_near_zero(ordinary, change):
    # half the units with weights far below the others': formed again one at a time, their sums took fifty steps' time
    assert best_time(step(change)) < 4 * ordinary


@pytest.mark.parametrize("weak", [0, -20])
def test_near_zero_units_are_on_where_the_float32_sum_is_positive(weak):
    # mirrored inputs: half the rows cancel to within rounding of zero in every unit; half the units' weights are 2^weak of
    # the others'.  float32 sums with k ascending decide, and a wrong decision moves a whole unit of a node.
    n, d_in, hid, cls = 300, 50, 64, 5
    rng = np.random.Generator(np.random.Philox(key=17))
    X = rng.standard_normal((n, d_in), dtype=np.float32)
    W1 = (rng.standard_normal((d_in, hid), dtype=np.float32) / 8).astype(np.float32)
    W1[d_in // 2:] = -W1[:d_in // 2]
    W1[:, ::2] *= np.float32(2.0 ** weak)
    jitter = rng.integers(-1, 2, (n // 2, d_in // 2)) * np.float32(2.0 ** -23)
    X[::2, d_in // 2:] = X[::2, :d_in // 2] * (1 + jitter).astype(np.float32)
    Wc = rng.standard_normal((hid, cls), dtype=np.float32)
    y = rng.integers(0, cls, n).astype(np.int32)
    acc = np.zeros((n, hid), np.float32)
    for k in range(d_in):                      # a product of two float32 is exact in 64 bits: one rounding per step
        acc = (acc.astype(np.float64) + X[:, k:k + 1].astype(np.float64) * W1[k].astype(np.float64)).astype(np.float32)
    on = acc > 0
    exact = X.astype(np.float64) @ W1.astype(np.float64)
    assert 0.02 < np.mean(on != (exact > 0)) < 0.4         # the decisions differ from the exact sums' in many units
    L = np.where(on, exact, 0.0) @ Wc.astype(np.float64)
    P = np.exp(L - L.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    P[np.arange(n), y] -= 1.0
    dA = np.where(on, (P / n) @ Wc.astype(np.float64).T, 0.0)
    d, zero = Hn.dev, lambda k: torch.zeros(k, device="cuda")
    B.check(B.retexo_set_option("transform_few_blocks", 0), "set_option")
    try:
        _, gW1, gb1, _, _ = Hn.layer_grad(d(X), d_in, d(y), d(W1), zero(hid), d(Wc), zero(cls))
    finally:
        B.check(B.retexo_set_option("transform_few_blocks", 128), "set_option")
    assert_close(gW1.cpu().numpy(), X.astype(np.float64).T @ dA, what="gW1")
    assert_close(gb1.cpu().numpy()[None, :], dA.sum(0)[None, :], what="gb1")


def test_units_whose_products_cancel_exactly_are_off():
    # two equal inputs with opposite weights: zero, where a chain of float32 multiply-adds would leave the rounding of the
    # first product, positive about half the time
    n, hid, cls = 300, 64, 5
    rng = np.random.Generator(np.random.Philox(key=18))
    X = np.repeat(rng.standard_normal((n, 1), dtype=np.float32), 2, axis=1)
    W1 = np.repeat(rng.standard_normal((1, hid), dtype=np.float32), 2, axis=0)
    W1[1] = -W1[1]
    W1[:, ::2] = np.abs(W1[:, ::2])                        # every second unit is an ordinary one (of two equal weights)
    on = X.astype(np.float64) @ W1.astype(np.float64) > 0
    assert 0 < on.mean() < 0.5
    Wc = rng.standard_normal((hid, cls), dtype=np.float32)
    y = rng.integers(0, cls, n).astype(np.int32)
    L = np.where(on, X.astype(np.float64) @ W1.astype(np.float64), 0.0) @ Wc.astype(np.float64)
    P = np.exp(L - L.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    P[np.arange(n), y] -= 1.0
    dA = np.where(on, (P / n) @ Wc.astype(np.float64).T, 0.0)
    d, zero = Hn.dev, lambda k: torch.zeros(k, device="cuda")
    B.check(B.retexo_set_option("transform_few_blocks", 0), "set_option")
    try:
        _, gW1, gb1, _, _ = Hn.layer_grad(d(X), 2, d(y), d(W1), zero(hid), d(Wc), zero(cls))
    finally:
        B.check(B.retexo_set_option("transform_few_blocks", 128), "set_option")
    assert_close(gW1.cpu().numpy(), X.astype(np.float64).T @ dA, what="gW1")
    assert_close(gb1.cpu().numpy()[None, :], dA.sum(0)[None, :], what="gb1")


def test_an_infinite_input_leaves_the_weight_gradient_its_time():
    # the tiles it reaches are formed by the float32 instruction, over two thousand nodes each: 2.1 to 2.2 times the time of
    # the ordinary call, 3.0 with one pair of nodes in flight
    n, d_in, d_out = 232965, 1204, 256
    H, G = torch.randn((n, 1216), device="cuda"), torch.randn((n, d_out), device="cuda")
    ws = Hn.ws_tensor(B.retexo_transform_backward_workspace_bytes(n, d_in, d_out))
    call = lambda: Hn.transform_backward(H, d_in, G, d_out, ws)
    ordinary = best_time(call)
    H[n // 2, 7] = np.inf
    assert best_time(call) < 2.75 * ordinary
