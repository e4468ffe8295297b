"""Sum, mean, gcn_sym and edge softmax over 16-bit tables, several rows (or shares of a long row) per wave: one lane count after the other, rows
that end with a lane's batch, a group or a tile of the walk, empty rows, long rows shared by a workgroup, slabs with a last one
that is not full, rows padded or, at 4-byte addresses, with their last eight columns over the ones before them."""
import numpy as np
import pytest
import torch

import oracle
from oracle import storage as ost
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close, assert_cond_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graphs():
    src, dst, at = [], [], 600
    for c, d in enumerate((15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 7, 8, 9)):
        for leaf in range(d):
            src.append(c), dst.append(20 + (at + leaf) % 1000)
        at += d
    specs = {"edges": (1027, np.array(src, np.int32), np.array(dst, np.int32)),
             "skewed": (9001, *wl.random_pairs(9001, 40000, 2, skew=3.0)),
             "dense": (3001, *wl.random_pairs(3001, 180000, 3, skew=0.5))}
    out = {}
    for name, (n, s, d) in specs.items():
        out[name] = (Hn.make_plan(Hn.csr_from_coo(Hn.dev(s), Hn.dev(d), n, False)), *oracle.csr_from_coo(s, d, n, False))
    assert (np.diff(out["edges"][1]) == 0).any() and np.diff(out["skewed"][1]).max() > 1000
    yield out
    for g, _, _ in out.values():
        g.destroy()


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("name", ["edges", "skewed", "dense"])
@pytest.mark.parametrize("F,ld,offset", [(1, 8, 0), (8, 8, 0), (31, 32, 0), (32, 34, 2), (33, 40, 0), (64, 64, 0), (50, 50, 0),
                                         (65, 72, 0), (130, 130, 2), (200, 200, 0), (300, 302, 0), (602, 602, 0)])
def test_stored_row_groups(graphs, name, fmt, F, ld, offset):
    g, rp, ci = graphs[name]
    n = g.n_nodes
    Zh = wl.random_matrix(n, F, F)
    bits = ost.store(Zh, fmt)
    stored = ost.load(bits, fmt)
    # what lies between the rows (NaN) must not reach a result; but where rows hold whole vectors the table ends with its last
    # row's last column
    padded = ld % 8 == 0 and offset % 8 == 0
    buf = torch.full((offset + (n - 1) * ld + (ld if padded else F),), -1, dtype=torch.int16, device="cuda")
    Z = torch.as_strided(buf, (n, F), (ld, 1), offset)
    Z.copy_(torch.from_numpy(bits.view(np.int16)))
    for mode in ("sum", "mean", "gcn_sym"):
        out = torch.full((n, 2 * F + 1), 777.0, device="cuda")
        got = Hn.aggregate_stored(g, mode, Z, F, fmt, concat=True, out=out).cpu().numpy()
        want = oracle.aggregate(mode, rp, ci, stored, F, self_concat=True)
        assert_cond_close(got[:, :2 * F], want, oracle.aggregate_abs(mode, rp, ci, stored, F, self_concat=True), what=mode)
        assert np.array_equal(got[:, :F].astype(np.float64), want[:, :F]) and np.all(got[:, 2 * F:] == 777.0)


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("name", ["edges", "skewed", "dense"])
@pytest.mark.parametrize("heads,dh,pad", [(1, 4, 0), (3, 8, 8), (8, 4, 0), (1, 64, 0), (3, 16, 0), (5, 16, 4), (2, 64, 0),
                                          (1, 256, 0), (3, 64, 8), (8, 32, 0)])
def test_stored_softmax_row_groups(graphs, name, fmt, heads, dh, pad):
    """Groups of 8, 16, 32 and 64 lanes, full and not, the smallest and largest heads in each."""
    g, rp, ci = graphs[name]
    n, F = g.n_nodes, heads * dh
    ld = -(-F // 8) * 8 + pad
    Zh = wl.random_matrix(n, F, F)
    bits = np.full((n, ld), -1, np.int16)                     # NaN between the rows
    bits[:, :F] = ost.store(Zh, fmt).view(np.int16)
    stored = ost.load(ost.store(Zh, fmt), fmt)
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.3) for k in (1, 2)]
    out = torch.full((n, 2 * F + 1), 777.0, device="cuda")
    kw = dict(heads=heads, a_src=Hn.dev(a[0]), a_dst=Hn.dev(a[1]))
    got = Hn.aggregate_stored(g, "gat_softmax", torch.from_numpy(bits).cuda(), F, fmt, concat=True, out=out, **kw).cpu().numpy()
    okw = dict(heads=heads, a_src=a[0], a_dst=a[1], self_concat=True)
    want = oracle.aggregate("gat_softmax", rp, ci, stored, F, **okw)
    assert_cond_close(got[:, :2 * F], want, oracle.aggregate_abs("gat_softmax", rp, ci, stored, F, **okw), what="softmax")
    if F >= 64:
        assert_close(got[:, :2 * F], want, what="softmax, row by row")
    assert np.array_equal(got[:, :F].astype(np.float64), want[:, :F]) and np.all(got[:, 2 * F:] == 777.0)


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("name", ["edges", "skewed", "dense"])
@pytest.mark.parametrize("heads,dh", [(1, 4), (8, 4), (3, 8), (5, 16), (2, 32), (8, 32), (3, 64), (2, 128), (1, 256)])
@pytest.mark.parametrize("how", ["offsets", "vector"])
def test_stored_softmax_one_row_per_wave(graphs, name, fmt, heads, dh, how):
    """What row groups do not take: rows with 64-bit offsets (tables of 4 GiB and more) and a destination vector that is not at a
    16-byte address; every width of a head."""
    g, rp, ci = graphs[name]
    n, F = g.n_nodes, heads * dh
    ld = -(-F // 8) * 8
    Zh = wl.random_matrix(n, F, F + 1)
    bits = np.full((n, ld), -1, np.int16)                     # NaN between the rows
    bits[:, :F] = ost.store(Zh, fmt).view(np.int16)
    stored = ost.load(ost.store(Zh, fmt), fmt)
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.3) for k in (1, 2)]
    vector = torch.zeros(F + 1, device="cuda")[1:].view(heads, dh) if how == "vector" else torch.zeros((heads, dh), device="cuda")
    vector.copy_(torch.from_numpy(a[1]))
    out = torch.full((n, 2 * F + 1), 777.0, device="cuda")
    try:
        B.check(B.retexo_set_option("agg_wide_offsets", 1 if how == "offsets" else 0), "set_option")
        Hn.aggregate_stored(g, "gat_softmax", torch.from_numpy(bits).cuda(), F, fmt, concat=True, out=out, heads=heads,
                            a_src=Hn.dev(a[0]), a_dst=vector)
    finally:
        B.check(B.retexo_set_option("agg_wide_offsets", 0), "set_option")
    got = out.cpu().numpy()
    okw = dict(heads=heads, a_src=a[0], a_dst=a[1], self_concat=True)
    want = oracle.aggregate("gat_softmax", rp, ci, stored, F, **okw)
    assert_cond_close(got[:, :2 * F], want, oracle.aggregate_abs("gat_softmax", rp, ci, stored, F, **okw), what="softmax")
    assert np.array_equal(got[:, :F].astype(np.float64), want[:, :F]) and np.all(got[:, 2 * F:] == 777.0)
