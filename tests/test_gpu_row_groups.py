"""Narrow rows, several rows of the schedule (or shares of a long row) per wave: edge softmax forward, save mode and the backward
after it, and sum, mean and gcn_sym, whose wider rows are walked in slabs, against the fp64 oracle.  Rows that end with a wave, a group or a tile of the walk (32 and 64 entries), row
counts that leave groups without a row, empty rows, long rows shared by a workgroup, rows padded or not."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close, assert_cond_close
from test_gpu_softmax_rows import decided_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graphs():
    """few: below the line from which the plain forward takes the kernel; edges: rows of 31 to 33, 63 to 65 and 127 to 129
    entries, and the row of their centres; skewed: most of 16,501 rows short, some empty, one of thousands of entries"""
    src, dst, at = [], [], 600
    for c, d in enumerate((31, 32, 33, 63, 64, 65, 127, 128, 129, 4, 5, 8, 9)):
        for leaf in range(d):
            src.append(c), dst.append(20 + (at + leaf) % 1000)
        at += d
    ring = np.arange(1021)
    for k in range(1, 9):
        src.extend(20 + ring[:1000]), dst.extend(20 + (ring[:1000] + 7 * k) % 1000)
    specs = {"few": (1003, *wl.random_pairs(1003, 5000, 1, skew=1.0)),
             "edges": (1030, np.array(src, np.int32), np.array(dst, np.int32)),
             "skewed": (16501, *wl.random_pairs(16501, 60000, 2, skew=3.0)),
             "dense": (9001, *wl.random_pairs(9001, 400000, 3, skew=0.5)),
             "mid": (17003, *wl.random_pairs(17003, 190000, 4, skew=0.5))}
    out = {}
    for name, (n, s, d) in specs.items():
        g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(s), Hn.dev(d), n, False))
        out[name] = (g, *oracle.csr_from_coo(s, d, n, False))
    assert out["few"][1][-1] < 16384 <= out["edges"][1][-1]
    assert (np.diff(out["skewed"][1]) == 0).any() and np.diff(out["skewed"][1]).max() > 2000
    yield out
    for g, _, _ in out.values():
        g.destroy()


@pytest.mark.parametrize("name", ["few", "edges", "skewed"])
@pytest.mark.parametrize("heads,dh,pad", [(1, 4, 0), (8, 4, 0), (3, 8, 8), (1, 32, 0), (3, 16, 0), (8, 8, 4), (1, 64, 0),
                                          (3, 32, 0), (8, 16, 0), (8, 32, 0)])
def test_row_groups(graphs, name, heads, dh, pad):
    g, rp, ci = graphs[name]
    n, F = g.n_nodes, heads * dh
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Zh = decided_rows(rp, ci, heads, dh, a)[:, :F]
    Zh = np.ascontiguousarray(np.pad(Zh, ((0, 0), (0, pad)), constant_values=np.nan))      # padding that must not be read
    Gh = wl.random_matrix(n, F, F + 1)
    Z, G, As, Ad = (Hn.dev(x) for x in (Zh, Gh, *a))
    kw = dict(heads=heads, a_src=As, a_dst=Ad)
    plain = Hn.aggregate(g, "gat_softmax", Z, F, **kw)
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
    out = Hn.aggregate(g, "gat_softmax", Z, F, workspace=ws, save=True, **kw)
    got = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, saved=ws, **kw)
    okw = dict(heads=heads, a_src=a[0], a_dst=a[1])
    fwd = oracle.aggregate("gat_softmax", rp, ci, Zh[:, :F], F, **okw)
    want = oracle.aggregate_backward("gat_softmax", rp, ci, Zh[:, :F], F, Gh, **okw)
    assert_close(plain.cpu().numpy()[:, :F], fwd, what="forward")
    assert_close(out.cpu().numpy()[:, :F], fwd, what="save mode")
    # rows of a few columns have no robust magnitude: one ratio over all rows
    assert_close(got[0].cpu().numpy()[:, :F].reshape(1, -1), want[0].reshape(1, -1), what="backward")
    if F >= 64:
        assert_close(got[0].cpu().numpy()[:, :F], want[0], what="backward, row by row")
    for grad, ref, what in zip(got[1:], want[1:], ("source", "destination")):
        assert_close(grad.cpu().numpy().reshape(1, -1), ref.reshape(1, -1), what=what + " attention vector")


@pytest.mark.parametrize("name,F", [("few", 1), ("few", 33), ("edges", 3), ("edges", 32), ("edges", 45), ("edges", 64), ("skewed", 8),
                                    ("skewed", 31), ("skewed", 61), ("dense", 30), ("dense", 64), ("dense", 125), ("dense", 250),
                                    ("mid", 200), ("mid", 185), ("mid", 602)])
@pytest.mark.parametrize("mode", ["sum", "mean", "gcn_sym"])
def test_linear(graphs, name, F, mode):
    """One group size and slab count after the other: 8 lanes, 16, slabs of 32 lanes ("dense", 250: two) and of 16 ("mid" without
    weights: four, three with a last one of 57 columns, and ten), beside whole rows in slabs of 256 columns ("mid" with weights)."""
    g, rp, ci = graphs[name]
    n, ld = g.n_nodes, (F + 3) // 4 * 4
    Zh = np.full((n, ld + 4), np.nan, np.float32)             # what lies past a row is fetched with its last vector, and no more
    Zh[:, :F] = wl.random_matrix(n, F, F)
    out = Hn.aggregate(g, mode, Hn.dev(Zh), F, concat=F % 2 == 1, ld_out=2 * F + 3)
    got = out.cpu().numpy()
    kw = dict(self_concat=F % 2 == 1)
    want = oracle.aggregate(mode, rp, ci, Zh[:, :F], F, **kw)
    assert_cond_close(got[:, :want.shape[1]], want, oracle.aggregate_abs(mode, rp, ci, Zh[:, :F], F, **kw), what=mode)
    again = Hn.aggregate(g, mode, Hn.dev(Zh), F, concat=F % 2 == 1, ld_out=2 * F + 3).cpu().numpy()
    assert np.array_equal(got[:, :want.shape[1]], again[:, :want.shape[1]])


@pytest.mark.parametrize("name", ["few", "edges", "skewed"])
@pytest.mark.parametrize("F,ld,offset", [(4, 5, 1), (5, 5, 0), (7, 7, 2), (31, 31, 1), (33, 34, 0), (45, 45, 3), (48, 49, 0), (49, 49, 0)])
def test_linear_unpadded(graphs, name, F, ld, offset):
    """Rows at any float's address whose last four columns lie over the ones before them; the table ends with its last row's last
    column, and what lies between the rows must not reach a sum."""
    g, rp, ci = graphs[name]
    n = g.n_nodes
    Zh = np.full((n, ld), np.nan, np.float32)
    Zh[:, :F] = wl.random_matrix(n, F, F)
    buf = torch.zeros(offset + (n - 1) * ld + F, device="cuda")
    Z = torch.as_strided(buf, (n, F), (ld, 1), offset)
    Z.copy_(torch.from_numpy(Zh[:, :F].copy()))
    for mode in ("sum", "mean", "gcn_sym"):
        out = torch.full((n, 2 * F + 1), 777.0, device="cuda")
        got = Hn.aggregate(g, mode, Z, F, concat=True, out=out).cpu().numpy()
        want = oracle.aggregate(mode, rp, ci, Zh[:, :F], F, self_concat=True)
        mag = oracle.aggregate_abs(mode, rp, ci, Zh[:, :F], F, self_concat=True)
        assert_cond_close(got[:, :2 * F], want, mag, what=mode)
        assert np.array_equal(got[:, :F], Zh[:, :F]) and np.all(got[:, 2 * F:] == 777.0)


@pytest.mark.parametrize("n,entries,F", [(52433, 59, 20), (52433, 59, 25), (52433, 59, 37), (70001, 132, 12), (150017, 164, 9)])
def test_linear_over_flat_graphs(n, entries, F):
    """Nodes of nearly equal degrees, padded rows that are not whole lines: in ranges or in row groups."""
    src, dst = wl.random_pairs(n, n * entries // 2, 6, skew=0.0)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False))
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    ld = (F + 3) // 4 * 4
    Zh = np.full((n, ld), np.nan, np.float32)
    Zh[:, :F] = wl.random_matrix(n, F, F)
    for mode in ("mean", "gcn_sym"):
        got = Hn.aggregate(g, mode, Hn.dev(Zh), F, concat=True, ld_out=2 * F + 3).cpu().numpy()
        want = oracle.aggregate(mode, rp, ci, Zh[:, :F], F, self_concat=True)
        mag = oracle.aggregate_abs(mode, rp, ci, Zh[:, :F], F, self_concat=True)
        assert_cond_close(got[:, :2 * F], want, mag, what=mode)
    g.destroy()


@pytest.mark.parametrize("heads,dh", [(4, 64), (5, 32), (2, 64)])
def test_slabs_of_heads(heads, dh):
    """Rows of several slabs (of one head; of two heads with a last one of one): 50,001 nodes of 180
    entries, one row of thousands."""
    n, F = 50001, heads * dh
    src, dst = wl.random_pairs(n, 4700000, 5, skew=1.2)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False))
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    assert rp[-1] >= 48 * n and n * F * 4 >= 24 << 20 and rp[-1] * F * 4 >= 4 << 30
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Zh = wl.random_matrix(n, F, 7)
    kw = dict(heads=heads, a_src=Hn.dev(a[0]), a_dst=Hn.dev(a[1]), concat=True)
    Z = Hn.dev(Zh)
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
    want = oracle.aggregate("gat_softmax", rp, ci, Zh, F, heads=heads, a_src=a[0], a_dst=a[1], self_concat=True)
    for what, save in (("forward", {}), ("save mode", dict(save=True, workspace=ws))):
        assert_close(Hn.aggregate(g, "gat_softmax", Z, F, **kw, **save).cpu().numpy()[:, :2 * F], want, what=what)
    g.destroy()


@pytest.mark.parametrize("heads,dh", [(4, 64), (5, 32), (2, 64)])
def test_backward_from_the_state_of_slabs(heads, dh):
    """What save mode leaves in slabs of heads: statistics of every slab's heads and of the padded ones, positive and negative parts
    at their columns.  Values and vectors are small multiples of 1/8 and 1/32, so that a score is exact and has the same sign
    here and in the oracle."""
    n, F = 50001, heads * dh
    src, dst = wl.random_pairs(n, 4700000, 5, skew=1.2)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False))
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    assert rp[-1] >= 48 * n and n * F * 4 >= 24 << 20 and rp[-1] * F * 4 >= 4 << 30
    a = [np.rint(wl.random_matrix(heads, dh, k) * 4).astype(np.float32) / 32 for k in (1, 2)]
    Zh, Gh = np.rint(wl.random_matrix(n, F, 7) * 8).astype(np.float32) / 8, wl.random_matrix(n, F, 8)
    kw = dict(heads=heads, a_src=Hn.dev(a[0]), a_dst=Hn.dev(a[1]))
    Z = Hn.dev(Zh)
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
    Hn.aggregate(g, "gat_softmax", Z, F, save=True, workspace=ws, **kw)
    got = Hn.aggregate_backward(g, "gat_softmax", F, Hn.dev(Gh), Z=Z, saved=ws, **kw)
    want = oracle.aggregate_backward("gat_softmax", rp, ci, Zh, F, Gh, heads=heads, a_src=a[0], a_dst=a[1])
    assert_close(got[0].cpu().numpy()[:, :F], want[0], what="gradient of Z")
    for grad, ref, what in zip(got[1:], want[1:], ("source", "destination")):
        assert_close(grad.cpu().numpy(), ref, what=what + " attention vector, head by head")
    g.destroy()


@pytest.mark.parametrize("name", ["few", "edges", "skewed"])
@pytest.mark.parametrize("heads,dh", [(1, 4), (8, 4), (3, 8), (1, 32), (3, 16)])
def test_backward_of_narrow_rows_by_length(graphs, name, heads, dh):
    """Rows of a few columns have no robust magnitude of their own: one ratio over the rows of similar length, so that the long
    ones, whose gradients are the largest, hide no error in the short ones."""
    g, rp, ci = graphs[name]
    n, F = g.n_nodes, heads * dh
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Zh = np.ascontiguousarray(decided_rows(rp, ci, heads, dh, a)[:, :F])
    Gh = wl.random_matrix(n, F, F + 2)
    Z, G, As, Ad = (Hn.dev(x) for x in (Zh, Gh, *a))
    kw = dict(heads=heads, a_src=As, a_dst=Ad)
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
    Hn.aggregate(g, "gat_softmax", Z, F, workspace=ws, save=True, **kw)
    want = oracle.aggregate_backward("gat_softmax", rp, ci, Zh, F, Gh, heads=heads, a_src=a[0], a_dst=a[1])[0]
    deg = np.diff(rp)
    for what, saved in (("plain", None), ("saved", ws)):
        got = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, saved=saved, **kw)[0].cpu().numpy()[:, :F]
        for lo, hi in ((0, 1), (1, 2), (2, 5), (5, 9), (9, 17), (17, 33), (33, 129), (129, 1025), (1025, n + 1)):
            at = (deg >= lo) & (deg < hi)
            if at.any():
                assert_close(got[at].reshape(1, -1), want[at].reshape(1, -1), what="%s, %d to %d entries" % (what, lo, hi - 1))


@pytest.mark.parametrize("name", ["edges", "skewed"])
@pytest.mark.parametrize("heads,dh", [(1, 4), (3, 8), (1, 64), (8, 16), (8, 32)])
def test_values_that_no_entry_reads(graphs, name, heads, dh):
    """The own row of a node without entries reaches no gradient of Z, whatever it holds and whichever rows share its wave."""
    g, rp, _ = graphs[name]
    n, F = g.n_nodes, heads * dh
    empty = np.flatnonzero(np.diff(rp) == 0)
    a = [Hn.dev(wl.random_matrix(heads, dh, k) * np.float32(0.1)) for k in (1, 2)]
    Zh = wl.random_matrix(n, F, F)
    G = Hn.dev(wl.random_matrix(n, F, F + 1))
    kw = dict(heads=heads, a_src=a[0], a_dst=a[1])
    want = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Hn.dev(Zh), **kw)[0].cpu().numpy()[:, :F]
    Zh[empty] = np.array([np.inf, -np.inf, np.nan], np.float32)[np.arange(empty.size) % 3, None]
    Z = Hn.dev(Zh)
    plain = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, **kw)[0].cpu().numpy()[:, :F]
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
    Hn.aggregate(g, "gat_softmax", Z, F, workspace=ws, save=True, **kw)
    saved = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, saved=ws, **kw)[0].cpu().numpy()[:, :F]
    assert empty.size and np.array_equal(plain, want) and np.array_equal(saved[empty], want[empty])
    assert np.all(np.isfinite(saved))
