"""Rows with a workgroup of their own beside rows with one wave, in one launch: lengths around the batch sizes, the tile of 64
entries and the threshold (64 on graphs of this size), against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close, assert_cond_close

pytestmark = pytest.mark.gpu

LENGTHS = {
    "mixed": [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 62, 63, 64, 65, 127, 128, 129, 511, 512, 513, 600],
    "all long": [64, 70, 128, 400, 576, 577],
    "none long": [1, 0, 63, 8, 3, 33],
    "one row": [513],
}


def graph(name):
    lengths = LENGTHS[name]
    n = 700
    rng = np.random.Generator(np.random.Philox(key=len(lengths)))
    deg = np.zeros(n, np.int64)
    if name == "all long":
        n = len(lengths)
        deg = np.array(lengths, np.int64)
        n_src = 600
    else:
        n_src = n
        at = rng.permutation(n)[:len(lengths)]
        deg[at] = lengths
    if name == "all long":               # every row of the graph is long: columns repeat over the few nodes there are
        ci = np.concatenate([np.sort(rng.integers(0, n, d)) for d in deg]).astype(np.int32)
    else:
        ci = np.concatenate([np.sort(rng.permutation(n_src)[:d]) for d in deg]).astype(np.int32)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(deg)
    g = Hn.DeviceGraph(n, int(rp[-1]), Hn.dev(rp), Hn.dev(ci if ci.size else np.zeros(1, np.int32)))
    return Hn.make_plan(g, validate=True), rp, ci


@pytest.fixture(autouse=True)
def threshold():
    """Long from 64 entries on, whatever the graph's mean row (the default draws the line at twice the mean at least)."""
    B.load()
    B.check(B.retexo_set_option("agg_heavy_degree", 64), "set_option")
    yield
    B.check(B.retexo_set_option("agg_heavy_degree", 2048), "set_option")


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("F", [1, 31, 128, 256, 257, 500, 1433])
@pytest.mark.parametrize("mode", ["mean", "sum", "gcn_sym", "max"])
def test_row_classes_in_one_launch(name, F, mode):
    g, rp, ci = graph(name)
    ld = wl.pad_ld(F) if F != 31 else 31
    Z = wl.random_matrix(g.n_nodes, F, F, ld=ld)
    got = Hn.aggregate(g, mode, Hn.dev(Z), F, concat=True).cpu().numpy()[:, :2 * F]
    want = oracle.aggregate(mode, rp, ci, Z, F, self_concat=True)
    if mode == "max":
        assert np.array_equal(got.astype(np.float64), want)
    else:
        # a sum of 600 terms in float32: 600 roundings of 2^-24 of the terms' size at worst is 3.6e-5, 1.5e-6 as they fall
        # (where a row names the same few columns again and again the roundings repeat too: the worst counts)
        assert_cond_close(got, want, oracle.aggregate_abs(mode, rp, ci, Z, F, self_concat=True), what=name,
                          tol=600 * 2.0 ** -24 if name == "all long" else 1e-5)
    again = Hn.aggregate(g, mode, Hn.dev(Z), F, concat=True).cpu().numpy()[:, :2 * F]
    assert np.array_equal(got, again)
    g.destroy()


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("heads,dh", [(4, 16), (4, 47), (1, 64), (8, 5)])
def test_edge_softmax_row_classes(name, heads, dh):
    g, rp, ci = graph(name)
    F = heads * dh
    Z = wl.random_matrix(g.n_nodes, F, F, ld=wl.pad_ld(F))
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.2) for k in (1, 2)]
    got = Hn.aggregate(g, "gat_softmax", Hn.dev(Z), F, heads=heads, a_src=Hn.dev(a[0]), a_dst=Hn.dev(a[1]))
    want = oracle.aggregate("gat_softmax", rp, ci, Z, F, heads=heads, a_src=a[0], a_dst=a[1])
    # a softmax average of 600 rows of at least 40 columns: no worse than the sums above, and rows of robust magnitude
    assert_close(got.cpu().numpy()[:, :F], want, what=name)
    g.destroy()


def test_default_threshold_is_an_upper_bound():
    # the same graph with the classes drawn elsewhere: the same sums in another order
    g, rp, ci = graph("mixed")
    Z = wl.random_matrix(g.n_nodes, 96, 1)
    B.check(B.retexo_set_option("agg_heavy_degree", 2048), "set_option")     # the default
    first = Hn.aggregate(g, "sum", Hn.dev(Z), 96).clone()
    try:
        B.check(B.retexo_set_option("agg_heavy_degree", 1 << 20), "set_option")      # no long rows at all
        other = Hn.aggregate(g, "sum", Hn.dev(Z), 96)
    finally:
        B.check(B.retexo_set_option("agg_heavy_degree", 2048), "set_option")
    mag = oracle.aggregate_abs("sum", rp, ci, Z, 96)
    assert_cond_close(first.cpu().numpy()[:, :96], other.cpu().numpy()[:, :96].astype(np.float64), mag, what="classes")
    assert not torch.equal(first[:, :96], other[:, :96])       # 600 entries in eight interleaved sums round differently
    g.destroy()


def test_every_row_can_be_given_a_workgroup():
    # rows of 40 entries in slabs of 32 columns: a workgroup each with the line at one entry, bundled with the line at 64;
    # the two add up in other orders
    n, F = 500, 96
    rng = np.random.Generator(np.random.Philox(key=40))
    rp = np.arange(n + 1, dtype=np.int64) * 40
    ci = np.concatenate([np.sort(rng.permutation(n)[:40]) for _ in range(n)]).astype(np.int32)
    g = Hn.make_plan(Hn.DeviceGraph(n, int(rp[-1]), Hn.dev(rp), Hn.dev(ci)), validate=True)
    Z = wl.random_matrix(n, F, 41)
    want, mag = oracle.aggregate("sum", rp, ci, Z, F), oracle.aggregate_abs("sum", rp, ci, Z, F)
    got = {}
    try:
        B.check(B.retexo_set_option("agg_slab_cols", 32), "set_option")
        for line in (1, 64):
            B.check(B.retexo_set_option("agg_narrow_heavy", line), "set_option")
            got[line] = Hn.aggregate(g, "sum", Hn.dev(Z), F).cpu().numpy()[:, :F]
            assert_cond_close(got[line], want, mag, what="line at %d" % line)
    finally:
        B.check(B.retexo_set_option("agg_slab_cols", 0), "set_option")
        B.check(B.retexo_set_option("agg_narrow_heavy", 1024), "set_option")
    assert not np.array_equal(got[1], got[64])
    g.destroy()


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("F", [31, 128, 700])
@pytest.mark.parametrize("mode", ["mean", "gcn_sym", "max", "gat_softmax"])
def test_default_line(name, F, mode):
    # the line that the size of the call draws, not the one the fixture pins
    B.check(B.retexo_set_option("agg_heavy_degree", 2048), "set_option")
    g, rp, ci = graph(name)
    Z = wl.random_matrix(g.n_nodes, F, F, ld=wl.pad_ld(F))
    a = wl.random_matrix(1, F, 1) * np.float32(0.02)
    kw = dict(heads=1, a_src=a, a_dst=a) if mode == "gat_softmax" else {}
    dev = {k: Hn.dev(v) if k != "heads" else v for k, v in kw.items()}
    got = Hn.aggregate(g, mode, Hn.dev(Z), F, **dev).cpu().numpy()[:, :F]
    want = oracle.aggregate(mode, rp, ci, Z, F, **kw)
    if mode == "max":
        assert np.array_equal(got.astype(np.float64), want)
    elif mode == "gat_softmax":
        assert_close(got, want, what=name)
    else:
        assert_cond_close(got, want, oracle.aggregate_abs(mode, rp, ci, Z, F),
                          tol=600 * 2.0 ** -24 if name == "all long" else 1e-5, what=name)
    g.destroy()
