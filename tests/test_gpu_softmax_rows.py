"""Edge softmax, forward, save mode and backward, with long and short rows in one launch: workgroups of eight waves (graphs of
short rows) and of four (a mean row of 128 entries or more), at head widths of each kernel, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graphs():
    out = {}
    for waves, n, pairs, skew in ((8, 901, 70000, 1.0), (4, 403, 60000, 1.5)):
        src, dst = wl.random_pairs(n, pairs, n, skew=skew)
        g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False))
        rp, ci = oracle.csr_from_coo(src, dst, n, False)
        assert (rp[-1] >= 128 * n) == (waves == 4)
        out[waves] = g, rp, ci
    yield out
    for g, _, _ in out.values():
        g.destroy()


def decided_rows(rp, ci, heads, dh, a):
    """[n, heads * dh] normal values whose scores are all further from zero than float32 can put them on the other side, where
    the slope and with it the gradient jump: sixteen roundings (a lane's columns, the lanes of a head and the two halves one
    after the other) of 2^-24 of the terms' sizes.  Of 100,000 entries times the heads one or two are closer for most seeds."""
    n = len(rp) - 1
    row = np.repeat(np.arange(n), np.diff(rp))
    for seed in range(100):
        Z = wl.random_matrix(n, heads * dh, 1000 * dh + seed, ld=wl.pad_ld(heads * dh))
        z = Z[:, :heads * dh].reshape(n, heads, dh).astype(np.float64)
        el, er = (np.einsum("nhd,hd->nh", z, x) for x in a)
        size = sum(np.einsum("nhd,hd->nh", np.abs(z), np.abs(x))[at] for x, at in zip(a, (ci, row)))
        if np.all(np.abs(el[ci] + er[row]) > 16 * 2.0 ** -24 * size):
            return Z
    raise AssertionError("no decided input")


@pytest.mark.parametrize("line", ["none", "some", "most"])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("heads,dh", [(4, 16), (1, 256), (8, 8), (4, 47), (8, 12), (2, 150)])
def test_row_classes(graphs, waves, heads, dh, line):
    g, rp, ci = graphs[waves]
    n, F = g.n_nodes, heads * dh
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Zh, Gh = decided_rows(rp, ci, heads, dh, a), wl.random_matrix(n, F, F + 1, ld=wl.pad_ld(F))
    Z, G, As, Ad = (Hn.dev(x) for x in (Zh, Gh, *a))
    deg = np.diff(rp)
    # some: a tile for each of the waves that share a row; most: the eight-wave graph's 885 of 901, all of the other
    at = {"none": 1 << 20, "some": 64 * waves, "most": 64}[line]
    few, many = {"none": (0, 0), "some": (5, n // 10), "most": (n * 9 // 10, n)}[line]
    assert few <= (deg >= at).sum() <= many
    kw = dict(heads=heads, a_src=As, a_dst=Ad)
    B.check(B.retexo_set_option("agg_heavy_degree", at), "set_option")
    try:
        plain = Hn.aggregate(g, "gat_softmax", Z, F, **kw)
        ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], heads, B.F_SAVE))
        out = Hn.aggregate(g, "gat_softmax", Z, F, workspace=ws, save=True, **kw)
        dZ, das, dad = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, saved=ws, **kw)
        again = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, saved=ws, **kw)
        both = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, **kw)
    finally:
        B.check(B.retexo_set_option("agg_heavy_degree", 2048), "set_option")
    okw = dict(heads=heads, a_src=a[0], a_dst=a[1])
    fwd = oracle.aggregate("gat_softmax", rp, ci, Zh, F, **okw)
    want = oracle.aggregate_backward("gat_softmax", rp, ci, Zh, F, Gh, **okw)
    assert_close(plain.cpu().numpy()[:, :F], fwd, what="forward")
    assert_close(out.cpu().numpy()[:, :F], fwd, what="save mode")
    for name, got in (("after save mode", (dZ, das, dad)), ("two passes", both)):
        assert_close(got[0].cpu().numpy()[:, :F], want[0], what="backward " + name)
        for grad, ref, what in zip(got[1:], want[1:], ("source", "destination")):     # (one ratio over each whole gradient)
            assert_close(grad.cpu().numpy().reshape(1, -1), ref.reshape(1, -1), what="%s attention vector %s" % (what, name))
    assert all(torch.equal(x[..., :F], y[..., :F]) for x, y in zip((dZ, das, dad), again))


def best(run):
    t = float("inf")
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        b.synchronize()
        t = min(t, a.elapsed_time(b))
    return t


def test_short_rows_alone_keep_four_waves():
    """60,000 nodes of 50 entries, none long.  Save mode with scores from the table (heads of 25 columns) in units of the one
    that forms them itself (64 columns): 0.62 in workgroups of four waves, 0.80 in workgroups of eight."""
    n = 60000
    gen = torch.Generator(device="cuda").manual_seed(3)
    src, dst = (torch.randint(0, n, (n * 25,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    g = Hn.make_plan(Hn.csr_from_coo(src, dst, n, False))
    times = []
    for dh in (25, 64):
        F = 4 * dh
        Z = torch.randn((n, wl.pad_ld(F)), generator=gen, device="cuda")
        a = torch.randn((4, dh), generator=gen, device="cuda") * 0.1
        ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], 4, B.F_SAVE))
        out = torch.zeros_like(Z)
        times.append(best(lambda: Hn.aggregate(g, "gat_softmax", Z, F, heads=4, a_src=a, a_dst=a, out=out, workspace=ws, save=True)))
    g.destroy()
    assert times[0] <= 0.7 * times[1], times


def test_one_very_long_row_is_shared_by_eight_waves():
    """300,000 nodes of 40 entries, 256 columns, one row of 200,000 entries more: 2.8 times as long as without it, 4.7 where
    four waves share the row."""
    n, F = 300000, 256
    gen = torch.Generator(device="cuda").manual_seed(4)
    src, dst = (torch.randint(0, n, (n * 20,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    hub = torch.arange(200000, dtype=torch.int32, device="cuda")
    Z = torch.randn((n, F), generator=gen, device="cuda")
    a = torch.randn((4, F // 4), generator=gen, device="cuda") * 0.1
    out = torch.zeros_like(Z)
    times = []
    for s, d in ((src, dst), (torch.cat([src, torch.full_like(hub, 7)]), torch.cat([dst, hub]))):
        g = Hn.make_plan(Hn.csr_from_coo(s, d, n, False))
        ws = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, B.MODES["gat_softmax"], 4, 0))
        times.append(best(lambda: Hn.aggregate(g, "gat_softmax", Z, F, heads=4, a_src=a, a_dst=a, out=out, workspace=ws)))
        g.destroy()
    assert times[1] <= 3.7 * times[0], times
