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
    for waves, n, pairs in ((8, 901, 9000), (4, 403, 60000)):
        src, dst = wl.random_pairs(n, pairs, n, skew=1.5)
        g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False))
        rp, ci = oracle.csr_from_coo(src, dst, n, False)
        assert (rp[-1] >= 128 * n) == (waves == 4)
        out[waves] = g, rp, ci
    yield out
    for g, _, _ in out.values():
        g.destroy()


@pytest.mark.parametrize("line", ["none", "some", "most"])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("heads,dh", [(4, 16), (1, 256), (8, 8), (4, 47), (8, 12), (2, 150)])
def test_row_classes(graphs, waves, heads, dh, line):
    g, rp, ci = graphs[waves]
    n, F = g.n_nodes, heads * dh
    Zh, Gh = wl.random_matrix(n, F, F, ld=wl.pad_ld(F)), wl.random_matrix(n, F, F + 1, ld=wl.pad_ld(F))
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Z, G, As, Ad = (Hn.dev(x) for x in (Zh, Gh, *a))
    deg = np.diff(rp)
    at = {"none": 1 << 20, "some": int(np.sort(deg)[-n // 10]), "most": 16}[line]
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
    for name, got in (("after save mode", dZ), ("two passes", both[0])):
        assert_close(got.cpu().numpy()[:, :F], want[0], what="backward " + name)
    assert all(torch.equal(x[..., :F], y[..., :F]) for x, y in zip((dZ, das, dad), again))
