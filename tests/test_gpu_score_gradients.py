"""The gradient of a node's source score, the difference of two sums over its entries that are large beside it: its error against 64
bits.  A column in which the incoming gradient and the destination vector are zero and the source vector is a power of two shows
it as it is, times that power.  Values of one sign; small multiples of powers of two, so that scores are exact."""
import numpy as np
import pytest

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl

pytestmark = pytest.mark.gpu


def as_one_running_sum(rp, ci, Z, G, w, c):
    """The difference with the products w <G, z> in one float32 running sum per four columns, and the sums w c added up exactly."""
    n, f32 = len(rp) - 1, np.float32
    out = np.zeros((n, Z.shape[1] // 4), f32)
    deg = np.diff(rp)
    for j in range(deg.max()):
        u = np.flatnonzero(deg > j)
        e = rp[u] + j
        pd = np.zeros((u.size, out.shape[1]), f32)
        for k in range(4):
            pd = (G[ci[e], k::4].astype(np.float64) * Z[u, k::4] + pd).astype(f32)
        out[u] = (w[e].astype(f32).astype(np.float64)[:, None] * pd + out[u]).astype(f32)
    exact = np.add.reduceat(np.append(w * c.astype(f32)[ci], 0.0), np.minimum(rp[:-1], rp[-1]))
    return out.astype(f32).sum(1, dtype=f32).astype(np.float64) - np.where(deg > 0, exact, 0.0).astype(f32)


@pytest.mark.parametrize("entries,dh", [(30, 16), (117, 16), (117, 32), (117, 64), (300, 32)])
@pytest.mark.parametrize("save", [False, True])
def test_error_of_the_score_gradient(entries, dh, save):
    n, slope = 3001, np.float64(np.float32(0.2))
    src, dst = wl.random_pairs(n, n * entries // 2, 9, skew=0.3)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, True))
    rp, ci = (x.astype(np.int64) for x in oracle.csr_from_coo(src, dst, n, True))
    Zh = np.abs(np.rint(wl.random_matrix(n, dh, 3) * 8)).astype(np.float32) / 8
    Gh = np.abs(wl.random_matrix(n, dh, 4))
    a = [np.rint(wl.random_matrix(1, dh, k) * 8).astype(np.float32) / 64 for k in (1, 2)]
    Gh[:, 5], a[0][0, 5], a[1][0, 5] = 0.0, 0.125, 0.0
    # 64 bits: entry e of row v holds node ci[e]
    row = np.repeat(np.arange(n), np.diff(rp))
    Z, G = Zh.astype(np.float64), Gh.astype(np.float64)
    p = (Z @ a[0][0])[ci] + (Z @ a[1][0])[row]
    s = np.where(p > 0, p, slope * p)
    x = np.exp(s - np.maximum.reduceat(s, rp[:-1])[row])
    al = x / np.add.reduceat(x, rp[:-1])[row]
    da = np.concatenate([np.einsum("ed,ed->e", G[row[k:k + 100000]], Z[ci[k:k + 100000]]) for k in range(0, row.size, 100000)])
    c = np.add.reduceat(al * da, rp[:-1])
    t = np.where(p > 0, 1.0, slope) * al
    want = np.zeros(n)
    np.add.at(want, ci, t * (da - c[row]))
    # the same entries seen from their source: the graph is symmetric
    turned = np.lexsort((row, ci))
    assert np.array_equal(row[turned], ci)
    emulated = as_one_running_sum(rp, ci, Zh, Gh, t[turned], c)
    kw = dict(heads=1, a_src=Hn.dev(a[0]), a_dst=Hn.dev(a[1]))
    saved, Zd = None, Hn.dev(Zh)
    if save:
        saved = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, dh, B.MODES["gat_softmax"], 1, B.F_SAVE))
        Hn.aggregate(g, "gat_softmax", Zd, dh, workspace=saved, save=True, **kw)
    dZ = Hn.aggregate_backward(g, "gat_softmax", dh, Hn.dev(Gh), Z=Zd, saved=saved, **kw)[0].cpu().numpy()
    g.destroy()
    got = dZ[:, 5].astype(np.float64) * 8
    error, bound = (np.linalg.norm(y - want) for y in (got, emulated))
    print("entries %d, %d columns: error %.3g, with one running sum of the products %.3g" % (entries, dh, error, bound))
    assert error <= bound
