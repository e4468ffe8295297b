"""A mean divides by the plan's degrees, which retexo_plan_set_degrees may have replaced by others than the row lengths (a sampled
neighbourhood scaled by the whole one), whichever kernel the call takes: row groups, whole rows, source ranges, 16-bit tables."""
import numpy as np
import pytest
import torch

import oracle
from oracle import storage as ost
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_cond_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    n, (s, d) = 9001, wl.random_pairs(9001, 60000, 2, skew=3.0)
    rp, ci = oracle.csr_from_coo(s, d, n, False)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(s), Hn.dev(d), n, False), split_rows=True)
    deg = np.diff(rp)
    assert (deg == 0).any() and deg.max() > 1000
    set_to = (2 * deg + np.arange(n) % 3 + 1).astype(np.int32)
    held = Hn.dev(set_to)
    B.check(B.retexo_plan_set_degrees(g.plan, held.data_ptr()), "set_degrees")
    yield g, rp, ci, set_to.astype(np.float64)[:, None]
    g.destroy()


@pytest.fixture
def options():
    defaults = {"agg_slab_cols": 0, "agg_parts": -1, "agg_max_vec": 4}
    yield lambda name, value: B.check(B.retexo_set_option(name, value), "set_option")
    for name, value in defaults.items():
        B.check(B.retexo_set_option(name, value), "set_option")


@pytest.mark.parametrize("fmt", ["fp32", "bf16"])
@pytest.mark.parametrize("F", [30, 64, 200, 602])
@pytest.mark.parametrize("option", [None, ("agg_slab_cols", 256), ("agg_slab_cols", 64), ("agg_parts", 4), ("agg_max_vec", 1)])
def test_mean_uses_them(graph, options, option, F, fmt):
    g, rp, ci, deg = graph
    if option:
        options(*option)
    Zh = wl.random_matrix(g.n_nodes, F, F)
    ld = (F + 7) // 8 * 8
    if fmt == "fp32":
        Z = torch.zeros(g.n_nodes, ld, device="cuda")
        Z[:, :F] = torch.from_numpy(Zh)
        got = Hn.aggregate(g, "mean", Z, F)
    else:
        bits = ost.store(Zh, fmt)
        Zh = ost.load(bits, fmt)
        Z = torch.zeros(g.n_nodes, ld, dtype=torch.int16, device="cuda")
        Z[:, :F] = torch.from_numpy(bits.view(np.int16))
        got = Hn.aggregate_stored(g, "mean", Z, F, fmt)
    assert_cond_close(got.cpu().numpy()[:, :F], oracle.aggregate("sum", rp, ci, Zh, F) / deg,
                      oracle.aggregate_abs("sum", rp, ci, Zh, F) / deg, what="mean")
