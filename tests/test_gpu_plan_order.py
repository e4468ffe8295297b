"""The plan's row schedule where its sort can go wrong: either side of the sizes that take one workgroup or more of them,
partial pieces of a wave and of a workgroup, degrees of one to four digits and rows longer than two digits of ten bits
(2^20 - 1 entries), which are placed by rank; and that a plan of very many rows takes a few passes over them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn

pytestmark = pytest.mark.gpu


def degrees(n, kind, rng):
    if kind == "ties":                    # every wave full of one degree, with others between
        return np.where(rng.random(n) < 0.9, 3, rng.integers(0, 9, n))
    if kind == "empty":
        return np.zeros(n, np.int64)
    if kind == "bytes":                   # either side of 8 and 10 bits
        return rng.choice([0, 1, 255, 256, 257, 511, 1023, 1024, 1025], n)
    d = rng.integers(0, 40, n)            # a few rows of three and four digits (8 bits) or three (10 bits)
    at = rng.permutation(n)[:6]
    d[at] = np.array([1 << 16, (1 << 16) + 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1025, 1 << 24])[:len(at)]
    return d


@pytest.mark.parametrize("kind", ["ties", "empty", "bytes", "long"])
@pytest.mark.parametrize("n", [1, 63, 65, 1024, 1025, 4095, 4096, 4097, 18433, 32769, 270001])
def test_order_and_normalisers(n, kind):
    deg = degrees(n, kind, np.random.default_rng(n)).astype(np.int64)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rp[1:])
    nnz = int(rp[-1])
    col = torch.zeros(max(nnz, 1), dtype=torch.int32, device="cuda")          # the plan does not look at the columns
    g = Hn.DeviceGraph(n_nodes=n, nnz=nnz, row_ptr=Hn.dev(rp), col_idx=col)
    ws = torch.full((B.retexo_plan_workspace_bytes(n, nnz, 0),), 0xA5, dtype=torch.uint8, device="cuda")
    Hn.make_plan(g, workspace=ws)
    try:
        got_deg, got_dinv, order = Hn.plan_arrays(g)
        assert np.array_equal(got_deg, deg)
        assert np.array_equal(got_dinv.view(np.uint32), oracle.degree(rp)[1].view(np.uint32))
        assert np.array_equal(order, np.argsort(-deg, kind="stable"))
        assert B.retexo_plan_max_degree(g.plan) == deg.max()
    finally:
        g.destroy()


@pytest.mark.parametrize("n", [500, 40000])
def test_refused_row_offsets(n):
    """Offsets that run backwards, and a row that claims more entries than there are."""
    rp = np.arange(n + 1, dtype=np.int64)
    rp[n // 2] = 1 << 30
    g = Hn.DeviceGraph(n_nodes=n, nnz=n, row_ptr=Hn.dev(rp), col_idx=torch.zeros(n, dtype=torch.int32, device="cuda"))
    ws = Hn.ws_tensor(B.retexo_plan_workspace_bytes(n, n, B.F_SPLIT_ROWS))
    st, _ = B.retexo_plan_create_in(n, n, g.row_ptr.data_ptr(), g.col_idx.data_ptr(), B.F_SPLIT_ROWS, ws.data_ptr(),
                                    ws.numel(), Hn._stream_ptr())
    assert st == B.E_CSR


def plan_of(deg, workspace=None):
    """A plan whose rows have these lengths (device, int64)."""
    n, rp = deg.numel(), torch.zeros(deg.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=rp[1:])
    nnz = int(rp[-1])
    col = torch.zeros(max(nnz, 1), dtype=torch.int32, device="cuda")
    return Hn.make_plan(Hn.DeviceGraph(n_nodes=n, nnz=nnz, row_ptr=rp, col_idx=col), workspace=workspace)


@pytest.mark.parametrize("n,long", [(4097, 1), (4097, 40), (20000, 300), (300001, 700), (5_999_999, 3), (6_000_001, 60), (60_000_001, 5)])
def test_longest_rows_and_many_rows(n, long):
    g = torch.Generator(device="cuda").manual_seed(n + long)
    deg = torch.randint(0, 3, (n,), generator=g, device="cuda")
    top = (1 << 20) - 1
    values = torch.tensor([top - 1, top, top + 1, top, top + 2, 1 << 21], device="cuda")
    deg[torch.randperm(n, generator=g, device="cuda")[:long]] = values[torch.randint(0, 6, (long,), generator=g, device="cuda")]
    want = torch.sort(deg, descending=True, stable=True).indices.to(torch.int32)
    plan = plan_of(deg)
    try:
        order = torch.empty(n, dtype=torch.int32, device="cuda")
        B.check(B.retexo_plan_export(plan.plan, 0, 0, order.data_ptr(), Hn._stream_ptr()), "retexo_plan_export")
        assert torch.equal(order, want)
        assert B.retexo_plan_max_degree(plan.plan) == int(deg.max())
    finally:
        plan.destroy()


def test_no_rows():
    ws = Hn.ws_tensor(B.retexo_plan_workspace_bytes(0, 0, B.F_SPLIT_ROWS))
    rp = torch.zeros(1, dtype=torch.int64, device="cuda")
    st, plan = B.retexo_plan_create_in(0, 0, rp.data_ptr(), 0, B.F_SPLIT_ROWS, ws.data_ptr(), ws.numel(), Hn._stream_ptr())
    assert st == B.OK and B.retexo_plan_num_nodes(plan) == 0 and B.retexo_plan_max_degree(plan) == 0
    B.retexo_plan_destroy(plan)


def test_many_rows_take_few_passes():
    """40 million rows, one of three million entries: as long as 9 copies of the row offsets on an MI355X; with 128 workgroups
    and a pass for every digit of the longest row as long as 23.  The line lies between."""
    n = 40_000_000
    deg = torch.ones(n, dtype=torch.int64, device="cuda")
    deg[n // 3] = 3_000_000
    ws = Hn.ws_tensor(B.retexo_plan_workspace_bytes(n, n + 3_000_000, 0))
    plan_of(deg, ws).destroy()
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=rp[1:])
    nnz = int(rp[-1])
    graph = Hn.DeviceGraph(n_nodes=n, nnz=nnz, row_ptr=rp, col_idx=torch.zeros(nnz, dtype=torch.int32, device="cuda"))
    other = torch.empty_like(rp)

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

    def plan():
        Hn.make_plan(graph, workspace=ws)
        graph.destroy()
    copy, build = best(lambda: other.copy_(rp)), best(plan)
    assert build <= 14 * copy, (build, copy)
