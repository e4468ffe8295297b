"""The plan's row schedule where its sort can go wrong: either side of the sizes that take one workgroup, partial pieces
of a wave and of a workgroup, and degrees of one, two, three and four digits."""
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
def test_order_counts_and_normalisers(n, kind):
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
