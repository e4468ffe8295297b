"""CSR construction of graphs that one workgroup builds in one launch: sizes at the ends of its range, rows at the ends of what
a thread sorts (4, 8, 16 entries) and a wave marks, repeats, hubs.  Whole numbers, so exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn

pytestmark = pytest.mark.gpu


def check(src, dst, n, loops):
    src, dst = np.asarray(src, np.int32), np.asarray(dst, np.int32)
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, loops)
    rp, ci = oracle.csr_from_coo(src, dst, n, loops)
    assert g.nnz == rp[-1] and np.array_equal(g.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(g.col_idx[:g.nnz].cpu().numpy(), ci)


@pytest.mark.parametrize("n,pairs,loops", [(1, 0, False), (1, 3, True), (2, 1, False), (8192, 8192, False), (8192, 8193, False),
                                           (8193, 8192, False), (4096, 4096, True), (4097, 4096, True), (8192, 1, True),
                                           (100, 8192, False), (2708, 5429, False), (33, 8000, True), (1024, 6000, False)])
@pytest.mark.parametrize("skew", [1, 4])
def test_sizes(n, pairs, loops, skew):
    rng = np.random.Generator(np.random.Philox(key=n + pairs))
    src, dst = rng.integers(0, n, pairs), (rng.random(pairs) ** skew * n).astype(np.int64)
    check(src, dst, n, loops)


@pytest.mark.parametrize("repeats", [1, 2])
@pytest.mark.parametrize("length", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 33, 63, 64, 65, 2000, 4000])
def test_row_lengths(length, repeats):
    """Rows of one length (the repeats fill them up and are dropped again) in descending order of the columns."""
    hubs = max(1, min(100, 4000 // length))
    src = np.repeat(np.arange(hubs), length)
    dst = hubs + np.tile(np.arange(length)[::-1], hubs) * 3 % 4001 + np.repeat(np.arange(hubs), length) % 3
    check(np.tile(src, repeats), np.tile(dst, repeats), hubs + 4003, False)


def test_one_pair_again_and_again():
    check(np.full(8192, 5), np.full(8192, 8191), 8192, False)
    check(np.full(8192, 5), np.full(8192, 5), 8192, False)


def test_errors_leave_the_output_alone():
    src, dst = np.array([0, 1, 7], np.int32), np.array([1, 2, 3], np.int32)
    s, d = Hn.dev(src), Hn.dev(dst)
    import torch
    ws = Hn.ws_tensor(B.retexo_csr_workspace_bytes(3, 8, False))
    for n, cap, want in ((7, 6, B.E_CSR), (8, 5, B.E_CAPACITY), (8, 6, B.OK)):
        rp, ci = torch.full((9,), -1, dtype=torch.int64, device="cuda"), torch.full((6,), -1, dtype=torch.int32, device="cuda")
        st, nnz = B.retexo_csr_from_coo(3, s.data_ptr(), d.data_ptr(), n, False, rp.data_ptr(), ci.data_ptr(), cap, ws.data_ptr(),
                                        ws.numel(), 0)
        torch.cuda.synchronize()
        assert st == want
        if st != B.OK:
            assert bool((rp == -1).all()) and bool((ci == -1).all())
        if st == B.E_CAPACITY:
            assert nnz == 6
