"""Narrow-slab aggregation and the 16-bit store at the edges of their vectors: widths around a vector and a slab, the last
row at the end of its buffer, rows without an entry in a step beside rows that have one, and infinities in rows that
only some gather."""
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
N = 1003


@pytest.fixture(scope="module")
def graphs():
    src, dst = wl.random_pairs(N, 9000, 17, skew=2.0)
    out = {}
    for loops in (False, True):
        g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), N, loops), split_rows=True)
        out[loops] = (g, *oracle.csr_from_coo(src, dst, N, loops))
    yield out
    for g, _, _ in out.values():
        g.destroy()


@pytest.mark.parametrize("fmt", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("mode", ["sum", "gcn_sym"])
@pytest.mark.parametrize("F", [1, 8, 31, 33, 63, 64, 65, 72, 130])
def test_widths_and_infinities(graphs, fmt, mode, F):
    g, rp, ci = graphs[mode == "gcn_sym"]
    bad = int(ci[len(ci) // 2])                       # a node that some rows gather
    Z = wl.random_matrix(N, F, F, ld=F)
    Z[bad] = np.inf
    Z[0] = np.inf                                     # what an entry that does not exist could be taken for
    ld = -(-F // 8) * 8
    flat = torch.full((N * ld,), float("nan"), device="cuda")       # ends with the last row's last vector
    table = flat.view(N, ld)
    table[:, :F] = Hn.dev(Z)
    stored = Z if fmt == "fp32" else ost.load(ost.store(Z, fmt), fmt)
    try:
        B.retexo_set_option("agg_slab_cols", 32 if fmt == "fp32" else 64)
        for parts in (1, 4):
            B.retexo_set_option("agg_parts", parts)
            if fmt == "fp32":
                out = Hn.aggregate(g, mode, table, F)
            else:
                out = Hn.aggregate_stored(g, mode, Hn.store_rows(table, F, fmt, ld=ld), F, fmt)
            got = out[:, :F].cpu().numpy()
            touched = np.array([np.isin([0, bad], ci[rp[v]:rp[v + 1]]).any() for v in range(N)])
            assert np.all(np.isinf(got[touched])) and np.all(np.isfinite(got[~touched]))
            rows = np.flatnonzero(~touched)
            want = oracle.aggregate(mode, rp, ci, np.where(np.isinf(stored), 0, stored), F, rows=rows)
            mag = oracle.aggregate_abs(mode, rp, ci, np.where(np.isinf(stored), 0, stored), F, rows=rows)
            assert_cond_close(got[rows], want, mag, what="%s %s F=%d parts=%d" % (fmt, mode, F, parts))
    finally:
        B.retexo_set_option("agg_slab_cols", 0)
        B.retexo_set_option("agg_parts", -1)


@pytest.mark.parametrize("F,ld,ld16,shift", [(1, 4, 4, 0), (3, 4, 8, 0), (4, 4, 4, 0), (255, 256, 256, 0), (257, 260, 264, 0),
                                             (602, 608, 640, 0), (602, 602, 602, 0), (64, 64, 64, 1)])
@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_store_widths_and_alignments(fmt, F, ld, ld16, shift):
    n = 130
    X = torch.from_numpy(wl.random_matrix(n, F, F + 3, ld=ld)).cuda()
    flat = torch.zeros(n * ld + 4, device="cuda")
    flat[shift:shift + n * ld] = X.reshape(-1)
    out = torch.full((n, ld16), 77, dtype=torch.int16, device="cuda")
    B.check(B.retexo_store_rows(B.STORAGE[fmt], n, F, flat.data_ptr() + 4 * shift, ld, out.data_ptr(), ld16, Hn._stream_ptr()),
            "retexo_store_rows")
    got = out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :F], ost.store(X.cpu().numpy()[:, :F], fmt)) and np.all(got[:, F:] == 77)
