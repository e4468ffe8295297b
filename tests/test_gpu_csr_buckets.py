"""CSR construction where its buckets change: rows whose neighbours together just fit or just miss what a bucket
holds (10,240 entries), runs of rows that overfill one, and sizes around the least and the largest target.  Whole
numbers, so exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2302_13053_amd import harness as Hn

pytestmark = pytest.mark.gpu

HUBS = 20000                                                     # hubs sit behind the nodes that they link to


@pytest.mark.parametrize("lengths", [
    (5120, 5120), (5120, 5121), (7167, 3073), (7168, 3073), (10239, 1), (10240, 1), (1, 10240), (10241,),
    (3400, 3400, 3400, 3400), (3413, 3413, 3414, 3414), (12000, 12000, 1, 1, 9000), (1024,) * 40, (1023, 1) * 20,
    (7168,) * 30, (7169, 2) * 20], ids=str)
@pytest.mark.parametrize("repeats", [1, 2])
def test_rows_around_the_bucket_sizes(lengths, repeats):
    n = HUBS + len(lengths)
    src = np.concatenate([np.full(k, HUBS + i) for i, k in enumerate(lengths)]).astype(np.int32)
    dst = np.concatenate([(np.arange(k) * 7 + i) % HUBS for i, k in enumerate(lengths)]).astype(np.int32)
    src, dst = np.tile(src, repeats), np.tile(dst, repeats)      # repeats fill the buckets and are dropped again
    order = np.random.Generator(np.random.Philox(key=n)).permutation(src.size)
    src, dst = np.ascontiguousarray(src[order]), np.ascontiguousarray(dst[order])
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False)
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    assert np.array_equal(g.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(g.col_idx[:g.nnz].cpu().numpy(), ci)


@pytest.mark.parametrize("pairs", [81919, 81920, 200000, 573000, 574000])     # 2 * pairs / 160 around 1,024 and 7,168
@pytest.mark.parametrize("n", [3000, 60000])
def test_sizes_around_the_targets(pairs, n):
    rng = np.random.Generator(np.random.Philox(key=pairs + n))
    src, dst = rng.integers(0, n, pairs).astype(np.int32), (rng.random(pairs) ** 2 * n).astype(np.int32)
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, True)
    rp, ci = oracle.csr_from_coo(src, dst, n, True)
    assert np.array_equal(g.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(g.col_idx[:g.nnz].cpu().numpy(), ci)
