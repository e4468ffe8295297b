"""A worker's share either side of the sizes whose tables fit LDS (owners of one to eight bits, the numbering), and rows
around the length that a workgroup's waves share."""
import numpy as np
import pytest

import oracle
from oracle import partition as op
from paper_2302_13053_amd import harness as Hn
from test_gpu_partition import check_share

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P", [
    (1, 2), (31, 2), (257, 64), (65535, 2), (65536, 2), (70000, 4), (70000, 5), (70001, 16), (70000, 17),
    (131000, 64), (131072, 64), (131200, 64),         # eight bits per owner fit up to 131,072 nodes
    (235900, 16), (236000, 16),                       # four bits: 235,929
    (294912, 3), (294913, 3), (393300, 4),            # the numbering: 294,912; two bits: 393,216
])
def test_sizes_and_long_rows(n, P):
    rng = np.random.Generator(np.random.Philox(key=n + P))
    m = min(3 * n, 200000) if n < 65000 else 640000   # the last worker's share then has more than 2^20 entries
    src, dst = [rng.integers(0, n, m)], [rng.integers(0, n, m)]
    for k in (2047, 2048, 2049, 2100, 30000):         # entries of a few rows, before what else they have
        if k < n:
            src.append(np.full(k, n // 2 + k))
            dst.append(rng.permutation(n)[:k])
    src, dst = (np.concatenate(x).astype(np.int32) % n for x in (src, dst))
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False)
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    part = rng.integers(0, P, n).astype(np.int32)
    part[rng.random(n) < 0.9] = P - 1                 # the last worker owns most
    part[[(n // 2 + k) % n for k in (2047, 2048, 2049, 2100, 30000)]] = P - 1
    for p in {0, P - 1}:
        want = op.share(rp, ci, part, P, p)
        check_share(Hn.partition_share(g, Hn.dev(part), P, p), want, P)
    assert n < 65000 or P == 1 or op.share(rp, ci, part, P, P - 1).col_idx.size > 1 << 20
