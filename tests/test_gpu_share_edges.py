"""Shares at the edges of the kernels that derive them: node counts around the blocks of 256 whose members the
lists are placed by, rows around the 64 entries of a tile and the tiles a wave holds in flight, and up to the
largest number of workers.  Whole numbers, so exact against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import partition as op
from paper_2302_13053_amd import harness as Hn
from test_gpu_partition import check_share

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P", [(1, 1), (63, 2), (255, 64), (256, 3), (257, 64), (4099, 64), (4099, 5)])
@pytest.mark.parametrize("owner", ["random", "runs", "one"])
def test_share_at_block_and_row_edges(n, P, owner):
    ends = [(0, v) for v in range(1, n)]                                       # a row over all nodes
    for h, k in ((1, 63), (2, 64), (3, 65), (4, 255), (5, 256), (6, 257), (7, 511), (8, 512), (9, 513)):
        ends += [(h, h + 9 + d) for d in range(k) if h + 9 + d < n]
    pairs = np.array(ends, dtype=np.int32).reshape(-1, 2)
    src, dst = np.ascontiguousarray(pairs[:, 0]), np.ascontiguousarray(pairs[:, 1])
    part = {"random": np.random.Generator(np.random.Philox(key=17 * n + P)).integers(0, P, n),
            "runs": np.arange(n) * P // n, "one": np.full(n, P - 1)}[owner].astype(np.int32)
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, True)
    rp, ci = oracle.csr_from_coo(src, dst, n, True)
    for p in sorted({0, P // 2, P - 1}):
        check_share(Hn.partition_share(g, Hn.dev(part), P, p), op.share(rp, ci, part, P, p), P)
