"""CSR construction of rows that alone overfill a bucket (10,240 entries): marked in a bit map of one or several stretches,
with rows of one or several words, or walked through in key ranges; and both forms of the entries between the two
bucket levels.  Whole numbers, so exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ordinary", [
    (12, 40000),            # fewer than 32 columns: key ranges, single keys repeated
    (1000, 30000),          # rows shorter than what a wave looks at
    (2048, 30000), (2049, 30000),
    (40000, 100000),        # two rows per bin
    (300000, 700000),       # sixteen rows per bin: sixteen stretches
    (3000000, 700000),      # 128 rows per bin: key ranges; entries of two words between the levels
])
@pytest.mark.parametrize("hubs", [(10241,), (30000, 12000), (60000, 3)], ids=str)
def test_hub_rows(n, ordinary, hubs):
    rng = np.random.Generator(np.random.Philox(key=n + sum(hubs)))
    src, dst = [rng.integers(0, n, ordinary)], [rng.integers(0, n, ordinary)]
    at = rng.integers(0, n - 1)
    for i, k in enumerate(hubs):                       # neighbouring ids, so that hubs share a bin; repeats where n < k
        src.append(np.full(k, (at + i) % n))
        dst.append(rng.permutation(n)[:k] if k <= n else rng.integers(0, n, k))
    src.append(np.full(20000, (at + 5) % n))           # one and the same entry more often than a bucket holds
    dst.append(np.full(20000, (at + 7) % n))
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    order = rng.permutation(src.size)
    src, dst = np.ascontiguousarray(src[order]), np.ascontiguousarray(dst[order])
    g = Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, False)
    rp, ci = oracle.csr_from_coo(src, dst, n, False)
    assert np.array_equal(g.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(g.col_idx[:g.nnz].cpu().numpy(), ci)


def test_sparse_hubs_are_not_read_once_per_stretch():
    """Twenty bins of 64 rows with 270,000 entries each: 7.7 times as long as the sorted-key construction, 12.6 times where they
    were marked in 256 stretches of the map, each of which reads all entries.  The line lies between."""
    n, hubs, entries = 1_200_000, 20, 270_000
    gen = torch.Generator(device="cuda").manual_seed(7)
    dst = torch.randint(0, n, (hubs * entries,), generator=gen, device="cuda", dtype=torch.int32)
    row = torch.randint(0, 64, (hubs, entries), generator=gen, device="cuda", dtype=torch.int32)
    src = (row + 64 * 900 * torch.arange(hubs, dtype=torch.int32, device="cuda")[:, None]).reshape(-1)
    m = src.numel()
    ws = Hn.ws_tensor(B.retexo_csr_workspace_bytes(m, n, False))
    rp, ci = torch.empty(n + 1, dtype=torch.int64, device="cuda"), torch.empty(2 * m, dtype=torch.int32, device="cuda")

    def best():
        t = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g = Hn.csr_from_coo(src, dst, n, False, ws, rp, ci)
            b.record()
            b.synchronize()
            t = min(t, a.elapsed_time(b))
        return t, g.nnz, rp.clone(), ci[:g.nnz].clone()
    bucketed = best()
    B.check(B.retexo_set_option("csr_sorted_keys", 1), "set_option")
    try:
        keys = best()
    finally:
        B.check(B.retexo_set_option("csr_sorted_keys", 0), "set_option")
    assert bucketed[1] == keys[1] and torch.equal(bucketed[2], keys[2]) and torch.equal(bucketed[3], keys[3])
    assert bucketed[0] <= 10 * keys[0], (bucketed[0], keys[0])
