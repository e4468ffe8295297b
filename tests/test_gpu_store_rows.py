"""Rows into 16-bit storage: every width class of its kernels at the edges of rows per workgroup, runs without padding whose
length is no multiple of a vector, and the last row at the end of its buffer; and that a narrow table takes no longer than its
bytes do."""
import numpy as np
import pytest
import torch

from oracle import storage as ost
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl

pytestmark = pytest.mark.gpu


def store(fmt, n, F, src, ld, dst, ld16):
    B.check(B.retexo_store_rows(B.STORAGE[fmt], n, F, src.data_ptr(), ld, dst.data_ptr(), ld16, Hn._stream_ptr()), "retexo_store_rows")


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("F", [1, 2, 3, 5, 8, 17, 31, 64, 65, 130, 255, 257, 258, 603])
@pytest.mark.parametrize("n", [1, 2, 129, 1025, 4097])
def test_exact(fmt, F, n):
    X = wl.random_matrix(n, F, n + F, ld=F)
    want = ost.store(X, fmt)
    up = -(-F // 4) * 4
    for ld, ld16 in [(F, F), (up, up), (up + 4, up + 8), (F + 1, F + 3), (up, F + 1)]:
        src = torch.full((n, ld), float("nan"), device="cuda")
        src[:, :F] = Hn.dev(X)
        src = src.reshape(-1)[:(n - 1) * ld + F].clone()          # ends with the last row's last element
        dst = torch.full((n, ld16), 77, dtype=torch.int16, device="cuda")
        store(fmt, n, F, src, ld, dst, ld16)
        got = dst.cpu().numpy().view(np.uint16)
        assert np.array_equal(got[:, :F], want) and np.all(got[:, F:] == 77), (ld, ld16)


@pytest.mark.parametrize("ld", [8, 9])
def test_narrow_rows_take_no_longer_than_their_bytes(ld):
    """The same number of elements in rows of 8 and of 256: about 20 us both on an MI355X; with a wave for each row of 8 more than
    110.  The line lies between."""
    def time(n, F, ld):
        src = torch.zeros(n * ld, device="cuda")
        dst = torch.zeros(n * ld, dtype=torch.int16, device="cuda")
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                store("bf16", n, F, src, ld, dst, ld)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    wide, narrow = time(1 << 16, 256, 256), time(1 << 21, 8, ld)
    assert narrow <= 3 * wide, (narrow, wide)
