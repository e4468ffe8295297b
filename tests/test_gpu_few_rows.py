"""Dense transform of few rows over long sums (operands through LDS in chunks of 128 k): shapes at the edges of its tiles and
chunks and of the rules that lead there, rows at any alignment, garbage past the rows, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_cond_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d_in,d_out,ld,offset", [
    (1, 768, 4, 768, 0), (31, 769, 5, 771, 1), (32, 771, 31, 776, 0), (33, 895, 32, 897, 3), (95, 896, 33, 896, 0),
    (2708, 1433, 63, 1440, 0), (70, 1025, 3, 1025, 2), (2600, 256, 100, 257, 1), (2600, 383, 126, 384, 0), (26624, 257, 30, 260, 0),
    (26600, 300, 33, 300, 0), (500, 64, 2866, 64, 0), (5000, 300, 300, 301, 1), (14000, 260, 200, 260, 0)])
@pytest.mark.parametrize("relu", [False, True])
def test_long_sums_of_few_rows(n, d_in, d_out, ld, offset, relu):
    Hh = np.full((n, ld), np.nan, np.float32)                 # what lies past a row must not reach a sum
    Hh[:, :d_in] = wl.random_matrix(n, d_in, d_in)
    buf = torch.full((n * ld + offset + 8,), float("nan"), device="cuda")
    H = buf[offset:offset + n * ld].view(n, ld)
    H.copy_(torch.from_numpy(Hh))
    W, b = wl.random_matrix(d_in, d_out, d_out), wl.random_matrix(1, d_out, 3)[0]
    out = torch.full((n, d_out + 5), 777.0, device="cuda")
    Hn.transform(H, d_in, Hn.dev(W), Hn.dev(b), relu, out=out)
    got = out.cpu().numpy()
    assert np.all(got[:, d_out:] == 777.0)
    want = oracle.transform(Hh[:, :d_in], d_in, W, b, relu)
    # an element against the size of the terms it is the sum of
    mag = np.abs(Hh[:, :d_in]).astype(np.float64) @ np.abs(W).astype(np.float64) + np.abs(b)
    assert_cond_close(got[:, :d_out], want, mag, what="transform")
