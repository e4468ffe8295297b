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


def eight_slices(H, W):
    """H W with every sum as eight slices of k, each one chain of float32 multiply-adds: what a call over few rows is held to."""
    def chain(h, w):
        acc = np.zeros((h.shape[0], w.shape[1]), np.float32)
        for k in range(h.shape[1]):               # (products of two float32 are exact in 64 bits)
            acc = (acc.astype(np.float64) + h[:, k, None].astype(np.float64) * w[None, k].astype(np.float64)).astype(np.float32)
        return acc
    per = -(-(-(-H.shape[1] // 8)) // 8) * 8
    s = [chain(H[:, i * per:(i + 1) * per], W[i * per:(i + 1) * per]) for i in range(8)]
    s = [s[i] + s[i + 4] for i in range(4)]
    return ((s[0] + s[1]) + s[2]) + s[3]


@pytest.mark.parametrize("n,d_in,d_out", [
    (2708, 1433, 64), (4000, 2001, 31), (2708, 1201, 126), (2700, 1327, 99), (1400, 1999, 200), (2708, 1202, 255),   # few rows
    (14500, 129, 64), (14500, 700, 33),                                                                            # (832 tiles and more)
    (5000, 16, 300), (5000, 65, 301), (2708, 127, 500), (5000, 131, 301), (8000, 257, 256), (14000, 193, 250), (2708, 1203, 500),
    (4800, 700, 200)])                                                                                             # blocks
def test_terms_of_unlike_size(n, d_in, d_out):
    """[self | aggregate]: a few large terms, then many small ones.  As close to 64 bits as eight slices of k are, on the first rows and
    columns, and every element against the size of its terms."""
    half = d_in // 2
    H = np.abs(wl.random_matrix(n, d_in, d_in)) * np.float32(0.05)
    H[:, :half] = wl.random_matrix(n, half, 7) > 2.2
    W, b = wl.random_matrix(d_in, d_out, d_out) * np.float32(0.05), np.zeros(d_out, np.float32)
    got = Hn.transform(Hn.dev(H), d_in, Hn.dev(W), Hn.dev(b), False).cpu().numpy()[:, :d_out]
    want = H.astype(np.float64) @ W.astype(np.float64)
    assert_cond_close(got, want, H.astype(np.float64) @ np.abs(W).astype(np.float64), what="transform")
    r, c = slice(0, 256), slice(0, min(d_out, 64))
    err = lambda x: np.linalg.norm(x - want[r, c]) / np.linalg.norm(want[r, c])
    limit = err(eight_slices(H[r], W[:, c]))
    assert err(got[r, c]) <= 1.02 * limit, "%.2e, eight slices %.2e" % (err(got[r, c]), limit)
