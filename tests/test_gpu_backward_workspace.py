"""Scratch memory of the edge softmax's backward: scores, gradients of scores and statistics of every node, and one block of the
attention vectors' partial sums per 256 rows (up to 2,048 blocks).  A caller that keeps a buffer of that size is not refused, and
nothing past it is written, whichever width bounds the number of blocks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl
from parity import assert_close
from test_gpu_softmax_rows import decided_rows

pytestmark = pytest.mark.gpu


def up(x):
    return -(-x // 256) * 256


@pytest.mark.parametrize("n,heads,dh", [(1, 1, 4), (33, 1, 5), (1003, 2, 32), (1003, 8, 16), (2049, 4, 73), (2049, 4, 74), (1003, 1, 1024),
                                        (1003, 8, 128), (70001, 1, 4)])
@pytest.mark.parametrize("save", [False, True])
def test_workspace_of_one_block_per_256_rows(n, heads, dh, save):
    F, hp, fill = heads * dh, 4 if heads <= 4 else 8, 0x5a
    size = 4 * up(n * hp * 4) + up(n * hp * 16) + up(min(-(-n // 256), 2048) * 2 * F * 4)
    src, dst = wl.random_pairs(n, 4 * n, 1, skew=0.5)
    g = Hn.make_plan(Hn.csr_from_coo(Hn.dev(src), Hn.dev(dst), n, True))
    rp, ci = oracle.csr_from_coo(src, dst, n, True)
    mode = B.MODES["gat_softmax"]
    assert B.retexo_aggregate_backward_workspace_bytes(g.plan, mode, F, heads) == size
    a = [wl.random_matrix(heads, dh, k) * np.float32(0.1) for k in (1, 2)]
    Zh, Gh = decided_rows(rp, ci, heads, dh, a), wl.random_matrix(n, F, 4)
    Z, G, As, Ad = (Hn.dev(x) for x in (Zh, Gh, *a))
    saved = None
    if save:
        saved = Hn.ws_tensor(B.retexo_workspace_bytes(g.plan, F, mode, heads, B.F_SAVE))
        Hn.aggregate(g, "gat_softmax", Z, F, heads=heads, a_src=As, a_dst=Ad, workspace=saved, save=True)
        kept = saved.clone()
    buf = torch.full((size + 4096,), fill, dtype=torch.uint8, device="cuda")
    got = Hn.aggregate_backward(g, "gat_softmax", F, G, Z=Z, heads=heads, a_src=As, a_dst=Ad, saved=saved, workspace=buf[:size])
    assert bool((buf[size:] == fill).all()) and (saved is None or torch.equal(saved, kept))
    want = oracle.aggregate_backward("gat_softmax", rp, ci, np.ascontiguousarray(Zh[:, :F]), F, Gh, heads=heads, a_src=a[0], a_dst=a[1])
    for grad, ref, what in zip(got, want, ("Z", "source", "destination")):
        grad = grad.cpu().numpy()
        grad = grad[:, :F] if what == "Z" else grad
        assert_close(grad.reshape(1, -1), ref.reshape(1, -1), what="gradient of " + what)
    g.destroy()
