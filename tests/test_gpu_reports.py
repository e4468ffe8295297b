"""Result words of constructions, plans and shares that threads on streams of their own make at the same time: more threads
than there are pieces of host memory for them."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2302_13053_amd import binding as B
from paper_2302_13053_amd import harness as Hn
from paper_2302_13053_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_many_threads():
    wrong, sizes = [], [(50 + 37 * t, 200 + 101 * t) for t in range(40)]
    want = []
    for n, pairs in sizes:
        src, dst = wl.random_pairs(n, pairs, n)
        want.append((src, dst, *oracle.csr_from_coo(src, dst, n, False)))
    gate = threading.Barrier(len(sizes))

    def work(t):
        n, (src, dst, rp, ci) = sizes[t][0], want[t]
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                s, d = Hn.dev(src), Hn.dev(dst)
                gate.wait()
                for _ in range(5):
                    g = Hn.make_plan(Hn.csr_from_coo(s, d, n, False))
                    deg = np.diff(rp)
                    if g.nnz != rp[-1] or B.retexo_plan_max_degree(g.plan) != deg.max(initial=0):
                        wrong.append(t)
                    if not np.array_equal(g.col_idx[:g.nnz].cpu().numpy(), ci):
                        wrong.append(t)
                    g.destroy()
        except Exception as e:                                # a thread's exception must not be lost
            wrong.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


def test_errors_are_reported():
    src = Hn.dev(np.array([0, 1, 5], np.int32))
    for n, want in ((6, None), (5, B.E_CSR)):
        if want is None:
            assert Hn.csr_from_coo(src, src.roll(1), n, False).nnz == 6
        else:
            with pytest.raises(B.RetexoError):
                Hn.csr_from_coo(src, src.roll(1), n, False)
