"""Solves of several host threads, each on a stream of its own, whose launches each need many
workgroups resident on one XCD at once: the results are those of one call after another, and no
launch gave up its workgroups."""
import threading

import pytest
import torch

from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(300, 520, 700, 1100, 1500, 2048), (2304, 3000, 4096, 2200)])
def test_threads_equal_one_after_another(sizes):
    print(f"concurrent {sizes}", flush=True)
    mats = [torch.from_numpy(I.nearly_diagonal(n, 50 + n, 1e-11).a).to("cuda") for n in sizes]

    def solve(a, stream=None):
        return J.eigh(a, tol=1e-13, precond="none", max_rotations=3000, stream=stream)

    ref = [solve(a) for a in mats]
    out = [None] * len(mats)
    torch.cuda.synchronize()

    def work(i):
        s = torch.cuda.Stream()
        out[i] = solve(mats[i], s)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(mats))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
        assert not t.is_alive()
    for r, o in zip(ref, out):
        assert o.stats["jacobi_wgs"] == r.stats["jacobi_wgs"] > 1
        assert o.stats["rotations"] == r.stats["rotations"] > 0
        assert torch.equal(o.w, r.w) and torch.equal(o.v, r.v)


def test_svd_threads_equal_one_after_another():
    mats = [torch.from_numpy(I.svd_graded(m, n, seed=m, decades=4.0)).to("cuda")
            for m, n in ((1024, 256), (700, 511), (300, 200), (512, 257))]

    def solve(b, stream=None):
        return J.svd(b, pivot="gap", precond="none", max_rotations=300, stream=stream)

    ref = [solve(b) for b in mats]
    out = [None] * len(mats)
    torch.cuda.synchronize()

    def work(i):
        s = torch.cuda.Stream()
        out[i] = solve(mats[i], s)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(mats))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
        assert not t.is_alive()
    for r, o in zip(ref, out):
        assert torch.equal(o.s, r.s) and torch.equal(o.u, r.u) and torch.equal(o.v, r.v)
