"""Which kernel of the one-sided SVD ran: the workgroups that held B in LDS, 0 when B stayed in
device memory.  All of them give the same bits, so the results alone would not show a launch that
gave up its workgroups."""
import threading

import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu


# one LDS; slices of four to sixteen columns on up to 32 workgroups;
# B in device memory (both sides of the largest slice at n = 512)
@pytest.mark.parametrize("m,n,wgs,cap", [
    (2, 2, 1, 100), (100, 100, 1, 300), (128, 128, 1, 300), (1500, 8, 1, 300),
    (3953, 3, 1, 100), (3954, 3, 1, 100), (4066, 3, 1, 100), (4067, 3, 0, 100),
    (4917, 2, 1, 100), (5001, 2, 1, 100), (3300, 4, 1, 300), (4001, 4, 0, 100), (2500, 6, 2, 300),
    (130, 129, 26, 300), (512, 257, 29, 200),
    (700, 511, 32, 60), (1024, 512, 32, 60), (1088, 512, 32, 20), (1089, 512, 0, 20),
    (800, 768, 0, 20)])
@pytest.mark.parametrize("precond", ["none", "fp32"])
def test_workgroups(m, n, wgs, cap, precond):
    print(f"svd route m={m} n={n} precond={precond}", flush=True)
    b = I.svd_graded(m, n, seed=900 + n, decades=4.0)
    g = J.svd(torch.from_numpy(b).to("cuda"), max_rotations=cap, precond=precond)
    assert g.stats["jacobi_wgs"] == wgs
    if precond == "none":
        o = O.svd(b, 2.0 ** -53, pivot=O.GAP, abs_thr=g.stats["thr"], logcap=cap, maxrot=cap)
        assert g.stats["rotations"] == o.rotations
        assert np.array_equal(g.s.cpu().numpy(), o.s)
        assert np.array_equal(g.u.cpu().numpy(), o.u)
        assert np.array_equal(g.v.cpu().numpy(), o.v)


def test_threads_keep_their_workgroups():
    shapes = [(1024, 256), (700, 511), (300, 200), (512, 257)]
    mats = [torch.from_numpy(I.svd_graded(m, n, seed=m, decades=4.0)).to("cuda")
            for m, n in shapes]
    out = [None] * len(mats)
    torch.cuda.synchronize()

    def work(i):
        s = torch.cuda.Stream()
        out[i] = J.svd(mats[i], max_rotations=300, stream=s).stats["jacobi_wgs"]
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(mats))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
        assert not t.is_alive()
    assert out == [32, 32, 29, 29]


# up to eight columns the entries of A are stored as they change, above that formed at the end
@pytest.mark.parametrize("n", [2, 3, 5, 8, 9, 16])
@pytest.mark.parametrize("cap", [1, 2, 7])
def test_final_off_norm(n, cap):
    m = 200
    print(f"svd off-norm n={n} cap={cap}", flush=True)
    g = J.svd(torch.from_numpy(I.svd_graded(m, n, seed=40 + n, decades=2.0)).to("cuda"),
              max_rotations=cap)
    b = (g.u * g.s).cpu().numpy()
    a = b.T @ b
    off = np.linalg.norm(a - np.diag(np.diag(a)))
    # sums of m products on either side; U is B's columns divided by S, one rounding more
    assert abs(g.stats["final_off"] - off) <= 4 * m * 2.0 ** -53 * np.linalg.norm(a)
