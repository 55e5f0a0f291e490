"""The one-sided SVD with B in LDS: the oracle's pivots, rescans, S, U and V bit for bit at the
edges of its blocks (8 and 16 terms, 64 lanes, 128 columns, more rows than lanes), from a single
pair of columns on, and with equal scores throughout."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu
U = 2.0 ** -53
PIVOTS = [("gap", O.GAP, U), ("relative", O.RELATIVE, U), ("greedy", O.GREEDY, 1e-11)]


def check(b, pivot, piv_o, tol, cap):
    print(f"svd res {b.shape} pivot={pivot}", flush=True)
    g = J.svd(torch.from_numpy(b).to("cuda"), tol=tol, pivot=pivot, pivot_log_cap=cap,
              max_rotations=cap)
    o = O.svd(b, tol, pivot=piv_o, abs_thr=g.stats["thr"], logcap=cap, maxrot=cap)
    assert g.stats["rotations"] == o.rotations
    assert g.stats["rescans"] == o.rescans
    assert np.array_equal(g.pivots.cpu().numpy(), o.pivots[:cap])
    assert np.array_equal(g.s.cpu().numpy(), o.s)
    assert np.array_equal(g.u.cpu().numpy(), o.u)
    assert np.array_equal(g.v.cpu().numpy(), o.v)


@pytest.mark.parametrize("m,n", [(1, 1), (2, 2), (7, 3), (8, 8), (15, 9), (16, 16), (17, 17),
                                 (63, 63), (65, 64), (66, 65), (100, 99), (127, 127), (128, 128),
                                 (150, 128), (129, 100), (257, 60), (600, 30), (1500, 8)])
@pytest.mark.parametrize("pivot,piv_o,tol", PIVOTS)
def test_edges_match_oracle(m, n, pivot, piv_o, tol):
    check(I.svd_graded(m, n, seed=700 + m + n, decades=5.0), pivot, piv_o, tol, 1500)


@pytest.mark.parametrize("n", [12, 66, 128])
@pytest.mark.parametrize("pivot,piv_o,tol", PIVOTS)
def test_equal_scores_match_oracle(n, pivot, piv_o, tol):
    block = I.svd_graded(6, 3, seed=9, decades=1.0)[:3 + n % 2, :2 + n % 2]
    k = n // block.shape[1]
    check(np.ascontiguousarray(np.kron(np.eye(k), block)), pivot, piv_o, tol, 1500)
