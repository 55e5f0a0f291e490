"""The one-sided SVD on several workgroups (B beyond one LDS): the oracle's pivots, S, U and V
bit for bit at the edges of its slices (4 to 16 columns per workgroup, a partial last one, odd
row counts below and above the 16 rows in flight)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.mark.parametrize("m,n,cap", [(130, 129, 1500), (331, 150, 1500), (1009, 33, None),
                                     (4001, 4, None), (2500, 6, None), (512, 257, 400),
                                     (1024, 512, 150), (700, 511, 150)])
@pytest.mark.parametrize("pivot,piv_o,tol", [("gap", O.GAP, U), ("relative", O.RELATIVE, U),
                                             ("greedy", O.GREEDY, 1e-11)])
def test_several_workgroups_match_oracle(m, n, cap, pivot, piv_o, tol):
    print(f"svd mw m={m} n={n} pivot={pivot}", flush=True)
    b = I.svd_graded(m, n, seed=600 + n, decades=6.0)
    if cap is None and pivot == "greedy":
        cap = 2000
    lc = cap or 40 * n * n + 64
    g = J.svd(torch.from_numpy(b).to("cuda"), tol=tol, pivot=pivot, pivot_log_cap=lc,
              max_rotations=cap or 0)
    o = O.svd(b, tol, pivot=piv_o, abs_thr=g.stats["thr"], logcap=lc, maxrot=cap)
    assert g.stats["rotations"] == o.rotations > 0
    assert g.stats["rescans"] == o.rescans
    assert np.array_equal(g.pivots.cpu().numpy(), o.pivots[:lc])
    assert np.array_equal(g.s.cpu().numpy(), o.s)
    assert np.array_equal(g.u.cpu().numpy(), o.u)
    assert np.array_equal(g.v.cpu().numpy(), o.v)
