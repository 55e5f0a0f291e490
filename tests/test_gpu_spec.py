"""Speculative rounds of the FP64 phase: several rotations per exchange of candidates perform
the oracle's rotations, in its order, with its bits.  Without the preconditioner and the polish
both sides run the same IEEE operations, so pivots, W and V are compared exactly."""
import sys

import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def check(a, pivot, stop, thr, cap=None, **kw):
    n = a.shape[0]
    print("spec", n, pivot, stop, kw, flush=True)
    sys.stdout.flush()
    logcap = cap or 40 * n * n + 64
    r = J.eigh(torch.from_numpy(a).to("cuda"), precond="none", pivot=pivot, stop=stop, abs_thr=thr,
               pivot_log_cap=logcap, polish_v=False, max_rotations=cap or 0, **kw)
    so = {"cert": O.STOP_CERT, "score": O.STOP_SCORE}[stop]
    ref = O.jacobi(a, pivot=O.GAP if pivot == "gap" else O.GREEDY, stop=so, thr=thr, maxrot=cap,
                   scan=1, want_vj=True, logcap=logcap)
    d = np.diag(ref.a)
    order = np.argsort(d, kind="stable")
    assert r.stats["rotations"] == ref.rotations
    assert np.array_equal(r.pivots.cpu().numpy(), ref.pivots)
    assert np.array_equal(r.w.cpu().numpy(), d[order])
    assert np.array_equal(r.v.cpu().numpy(), ref.vj[:, order])
    return ref


def nearly(n, eps):
    p = I.nearly_diagonal(n, 7100 + n, eps)
    return p.a, 10 * n * U * float(p.lam.max()) / (2.0 * n * (n - 1))


# edges of the shapes: 16-lane groups, waves, LDS-resident up to 128, 256 / 512 threads, one and
# two rows per lane
@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 63, 64, 65, 127, 128, 129, 256, 257, 385])
@pytest.mark.parametrize("pivot,stop", [("gap", "cert"), ("gap", "score"), ("greedy", "score")])
def test_one_workgroup(n, pivot, stop):
    a, thr = nearly(n, 1e-9)
    check(a, pivot, stop, thr if stop == "cert" else 1e3 * thr, cap=6000, jacobi_wgs="one",
          update_mode="timestamp" if n == 257 else "auto")


# one row per lane up to 64 workgroups (n = 4096), two above; partly filled workgroups
@pytest.mark.parametrize("n", [130, 399, 400, 513, 1025, 2049, 4096, 4097])
@pytest.mark.parametrize("pivot,stop", [("gap", "cert"), ("greedy", "score")])
def test_several_workgroups(n, pivot, stop):
    a, thr = nearly(n, 1e-9 if n < 1000 else 1e-12)
    ref = check(a, pivot, stop, thr if stop == "cert" else 1e3 * thr,
                cap=6000 if n < 2000 else 2500, jacobi_wgs="many")
    assert ref.rotations > 100


# equal scores throughout (identical blocks), at the start (equispaced diagonal, equal entries)
# and tight clusters, where the next pivot mostly lies in the rows just rotated
@pytest.mark.parametrize("n", [36, 68, 132, 260])
@pytest.mark.parametrize("kind", ["blocks", "equal", "cluster"])
@pytest.mark.parametrize("wgs", ["one", "many"])
def test_ties_and_clusters(n, kind, wgs):
    if kind == "blocks":
        b = I.random_symmetric(4, 5)
        a = np.kron(np.eye(n // 4), b)
    elif kind == "equal":
        a = np.full((n, n), 2.0 ** -20) + np.diag(np.arange(n, dtype=np.float64))
    else:
        a = I.clustered(n, 7200 + n, n // 2, 1e-9).a
    thr = 10 * n * U * float(np.abs(a).max()) / (2.0 * n * (n - 1))
    ref = check(np.ascontiguousarray(a), "gap", "cert", thr, jacobi_wgs=wgs)
    assert ref.status == O.OK


# a rotation cap inside a round, a log drained inside a solve (batch members hold 2^16 entries)
@pytest.mark.parametrize("cap", [1, 2, 3, 50, 51, 52, 53])
def test_caps(cap):
    a, thr = nearly(150, 1e-9)
    for wgs in ("one", "many"):
        check(a, "gap", "cert", thr, cap=cap, jacobi_wgs=wgs)


def test_batch_members_equal_single_solves():
    # without the polish, whose products are tiled differently in a batch
    sizes = [20, 64, 65, 128, 200, 300, 513, 1100, 2100]
    mats = [torch.from_numpy(nearly(n, 1e-11)[0]).to("cuda") for n in sizes]
    for mode in ("mirror", "timestamp"):
        _, rs = J.eigh_batched(mats, precond="none", polish_v=False,
                               update_mode=mode, max_rotations=3000)
        for n, m, r in zip(sizes, mats, rs):
            s = J.eigh(m, precond="none", polish_v=False, max_rotations=3000)
            assert r.stats["rotations"] == s.stats["rotations"], n
            assert torch.equal(r.w, s.w), n
            assert torch.equal(r.v, s.v), n
