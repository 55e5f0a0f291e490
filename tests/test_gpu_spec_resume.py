"""Speculative rounds that end on a full rotation log and resume from the state they wrote back
(rows rotated since their last scan hold no candidate of their own): the rotations, W and V are
those of a call whose log holds all of them.  jacobi_eigh_noalloc's log holds 2^16 rotations, a
batch member's too; jacobi_eigh_ex's holds these problems' rotations at once."""
import pytest
import torch

from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu
LOG = 1 << 16


# one and several workgroups; 3 n^2 rotations and more from a dense start, the cap inside the
# third log (and the last of it right at the end of a log)
@pytest.mark.parametrize("n,wgs", [(200, "one"), (300, "one"), (300, "many"), (512, "many")])
@pytest.mark.parametrize("cap", [2 * LOG + 1001, 2 * LOG])
def test_log_drained_twice(n, wgs, cap):
    print(f"resume n={n} wgs={wgs} cap={cap}", flush=True)
    a = torch.from_numpy(I.random_symmetric(n, 8200 + n)).to("cuda")
    kw = dict(tol=1e-15, precond="none", polish_v=False, max_rotations=cap, jacobi_wgs=wgs,
              pivot_log_cap=cap)
    once = J.eigh(a, **kw)
    drained = J.eigh(a, noalloc=True, **kw)
    assert once.stats["jacobi_wgs"] == drained.stats["jacobi_wgs"]
    assert (once.stats["jacobi_wgs"] > 1) == (wgs == "many")
    assert drained.stats["rotations"] == once.stats["rotations"] > LOG
    assert torch.equal(drained.pivots, once.pivots)
    assert torch.equal(drained.w, once.w)
    assert torch.equal(drained.v, once.v)


def test_batch_members_drained():
    sizes = [200, 300, 512, 600]
    mats = [torch.from_numpy(I.random_symmetric(n, 8300 + n)).to("cuda") for n in sizes]
    kw = dict(tol=1e-15, precond="none", polish_v=False, max_rotations=LOG + 501)
    for mode in ("mirror", "timestamp"):
        _, rs = J.eigh_batched(mats, update_mode=mode, **kw)
        for n, a, r in zip(sizes, mats, rs):
            s = J.eigh(a, **kw)
            assert r.stats["rotations"] == s.stats["rotations"], n
            assert torch.equal(r.w, s.w) and torch.equal(r.v, s.v), n
    assert max(r.stats["rotations"] for r in rs) == LOG + 501
