"""The FP32 stage with either block size at the edges of its blocks: one subproblem that is the
whole matrix, a padded last block, an odd number of blocks, and both sides of the automatic
choice."""
import pytest
import torch

from paper_2607_23187_amd import inputs as I
from paper_2607_23187_amd import jacobi as J

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.mark.parametrize("n", [2, 15, 31, 32, 33, 47, 63, 64, 65, 96, 97, 200, 1024, 1025])
@pytest.mark.parametrize("block", [0, 16, 32])
def test_block_edges(n, block):
    print(f"fp32 blocks n={n} block={block}", flush=True)
    a = torch.from_numpy(I.random_symmetric(n, 4100 + n))
    r = J.eigh(a.to("cuda"), tol=1e-14, fp32_block=block)
    norm = float(a.norm())
    # the stage ends with off-diagonal entries of FP32 rounding size: 2^-22 of the norm in each
    # of the n rows at most
    assert r.stats["a_hat_off"] <= n * 2.0 ** -22 * norm
    w = torch.linalg.eigvalsh(a)
    assert float((r.w.cpu() - w).abs().max()) <= 10 * n * U * norm
    v = r.v.cpu()
    # (the stop rule bounds eigenvalue errors, not residuals: V is held to its polish)
    assert float((v.T @ v - torch.eye(n, dtype=v.dtype)).norm()) <= 8 * n * U
    b = J.eigh_batched([a.to("cuda")] * 2, tol=1e-14, fp32_block=block)[1]
    assert torch.equal(b[0].w, b[1].w) and torch.equal(b[0].v, b[1].v)
    assert float((b[0].w.cpu() - w).abs().max()) <= 10 * n * U * norm
