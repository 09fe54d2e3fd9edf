"""The re-orthonormalisation at the edges of its row groups and column counts, against
numpy's QR with a positive diagonal of R: one orbital, rows off the groups' multiples, N on
either side of 16 and 32, M on either side of 64, 80 and 128.  Tolerance 1e-12: twice-applied
Gram-Schmidt is orthonormal to a few 1e-16 per column at these condition numbers
(below 100)."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12

SIZES = [(1, 1), (2, 2), (16, 16), (63, 15), (64, 1), (64, 17), (80, 32), (81, 20), (65, 16),
         (128, 9), (128, 31), (129, 16), (160, 17), (130, 32), (40, 33), (160, 40)]


@pytest.mark.parametrize("size", SIZES)
def test_groups(size):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N = size
    print("qr groups", size, flush=True)
    sys.stdout.flush()
    P, nw = 2, 3
    s = ai.small_gaussian(M=M, N=N, n_chol=4, K=3, seed=M + N)
    phi = ai.random_walkers(np.random.default_rng(5), s, nw, spread=0.5)
    q, r = np.linalg.qr(phi)
    d = np.diagonal(r, axis1=-2, axis2=-1)
    q = q * (d / np.abs(d))[..., None, :]
    shift = np.log(np.abs(d)).sum((-1, -2))
    ctx = A.Context(s, P, 0.01, max_walkers=nw)
    x = torch.as_tensor(phi).cuda()
    lo = torch.full((nw, P), 0.5 + 0.25j, dtype=torch.complex128, device="cuda")
    A.afqmc_reorthogonalize(ctx, nw, x, lo)
    torch.cuda.synchronize()
    assert np.abs(x.cpu().numpy() - q).max() <= TOL
    assert np.abs(lo.cpu().numpy() - (0.5 + 0.25j - shift[:, None])).max() <= TOL * max(1, N)
    # without log-overlaps
    y = torch.as_tensor(phi).cuda()
    A.afqmc_reorthogonalize(ctx, nw, y, None)
    torch.cuda.synchronize()
    assert torch.equal(x, y)
