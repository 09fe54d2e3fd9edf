"""The back-propagated density at the edges of its tiles, against the FP64 oracle:
one orbital, orbitals on, below and past a multiple of 16 on either side of the one-
and two-tile forms, the largest system, electrons off the multiple of 4, 64 paths, a
path without overlap, and walker counts around the sixteen that the sum over the
walkers reads at a time.  Tolerance 1e-10, as for the other density tests."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10

# (M, N, paths, walkers)
SHAPES = [(1, 1, 1, 1), (5, 3, 2, 16), (16, 4, 64, 2), (17, 5, 3, 15), (48, 9, 2, 17),
          (64, 2, 5, 33), (65, 7, 2, 3), (97, 3, 2, 2), (160, 6, 3, 2)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("shape", SHAPES)
def test_edges(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    from paper_2505_18519_amd import driver as D
    M, N, P, nw = shape
    print("bp tiles", shape, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=5, K=3, seed=M + N)
    rng = np.random.default_rng(8)
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    phiT = O.trial_det(s, 0.7 * rng.normal(size=(nw, P, s.K)))
    logov = O.log_overlap(phiT, phi)
    if P > 1:
        logov[-1, 0] = complex(-np.inf, 0.0)
    w = rng.uniform(0.5, 1.5, size=nw)
    hx, hb = np.zeros((nw, 0, 5)), np.zeros((nw, 0, 5), dtype=complex)
    num, den, Rk = O.back_propagated_density(s, phi, hx, hb, phiT, logov, w, 0.01, 10)
    ctx = A.Context(s, P, 0.01, max_walkers=nw)
    bp = D.BackProp(ctx, nw, 1)
    out = torch.zeros(M * M + 1, dtype=torch.float64, device="cuda")
    A.afqmc_bp_density(ctx, nw, 0, dev(phi), None, None, dev(phiT), dev(logov), dev(w), bp.phit_bp,
                       bp.theta_bp, bp.logov_bp, bp.rho, out)
    torch.cuda.synchronize()
    g = out.cpu().numpy()
    assert np.abs(g[:-1].reshape(M, M) - num).max() <= TOL * np.abs(num).max()
    assert abs(g[-1] - den) <= 1e-14 * den
    assert np.abs(bp.rho.cpu().numpy() - Rk).max() <= TOL * np.abs(Rk).max()
