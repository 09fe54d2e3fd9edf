"""The overlap kernels at the edges of their column counts (8, 16, .. 40), with an odd last
path where a wavefront takes two, against the FP64 oracle: log-overlaps alone and with the Green's function, the diagonal, a
path of zero overlap and one with an infinite entry.  Tolerance 1e-10, as for every
FP64 overlap; the log-overlaps with and without Theta come from the same pivots
and products and agree to 1e-13."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10

# (M, N): up to and past M = 64, N = 16
SIZES = [(1, 1), (8, 2), (17, 8), (30, 9), (64, 16), (63, 15), (65, 1), (72, 7), (80, 8), (97, 9), (66, 16),
         (20, 17), (24, 24), (90, 25), (33, 32), (129, 33), (160, 40)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("cplx", [False, True])
def test_columns(size, cplx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N = size
    print("overlap columns", size, cplx, flush=True)
    sys.stdout.flush()
    P, nw = 3, 3
    s = ai.small_gaussian(M=M, N=N, n_chol=4, K=3, seed=M + N)
    if cplx:
        s = ai.imaginary_time_trial(s, 1, 0.05)
    rng = np.random.default_rng(5)
    phiT = O.trial_det(s, 0.5 * rng.normal(size=(nw, P, s.K)))
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    ell, theta = O.green(phiT, phi)
    try:
        ctx = A.Context(s, P, 0.01, max_walkers=nw)
    except A.AfqmcError as e:
        assert cplx and "E_UNSUPPORTED" in str(e)
        pytest.skip("past the complex trial's size limit")
    z = dict(dtype=torch.complex128, device="cuda")
    l0, l1 = torch.zeros(nw, P, **z), torch.zeros(nw, P, **z)
    th = torch.zeros(nw, P, 2, M, N, **z)
    A.afqmc_overlap(ctx, nw, dev(phi), dev(phiT), l0)
    A.afqmc_green(ctx, nw, dev(phi), dev(phiT), l1, th)
    torch.cuda.synchronize()
    g0, g1, gt = l0.cpu().numpy(), l1.cpu().numpy(), th.cpu().numpy()
    for g in (g0, g1):
        assert np.abs(np.exp(g - ell) - 1).max() <= TOL
    assert np.abs(g0 - g1).max() <= 1e-13 * max(1.0, np.abs(g1).max())
    assert np.linalg.norm(gt - theta) <= TOL * np.linalg.norm(theta)
    # a zero column: no overlap; an infinite entry: not a number
    bad = phiT.copy()
    bad[0, 1, :, 0] = 0.0
    bad[1, 2, M // 2, N - 1] = np.inf
    A.afqmc_overlap(ctx, nw, dev(phi), dev(bad), l0)
    A.afqmc_green(ctx, nw, dev(phi), dev(bad), l1, th)
    torch.cuda.synchronize()
    for l in (l0, l1):
        g = l.cpu().numpy()
        assert np.isneginf(g[0, 1].real) and g[0, 1].imag == 0
        assert np.isnan(g[1, 2].real) and np.isnan(g[1, 2].imag)
        keep = np.ones((nw, P), bool)
        keep[0, 1] = keep[1, 2] = False
        assert np.abs(np.exp(g - ell) - 1)[keep].max() <= TOL
    gt = th.cpu().numpy()
    assert not gt[0, 1].any() and not gt[1, 2].any()
    assert np.linalg.norm(gt[keep] - theta[keep]) <= TOL * np.linalg.norm(theta[keep])
