"""The FP64 Taylor propagation with all columns of a V side by side, against the
FP64 oracle: every number of row tiles, electrons that leave the last column
tile ragged, one to several workgroups per V, and V shared by the paths of a
back-propagation or owned by each trial slice; enough walkers that this form is
the one chosen.  Tolerances of the FP64 path."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("M,N,nw", [(18, 17, 60), (40, 18, 58), (50, 20, 55), (66, 3, 257),
                                    (72, 6, 130), (81, 21, 45), (100, 25, 37), (128, 24, 43),
                                    (130, 35, 29), (150, 36, 29)])
def test_walker_move(M, N, nw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    print("walker move", M, N, nw, flush=True)
    s = ai.small_gaussian(M=M, N=N, n_chol=7, K=3, seed=M)
    rng = np.random.default_rng(M)
    phi, P, dtau = ai.random_walkers(rng, s, nw, spread=0.5), 1, 0.01
    phiT = O.trial_det(s, ai.random_hidden(rng, s, nw, P))
    eloc, xbar, ep, vb, ell = O.local_energy(s, phi, phiT, dtau)
    xi, w0 = rng.normal(size=(nw, s.n_chol)), np.ones(nw)
    phin, wn, ref, elln = O.propagate(s, phi, xi, xbar, phiT, ell, w0, dtau, 10, 0.0, 0, eloc=eloc)
    ctx = A.Context(s, P, dtau, max_walkers=nw)
    dphi, dw = dev(phi), dev(w0)
    dref = torch.zeros(nw, dtype=torch.complex128, device="cuda")
    dln = torch.zeros(nw, P, dtype=torch.complex128, device="cuda")
    A.afqmc_propagate(ctx, nw, dphi, dev(xi), dev(xbar), dev(phiT), dev(ell), 0.0, dw, dref, dln,
                      dev(eloc))
    torch.cuda.synchronize()
    for w in range(nw):
        assert rel(host(dphi)[w], phin[w]) <= TOL
    assert np.abs(host(dw) - wn).max() <= TOL * np.abs(wn).max()


@pytest.mark.parametrize("M,N,nw,P,m", [(20, 5, 65, 4, 2), (37, 11, 64, 2, 1), (96, 3, 128, 2, 1)])
def test_trial_slices(M, N, nw, P, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    print("trial slices", M, N, nw, P, m, flush=True)
    s = ai.imaginary_time_trial(ai.small_gaussian(M=M, N=N, n_chol=6, K=3, seed=M), m, 0.05)
    y = np.random.default_rng(M).normal(size=(nw, P, s.K))
    ref = O.trial_det(s, y)
    ctx = A.Context(s, P, 0.01, max_walkers=nw)
    got = torch.zeros(nw, P, M, N, dtype=torch.complex128, device="cuda")
    A.afqmc_trial_build(ctx, nw, dev(y), got)
    torch.cuda.synchronize()
    assert rel(host(got), ref) <= 1e-12


@pytest.mark.parametrize("M,N,nw,P", [(33, 17, 24, 5), (66, 5, 40, 12)])
def test_back_propagation(M, N, nw, P):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    print("back-propagation", M, N, nw, P, flush=True)
    s = ai.small_gaussian(M=M, N=N, n_chol=9, K=3, seed=M)
    rng, h, dtau = np.random.default_rng(M), 3, 0.01
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    phiT = O.trial_det(s, ai.random_hidden(rng, s, nw, P))
    logov = O.log_overlap(phiT, phi)
    hxi = rng.normal(size=(nw, h, s.n_chol))
    hxb = 0.2 * (rng.normal(size=hxi.shape) + 1j * rng.normal(size=hxi.shape))
    w = rng.uniform(0.5, 1.5, size=nw)
    num, den, R = O.back_propagated_density(s, phi, hxi, hxb, phiT, logov, w, dtau, 10)
    ctx = A.Context(s, P, dtau, max_walkers=nw)
    z = dict(dtype=torch.complex128, device="cuda")
    rho = torch.zeros(nw, M, M, **z)
    out = torch.zeros(M * M + 1, dtype=torch.float64, device="cuda")
    A.afqmc_bp_density(ctx, nw, h, dev(phi), dev(hxi), dev(hxb), dev(phiT), dev(logov), dev(w),
                       torch.zeros(nw, P, M, N, **z), torch.zeros(nw, P, 2, M, N, **z),
                       torch.zeros(nw, P, **z), rho, out)
    torch.cuda.synchronize()
    for k in range(nw):
        assert rel(host(rho)[k], R[k]) <= TOL
    assert rel(host(out)[:-1].reshape(M, M), num) <= TOL
