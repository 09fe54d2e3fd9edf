"""The FP64 contraction at the edges of its tiles, against the FP64 oracle:
electrons around the multiples of 4 and 16 that its column tiles take (each
instantiated size), orbitals that end in either half of a 16-wide tile, a lone
or odd last path where two paths share a workgroup, vector counts that leave
the last group of four part full, and counts that split over several ranges;
real and complex (multi-slice) trials.  Tolerance 1e-10, as for every FP64
form of the contraction."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10

# (M, N, vectors, paths, walkers)
REAL = [(17, 2, 30, 1, 1), (9, 3, 3, 1, 3), (40, 7, 40, 3, 1), (57, 12, 17, 1, 5),
        (64, 14, 41, 5, 1), (81, 13, 30, 3, 1), (112, 18, 70, 3, 1), (120, 20, 30, 1, 2),
        (72, 21, 33, 2, 1), (130, 24, 16, 1, 2), (100, 27, 45, 1, 3), (66, 28, 5, 1, 1),
        (104, 29, 31, 2, 1), (144, 33, 30, 1, 2), (136, 36, 9, 1, 1), (160, 40, 28, 1, 2),
        (153, 37, 60, 1, 1), (64, 16, 12, 8, 120), (64, 15, 9, 1, 1030)]
COMPLEX = [(8, 1, 5, 1, 2), (33, 6, 40, 3, 1), (30, 11, 30, 1, 3), (100, 13, 33, 2, 1),
           (64, 20, 28, 1, 2), (58, 22, 17, 1, 1), (60, 27, 30, 1, 2), (64, 32, 40, 2, 1)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


def check(s, shape, phiT):
    from paper_2505_18519_amd import afqmc as A
    M, N, G, P, nw = shape
    print("contraction tiles", shape, s.name, flush=True)
    sys.stdout.flush()
    ctx = A.Context(s, P, 0.01, max_walkers=nw)
    phi = ai.random_walkers(np.random.default_rng(7), s, nw, spread=0.5)
    ell, theta = O.green(phiT, phi)
    vb, ep = O.sample_contraction(s, phiT, theta, ell)
    xbar, eloc = O.walker_estimates(vb, ep, ell, 0.01)
    z = dict(dtype=torch.complex128, device="cuda")
    d_vb, d_ep = torch.zeros(nw, P, G, **z), torch.zeros(nw, P, **z)
    d_el, d_xb = torch.zeros(nw, **z), torch.zeros(nw, G, **z)
    args = dev(phiT), dev(theta), dev(ell)
    A.afqmc_force_bias(ctx, nw, *args, d_xb, d_vb)
    A.afqmc_local_energy(ctx, nw, *args, d_el, d_ep, None)
    static = [torch.zeros_like(t) for t in (d_el, d_ep, d_xb)]
    A.afqmc_local_energy_static(ctx, nw, *args, *static)
    torch.cuda.synchronize()
    g_vb, g_ep, g_el, g_xb = (t.cpu().numpy() for t in (d_vb, d_ep, d_el, d_xb))
    assert np.linalg.norm(g_vb - vb) <= TOL * np.linalg.norm(vb)
    assert np.abs(g_ep - ep).max() <= TOL * max(np.abs(ep).max(), 1.0)
    assert np.abs(g_el - eloc).max() <= TOL * max(np.abs(eloc).max(), 1.0)
    assert np.linalg.norm(g_xb - xbar) <= TOL * np.linalg.norm(xbar)
    # the form without a workspace runs the same kernels on the same ranges
    for a, b in zip(static, (d_el, d_ep, d_xb)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("shape", REAL)
def test_real_trials(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    M, N, G, P, nw = shape
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N)
    y = np.random.default_rng(3).normal(size=(nw, P, s.K))
    check(s, shape, O.trial_det(s, y))


@pytest.mark.parametrize("shape", COMPLEX)
def test_complex_trials(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    M, N, G, P, nw = shape
    s = ai.imaginary_time_trial(ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N), 1, 0.02,
                                n_gen=min(G, 6))
    y = np.random.default_rng(3).normal(size=(nw, P, s.K))
    check(s, shape, O.trial_det(s, y))
