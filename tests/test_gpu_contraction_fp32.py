"""The FP32 contraction at the edges of its tiles, against the FP64 oracle:
electrons around the multiples of 8 that a path's or a vector's columns take
(each instantiated count), orbitals that end inside a 16-wide tile, paths that
leave the last pair or workgroup part empty, an odd and an even number of vectors
(the one-body matrix shares the last group of two or has it alone), and counts
that split over several ranges.  Tolerance 1e-4, as for every FP32 form of the
contraction; one path has a zero overlap and contributes nothing."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-4

# (M, N, vectors, paths, walkers)
SHAPES = [(8, 1, 4, 1, 1), (16, 8, 5, 3, 3), (33, 7, 40, 1, 2), (49, 8, 64, 2, 3),
          (80, 3, 7, 5, 1), (100, 8, 33, 1, 5), (128, 5, 16, 1, 3),
          (9, 9, 6, 1, 3), (30, 16, 33, 3, 3), (40, 10, 17, 7, 1), (64, 15, 40, 1, 2),
          (70, 12, 9, 2, 1), (96, 16, 34, 1, 1), (112, 9, 5, 3, 1), (120, 14, 16, 1, 2),
          (24, 17, 18, 1, 1), (48, 24, 33, 3, 2), (57, 20, 5, 1, 3), (73, 23, 40, 1, 5),
          (96, 18, 16, 2, 1),
          (32, 25, 4, 1, 1), (46, 32, 33, 1, 3), (64, 27, 17, 3, 1), (78, 26, 34, 1, 2),
          (96, 31, 5, 1, 1), (101, 28, 8, 1, 3), (128, 32, 35, 2, 1)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("shape", SHAPES)
def test_edges(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N, G, P, nw = shape
    print("fp32 contraction", shape, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N)
    phiT = O.trial_det(s, np.random.default_rng(3).normal(size=(nw, P, s.K)))
    ctx = A.Context(s, P, 0.01, max_walkers=nw, precision=A.PREC_FP32)
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
    for a, b in zip(static, (d_el, d_ep, d_xb)):
        assert torch.equal(a, b)
    # a path without overlap: zeros, and the others unchanged
    if nw * P > 1:
        dead = ell.copy()
        dead[-1, -1] = complex(-np.inf, 0.0)
        e_vb, e_ep = torch.ones_like(d_vb), torch.ones_like(d_ep)
        args = dev(phiT), dev(theta), dev(dead)
        A.afqmc_force_bias(ctx, nw, *args, d_xb, e_vb)
        A.afqmc_local_energy(ctx, nw, *args, d_el, e_ep, None)
        torch.cuda.synchronize()
        assert not e_vb[-1, -1].abs().any() and e_ep[-1, -1] == 0
        assert torch.equal(e_vb.flatten(0, 1)[:-1], d_vb.flatten(0, 1)[:-1])
        assert torch.equal(e_ep.flatten()[:-1], d_ep.flatten()[:-1])
