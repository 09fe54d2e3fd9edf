"""A walker's results do not depend on how many others share the call: the first
walkers of a large call against a call of those alone, bit for bit, at sizes where
the two run different kernels or split their work differently."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(*a):
    print("prefix", *a, flush=True)
    sys.stdout.flush()


def context(s, P, nw, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    return A, A.Context(s, P, 0.01, max_walkers=nw, **kw)


def normal(gen, *shape, cplx=False):
    return torch.randn(*shape, generator=gen, device="cuda",
                       dtype=torch.complex128 if cplx else torch.float64)


def walkers(s, gen, nw):
    base = torch.as_tensor(s.phi0, device="cuda").to(torch.complex128)
    return (base + 0.3 / np.sqrt(s.M) * normal(gen, nw, 2, s.M, s.N, cplx=True)).contiguous()


def zeros(*shape):
    return torch.zeros(*shape, dtype=torch.complex128, device="cuda")


def same(big, small, n):
    for a, b in zip(big, small):
        assert torch.isfinite(torch.view_as_real(a) if a.is_complex() else a).all()
        assert torch.equal(a[:n], b[:n])


# (M, N, walkers, of the small call): row tiles that end on, before and past a multiple of
# 16, one to three column tiles, one to several workgroups a V
MOVES = [(66, 3, 300, 5), (72, 18, 60, 7), (81, 21, 45, 1), (96, 24, 50, 3), (128, 8, 140, 30),
         (142, 35, 40, 2), (160, 40, 30, 3)]


@pytest.mark.parametrize("shape", MOVES)
def test_move(shape):
    M, N, many, few = shape
    say("move", shape)
    s = ai.small_gaussian(M=M, N=N, n_chol=9, K=3, seed=M)
    A, ctx = context(s, 2, many)
    gen = torch.Generator(device="cuda").manual_seed(M)
    phi = walkers(s, gen, many)
    phiT = torch.as_tensor(s.phi0, device="cuda").expand(many, 2, M, N).contiguous()
    xi, xbar = normal(gen, many, 9), 0.2 * normal(gen, many, 9, cplx=True)
    out = []
    for n in (many, few):
        ph, w, ref, ln = phi[:n].clone(), torch.ones(n, device="cuda", dtype=torch.float64), zeros(n), zeros(n, 2)
        A.afqmc_propagate(ctx, n, ph, xi[:n].contiguous(), xbar[:n].contiguous(), phiT[:n],
                          zeros(n, 2), 0.0, w, ref, ln)
        torch.cuda.synchronize()
        out.append((ph, ln, ref, w))
    same(*out, few)


# (M, N, walkers, of the small call, paths, slices)
SLICES = [(20, 5, 65, 1, 4, 2), (37, 11, 64, 3, 2, 1), (64, 18, 60, 5, 2, 1)]


@pytest.mark.parametrize("shape", SLICES)
def test_trial_slices(shape):
    M, N, many, few, P, m = shape
    say("slices", shape)
    s = ai.imaginary_time_trial(ai.small_gaussian(M=M, N=N, n_chol=6, K=3, seed=M), m, 0.05)
    A, ctx = context(s, P, many)
    y = normal(torch.Generator(device="cuda").manual_seed(M), many, P, s.K)
    out = []
    for n in (many, few):
        T = zeros(n, P, M, N)
        A.afqmc_trial_build(ctx, n, y[:n].contiguous(), T)
        torch.cuda.synchronize()
        out.append((T,))
    same(*out, few)


@pytest.mark.parametrize("shape", [(33, 17, 24, 2, 5), (66, 5, 40, 3, 12)])
def test_back_propagation(shape):
    M, N, many, few, P = shape
    say("back-propagation", shape)
    s = ai.small_gaussian(M=M, N=N, n_chol=9, K=3, seed=M)
    A, ctx = context(s, P, many)
    gen, h = torch.Generator(device="cuda").manual_seed(M), 3
    phi = walkers(s, gen, many)
    phiT = (torch.as_tensor(s.phi0, device="cuda") + 0.1 * normal(gen, many, P, M, N)).contiguous()
    xi, xbar = normal(gen, many, h, 9), 0.2 * normal(gen, many, h, 9, cplx=True)
    out = []
    for n in (many, few):
        bra, th, lb, rho = zeros(n, P, M, N), zeros(n, P, 2, M, N), zeros(n, P), zeros(n, M, M)
        A.afqmc_bp_density(ctx, n, h, phi[:n].contiguous(), xi[:n].contiguous(),
                           xbar[:n].contiguous(), phiT[:n].contiguous(), zeros(n, P),
                           torch.ones(n, device="cuda", dtype=torch.float64), bra, th, lb, rho,
                           torch.zeros(M * M + 1, device="cuda", dtype=torch.float64))
        torch.cuda.synchronize()
        out.append((bra, th, lb, rho))
    same(*out, few)
