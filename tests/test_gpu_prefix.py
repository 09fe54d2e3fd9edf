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


# (M, N, walkers, of the small call): the two calls of a pair run different kernels (at 81 and
# 128 orbitals the same one); 3 to 10 row tiles, one to three column tiles, one to several
# workgroups a V
MOVES = [(40, 18, 140, 7), (50, 20, 140, 5), (66, 3, 300, 5), (72, 18, 140, 7), (81, 21, 45, 1),
         (96, 24, 140, 3), (100, 25, 140, 4), (112, 28, 140, 3), (128, 8, 140, 30),
         (137, 19, 140, 30), (142, 35, 100, 40), (160, 40, 100, 3)]


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


@pytest.mark.parametrize("shape", [(33, 17, 24, 2, 5), (66, 5, 40, 3, 12), (125, 4, 140, 3, 4)])
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


# (M, N, vectors, hidden, paths, walkers, of the small call, precision, Ising)
STEPS = [(72, 18, 40, 9, 2, 150, 3, 0, False), (64, 16, 64, 8, 4, 300, 5, 0, False),
         (24, 6, 96, 8, 4, 300, 2, 0, False), (8, 2, 16, 4, 8, 200, 9, 0, True),
         (70, 22, 50, 6, 2, 150, 3, 1, False), (24, 10, 40, 6, 4, 200, 3, 1, False),
         (70, 22, 50, 6, 2, 150, 3, 2, False), (40, 9, 40, 6, 4, 150, 3, 3, False)]


@pytest.mark.parametrize("shape", STEPS)
def test_steps(shape):
    M, N, G, K, P, many, few, prec, ising = shape
    say("steps", shape)
    s = ai.workload(0)[0] if ising else ai.small_gaussian(M=M, N=N, n_chol=G, K=K, seed=M + N)
    A, ctx = context(s, P, many, precision=prec)
    from paper_2505_18519_amd import driver as D
    out = []
    for n in (many, few):
        w, est = D.init_walkers(ctx, s.phi0, n, 3), torch.zeros(2, device="cuda", dtype=torch.float64)
        for i in range(3):
            D.step(ctx, w, 3, i, est, n_qr=2)
        torch.cuda.synchronize()
        out.append((w.phi, w.w, w.y, w.phiT, w.logov, w.eloc, w.xbar))
    same(*out, few)


# (M, N, vectors, paths, walkers, of the small call, precision): FP64 on either kernel, FP32,
# BF16 and split BF16, with calls that split the vectors over several workgroups differently;
# 1100 paths of N = 30 split where the workspace has room, not in the fixed scratch
CONTRACTIONS = [(64, 16, 100, 4, 600, 3, 0), (60, 13, 70, 4, 300, 1, 0), (24, 6, 97, 4, 300, 5, 0),
                (45, 11, 180, 4, 333, 30, 0), (72, 18, 66, 3, 300, 11, 0),
                (96, 24, 130, 4, 130, 3, 0), (142, 35, 75, 3, 90, 2, 0), (40, 30, 192, 1, 1100, 3, 0),
                (33, 7, 100, 4, 300, 2, 1), (64, 15, 63, 4, 300, 9, 1), (96, 24, 70, 4, 300, 2, 1),
                (128, 32, 67, 4, 130, 3, 1),
                (40, 6, 65, 4, 520, 3, 2), (96, 20, 50, 2, 600, 9, 2), (128, 32, 100, 4, 150, 3, 2),
                (40, 12, 65, 4, 520, 3, 3), (64, 30, 51, 2, 600, 9, 3)]


@pytest.mark.parametrize("shape", CONTRACTIONS)
def test_contraction(shape):
    M, N, G, P, many, few, prec = shape
    say("contraction", shape)
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N)
    A, ctx = context(s, P, many, precision=prec)
    gen = torch.Generator(device="cuda").manual_seed(5)
    phiT, theta = normal(gen, many, P, M, N), normal(gen, many, P, 2, M, N, cplx=True) / M
    out = []
    for n in (many, few):
        check_contraction(A, ctx, n, G, P, phiT, theta, out)
    same(*out, few)


@pytest.mark.parametrize("shape", [(20, 5, 60, 4, 200, 2), (58, 22, 90, 2, 300, 3)])
def test_complex_contraction(shape):
    M, N, G, P, many, few = shape
    say("complex contraction", shape)
    s = ai.imaginary_time_trial(ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N), 1, 0.02,
                                n_gen=4)
    A, ctx = context(s, P, many)
    gen = torch.Generator(device="cuda").manual_seed(6)
    phiT = normal(gen, many, P, M, N, cplx=True)
    theta = normal(gen, many, P, 2, M, N, cplx=True) / M
    out = []
    for n in (many, few):
        check_contraction(A, ctx, n, G, P, phiT, theta, out)
    same(*out, few)


def check_contraction(A, ctx, n, G, P, phiT, theta, out):
    args = phiT[:n].contiguous(), theta[:n].contiguous(), zeros(n, P)
    el, ep, xb = zeros(n), zeros(n, P), zeros(n, G)
    A.afqmc_local_energy(ctx, n, *args, el, ep, xb)
    st = zeros(n), zeros(n, P), zeros(n, G)
    A.afqmc_local_energy_static(ctx, n, *args, *st)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(st, (el, ep, xb)))
    out.append((el, ep, xb))
