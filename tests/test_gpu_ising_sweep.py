"""Single-spin-flip sweeps with diagonal generators, against the FP64 oracle: one to
64 spins in one launch and 65 on the general path, electrons on either side of 8,
orbitals up to 64, a path alone in its wavefront, and a path whose overlap vanishes.
Decisions and spins are exact, determinants and log-overlaps to 1e-12 and 1e-10 as for
the other Metropolis tests."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (M, N, K, paths, walkers)
SHAPES = [(1, 1, 1, 1, 1), (8, 2, 4, 3, 5), (17, 8, 9, 5, 1), (30, 9, 33, 2, 3), (64, 16, 64, 1, 3),
          (63, 3, 5, 64, 1), (20, 5, 65, 2, 2)]


def system(M, N, K):
    g = ai.small_gaussian(M=M, N=N, n_chol=4, K=2, seed=M + N)
    rng = np.random.default_rng(K)
    A = np.zeros((K, M, M))
    A[:, np.arange(M), np.arange(M)] = rng.uniform(0.0, 1.0, (K, M)) * (rng.random((K, M)) < 0.5)
    return ai.System(M=M, N=N, n_chol=4, K=K, hidden_kind=ai.HIDDEN_ISING, coupling=0.2, h1=g.h1,
                     L=g.L, phi0=g.phi0, A=A, name=f"ising-M{M}-K{K}")


@pytest.mark.parametrize("shape", SHAPES)
def test_sweeps(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N, K, P, nw = shape
    print("ising sweep", shape, flush=True)
    sys.stdout.flush()
    s = system(M, N, K)
    rng = np.random.default_rng(5)
    y = rng.choice([-1.0, 1.0], size=(nw, P, K))
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    phiT = O.trial_det(s, y)
    ell = O.log_overlap(phiT, phi)
    ref = np.exp(0.3j * rng.uniform(-1, 1, size=nw))
    w0 = rng.uniform(0.5, 1.5, size=nw)
    ctx = A.Context(s, P, 0.01, max_walkers=nw)
    y2, phiT2, ell2, w2, nacc = O.metropolis(s, phi, y, phiT, ell, ref, w0, 12, 7, 2)

    def dev(x):
        return torch.as_tensor(np.ascontiguousarray(x)).cuda()

    dy, dp, dl, dw = dev(y), dev(phiT), dev(ell), dev(w0)
    acc = torch.zeros(nw, dtype=torch.int32, device="cuda")
    A.afqmc_metropolis_x(ctx, nw, dev(phi), dy, dp, dl, dev(ref), dw, 12, 7, 2, acc)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), nacc)
    assert np.array_equal(dy.cpu().numpy(), y2)
    assert np.linalg.norm(dp.cpu().numpy() - phiT2) <= 1e-12 * np.linalg.norm(phiT2)
    assert np.abs(np.exp(dl.cpu().numpy() - ell2) - 1).max() <= 1e-10
    assert np.abs(dw.cpu().numpy() - w2).max() <= 1e-10 * np.abs(w2).max()
    # a walker without overlap accepts nothing and stays as it is
    dead = phi.copy()
    dead[-1] = 0.0
    le = ell.copy()
    le[-1] = complex(-np.inf, 0.0)
    dy, dp, dl = dev(y), dev(phiT), dev(le)
    A.afqmc_metropolis_x(ctx, nw, dev(dead), dy, dp, dl, None, None, 12, 7, 1, acc)
    torch.cuda.synchronize()
    assert acc.cpu().numpy()[-1] == 0
    assert np.array_equal(dy.cpu().numpy()[-1], y[-1])
    assert np.array_equal(dp.cpu().numpy()[-1], phiT[-1])
    assert np.isneginf(dl.cpu().numpy()[-1].real).all()
