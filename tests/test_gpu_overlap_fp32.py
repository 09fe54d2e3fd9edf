"""Theta and log-overlaps of FP32 contexts at the edges of their kernels' column
counts, against the FP64 oracle (they are FP64 quantities: tolerance 1e-10), with a
path of zero overlap and one with an infinite entry; and the two kernels that share
the small systems, by the number of paths, bit for bit."""
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


def case(M, N, P, nw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    print("fp32 overlap", M, N, P, nw, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=4, K=3, seed=M + N)
    rng = np.random.default_rng(5)
    phiT = O.trial_det(s, 0.5 * rng.normal(size=(nw, P, s.K)))
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    return A, s, phiT, phi, A.Context(s, P, 0.01, max_walkers=nw, precision=A.PREC_FP32)


def green(A, ctx, nw, P, M, N, phi, phiT):
    l = torch.zeros(nw, P, dtype=torch.complex128, device="cuda")
    th = torch.zeros(nw, P, 2, M, N, dtype=torch.complex128, device="cuda")
    A.afqmc_green(ctx, nw, dev(phi), dev(phiT), l, th)
    torch.cuda.synchronize()
    return l.cpu().numpy(), th.cpu().numpy()


@pytest.mark.parametrize("M,N,P,nw", [(1, 1, 3, 3), (8, 2, 3, 3), (17, 8, 3, 3), (30, 9, 3, 3),
                                      (20, 9, 4, 257), (64, 16, 4, 257), (63, 15, 4, 257),
                                      (65, 1, 3, 3), (66, 16, 3, 3), (20, 17, 3, 3),
                                      (24, 24, 3, 3), (128, 32, 3, 3)])
def test_edges(M, N, P, nw):
    A, s, phiT, phi, ctx = case(M, N, P, nw)
    ell, theta = O.green(phiT, phi)
    l, th = green(A, ctx, nw, P, M, N, phi, phiT)
    assert np.abs(np.exp(l - ell) - 1).max() <= TOL
    assert np.linalg.norm(th - theta) <= TOL * np.linalg.norm(theta)
    bad = phiT.copy()
    bad[0, 1, :, 0] = 0.0
    bad[nw - 1, P - 1, M // 2, N - 1] = np.inf
    l, th = green(A, ctx, nw, P, M, N, phi, bad)
    assert np.isneginf(l[0, 1].real) and l[0, 1].imag == 0
    assert np.isnan(l[-1, -1].real) and np.isnan(l[-1, -1].imag)
    assert not th[0, 1].any() and not th[-1, -1].any()
    keep = np.ones((nw, P), bool)
    keep[0, 1] = keep[-1, -1] = False
    assert np.abs(np.exp(l - ell) - 1)[keep].max() <= TOL
    assert np.linalg.norm(th[keep] - theta[keep]) <= TOL * np.linalg.norm(theta[keep])


@pytest.mark.parametrize("M,N", [(16, 9), (40, 10), (47, 12), (64, 13), (33, 15), (64, 16)])
def test_forms_agree(M, N):
    P, nw, few = 4, 257, 3
    A, s, phiT, phi, ctx = case(M, N, P, nw)
    l, th = green(A, ctx, nw, P, M, N, phi, phiT)
    lf, thf = green(A, ctx, few, P, M, N, phi[:few], phiT[:few])
    assert np.array_equal(l[:few], lf) and np.array_equal(th[:few], thf)
