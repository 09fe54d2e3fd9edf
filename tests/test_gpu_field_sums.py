"""The sums over the auxiliary fields (V of the walkers, U of the trial paths) at
the edges of their tiles, through the propagation and the trial build, against the
FP64 oracle: vector counts below, on and past the 16 of a staged chunk, walkers and
matrix entries that leave the last tile part full, and populations on either side
of the narrow and the wide tile.  Tolerance 1e-10, as for every FP64 propagation."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10

# (M, N, vectors, generators, walkers)
SHAPES = [(3, 1, 2, 2, 1), (8, 2, 15, 15, 33), (9, 3, 16, 16, 32), (13, 2, 17, 33, 65),
          (40, 3, 31, 5, 64), (65, 2, 48, 17, 31), (80, 2, 33, 16, 330), (96, 2, 17, 32, 256)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("shape", SHAPES)
def test_edges(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N, G, K, nw = shape
    print("field sums", shape, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=K, seed=M + N)
    rng = np.random.default_rng(3)
    P, dtau = 1, 0.01
    ctx = A.Context(s, P, dtau, max_walkers=nw)
    y = rng.normal(size=(nw, P, K))
    d_phiT = torch.zeros(nw, P, M, N, dtype=torch.float64, device="cuda")
    A.afqmc_trial_build(ctx, nw, dev(y), d_phiT)
    phiT = O.trial_det(s, y)
    torch.cuda.synchronize()
    assert np.linalg.norm(d_phiT.cpu().numpy() - phiT) <= TOL * np.linalg.norm(phiT)
    phi = ai.random_walkers(rng, s, nw, spread=0.5)
    ell = O.log_overlap(phiT, phi)
    xi = rng.normal(size=(nw, G))
    xbar = 0.3 * (rng.normal(size=(nw, G)) + 1j * rng.normal(size=(nw, G)))
    w = rng.uniform(0.5, 1.5, size=nw)
    want = O.propagate(s, phi, xi, xbar, phiT, ell, w, dtau, 10, -1.3)[0]
    d_phi, d_w = dev(phi), dev(w)
    z = dict(dtype=torch.complex128, device="cuda")
    A.afqmc_propagate(ctx, nw, d_phi, dev(xi), dev(xbar), dev(phiT), dev(ell), -1.3, d_w,
                      torch.zeros(nw, **z), torch.zeros(nw, P, **z))
    torch.cuda.synchronize()
    assert np.linalg.norm(d_phi.cpu().numpy() - want) <= TOL * np.linalg.norm(want)
