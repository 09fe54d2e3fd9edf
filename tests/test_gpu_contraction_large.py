"""Reduced-precision contractions at 17 to 24 electrons and more than 96 orbitals,
where four paths a workgroup would not fit its LDS, against the FP64 oracle: both
sides of each size at which the split changes, whole and part-filled workgroups,
one and several ranges of the vectors.  Tolerances as for these forms elsewhere:
1e-4 for FP32 and split BF16, 5e-2 for BF16."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai
from oracle import afqmc_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {1: 1e-4, 2: 5e-2, 3: 1e-4}
# (M, N, vectors, paths, walkers)
SHAPES = [(96, 24, 17, 2, 2), (97, 17, 40, 3, 1), (107, 23, 9, 1, 5), (112, 20, 33, 2, 2),
          (113, 24, 16, 1, 3), (128, 17, 35, 4, 2), (128, 24, 8, 1, 1)]


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES)
def test_edges(shape, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N, G, P, nw = shape
    print("large contraction", shape, prec, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N)
    phiT = O.trial_det(s, np.random.default_rng(3).normal(size=(nw, P, s.K)))
    ctx = A.Context(s, P, 0.01, max_walkers=nw, precision=prec)
    phi = ai.random_walkers(np.random.default_rng(7), s, nw, spread=0.5)
    ell, theta = O.green(phiT, phi)
    vb, ep = O.sample_contraction(s, phiT, theta, ell)
    z = dict(dtype=torch.complex128, device="cuda")
    d_vb, d_ep = torch.zeros(nw, P, G, **z), torch.zeros(nw, P, **z)
    d_el, d_xb = torch.zeros(nw, **z), torch.zeros(nw, G, **z)
    args = dev(phiT), dev(theta), dev(ell)
    A.afqmc_force_bias(ctx, nw, *args, d_xb, d_vb)
    A.afqmc_local_energy(ctx, nw, *args, d_el, d_ep, None)
    static = [torch.zeros_like(t) for t in (d_el, d_ep, d_xb)]
    A.afqmc_local_energy_static(ctx, nw, *args, *static)
    torch.cuda.synchronize()
    assert np.linalg.norm(d_vb.cpu().numpy() - vb) <= TOL[prec] * np.linalg.norm(vb)
    assert np.abs(d_ep.cpu().numpy() - ep).max() <= TOL[prec] * max(np.abs(ep).max(), 1.0)
    for a, b in zip(static, (d_el, d_ep, d_xb)):
        assert torch.equal(a, b)
