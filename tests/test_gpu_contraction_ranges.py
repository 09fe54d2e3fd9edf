"""BF16 and split-BF16 contractions of a few paths, whose vectors are split over
several workgroups, against the same paths inside a population that fills the
chip, whose vectors are not: the force bias has the same bits, and the energies
differ by the order of FP64 sums over the vectors only (2e-15 per addition of
terms of the largest partial sum's size: 1e-12).  Vector counts end inside a
block of eight, on its edge and one past it."""
import sys

import numpy as np
import pytest

import afqmc_inputs as ai

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (M, N, vectors, paths of the small call, of the full one)
SHAPES = [(20, 5, 32, 3, 2060), (40, 10, 47, 1, 1030), (48, 16, 65, 5, 1030),
          (36, 20, 56, 2, 1030), (33, 27, 100, 7, 600), (64, 32, 33, 1, 600)]


@pytest.mark.parametrize("prec", [2, 3])
@pytest.mark.parametrize("shape", SHAPES)
def test_ranges(shape, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_18519_amd import afqmc as A
    M, N, G, few, many = shape
    print("contraction ranges", shape, prec, flush=True)
    sys.stdout.flush()
    s = ai.small_gaussian(M=M, N=N, n_chol=G, K=4, seed=M + N)
    z = dict(dtype=torch.complex128, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(5)
    ctx = A.Context(s, 1, 0.01, max_walkers=many, precision=prec)
    phiT = torch.randn(many, 1, M, N, generator=gen, dtype=torch.float64, device="cuda")
    theta = torch.randn(many, 1, 2, M, N, generator=gen, **z) / M
    ell = torch.zeros(many, 1, **z)
    out = []
    for n in (many, few):
        el, ep = torch.zeros(n, **z), torch.zeros(n, 1, **z)
        xb, vb = torch.zeros(n, G, **z), torch.zeros(n, 1, G, **z)
        args = phiT[:n].contiguous(), theta[:n].contiguous(), ell[:n].contiguous()
        A.afqmc_force_bias(ctx, n, *args, xb, vb)
        A.afqmc_local_energy(ctx, n, *args, el, ep, None)
        st = torch.zeros_like(el), torch.zeros_like(ep), torch.zeros_like(xb)
        A.afqmc_local_energy_static(ctx, n, *args, *st)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(st, (el, ep, xb)))
        out.append((vb[:few].cpu().numpy(), ep[:few].cpu().numpy()))
    (vb_m, ep_m), (vb_f, ep_f) = out
    assert np.abs(ep_m).min() > 0
    assert np.array_equal(vb_m, vb_f)
    assert np.abs(ep_f - ep_m).max() <= 1e-12 * np.abs(ep_m).max()
