"""The contraction kernel that bench.py names, for every form of the contraction:
small systems on either side of each limit of the one-wavefront kernel, larger
ones, complex trials, and the reduced precisions."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


@pytest.mark.parametrize("M,N,prec,cplx,name", [
    (64, 16, 0, False, "k_contract"), (64, 13, 0, False, "k_contract"),
    (57, 16, 0, False, "k_contract"), (56, 16, 0, False, "k_contract_q"),
    (64, 12, 0, False, "k_contract_q"), (64, 17, 0, False, "k_contract_q"),
    (65, 16, 0, False, "k_contract_q"), (8, 2, 0, False, "k_contract_q"),
    (128, 32, 0, False, "k_contract_q"), (64, 16, 0, True, "k_contract_q"),
    (64, 16, 1, True, "k_contract_g"), (64, 16, 1, False, "k_contract_f32"),
    (96, 24, 1, False, "k_contract_f32"), (128, 32, 2, False, "k_contract_sh"),
    (64, 16, 3, False, "k_contract_sh")])
def test_name(M, N, prec, cplx, name):
    import bench
    assert bench.contraction_kernel(M, N, prec, cplx) == name
