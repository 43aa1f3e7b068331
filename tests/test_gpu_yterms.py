"""The filter adds the terms of three recurrence steps to Y at a time; a chain of
single fused steps (chebfd_op, one term each) performs the same fused multiply-adds
in the same order, so the two agree bit for bit, at every remainder of the degree by
three and in every step kernel."""
import numpy as np
import pytest
import torch

from topi import random_phase_block, topi_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


# window (FP64 n_b = 32), LDS-staged, row and multi-row kernels (C = 64)
CASES = [((16, 16, 8), 0, 32, 32, 0.0, True), ((5, 4, 3), 0, 8, 32, 0.2, False), ((5, 4, 3), 1, 16, 32, 0.0, False),
         ((5, 4, 3), 0, 32, 64, 0.2, False), ((5, 4, 3), 1, 4, 64, 0.0, False)]


@pytest.mark.parametrize("dims,prec,n_b,C,dilution,lattice", CASES)
@pytest.mark.parametrize("n_p", [2, 3, 4, 5, 6, 10])
def test_filter_equals_chain_of_single_steps(P, dims, prec, n_b, C, dilution, lattice, n_p):
    from paper_1803_02156_amd.ordering import lattice_row_order
    H = topi_csr(*dims, m=1.0, W=1.5, seed=5, dilution=dilution, dilution_seed=3)
    n = len(H[0]) - 1
    M = P.chebfd_matrix_build(*H, C=C, sigma=256, prec=prec, order=lattice_row_order(*dims) if lattice else None)
    lo, hi = P.chebfd_bounds(M)
    al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, n_p)
    x = torch.from_numpy(np.ascontiguousarray(random_phase_block(n, n_b, 9).T)).cuda().T
    xb = P.chebfd_pack(M, x, n_b)
    ref = xb.clone()
    P.chebfd_filter(M, al, be, gam, n_b, n_b, xb)
    w2 = P.FilterWork(M, n_b, 2, n_b)
    P.chebfd_filter(M, al, be, gam[:3].copy(), n_b, n_b, ref, work=w2)   # w2.u = T_1 x, w2.w = T_2 x
    u, w = w2.w, w2.u
    opw = P.device_buffer(P.chebfd_filter_query(M, n_b))
    for p in range(3, n_p + 1):
        P.chebfd_op(M, al, be, gam[p], n_b, u, w, ref, opw, opw.numel())
        u, w = w, u
    torch.cuda.synchronize()
    assert torch.equal(xb, ref)
