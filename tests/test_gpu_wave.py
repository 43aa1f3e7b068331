"""The small-matrix step kernel: a launch steps several blocks of the search space.
Filtered blocks and moments of n_s = k n_b vectors equal, bit for bit, those of k
calls with one block each (the batch has the same launch shape per block), and one
block agrees with the CPU oracle.  Tolerance: the bound of a Chebyshev recurrence in
arithmetic of unit roundoff u, p (nnzr + 4) u / sqrt(1 - s^2) per filter term."""
import numpy as np
import pytest
import torch

import oracle as O
from topi import csr_to_dense, random_phase_block, topi_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


# a partial batch at the end (11 = 8 + 3 blocks), batches of 1 .. 8, every lane
# layout (1, 2, 4 .. 64 lanes per row, two wavefronts per row), ragged rows, chunks
# of one row and of 32, several passes per workgroup (23 x 17 x 19 at n_b = 64)
CASES = [((5, 4, 3), 0, 32, 11, 0.0, 32, 256), ((5, 4, 3), 1, 2, 3, 0.2, 32, 256), ((5, 3, 3), 0, 1, 9, 0.2, 1, 1),
         ((5, 4, 3), 0, 128, 2, 0.2, 8, 8), ((7, 5, 3), 1, 128, 3, 0.0, 32, 256), ((13, 11, 9), 0, 16, 5, 0.1, 32, 256),
         ((13, 11, 9), 1, 8, 7, 0.0, 32, 256), ((23, 17, 19), 0, 64, 2, 0.1, 32, 256), ((23, 17, 19), 1, 1, 2, 0.1, 32, 256)]


@pytest.mark.parametrize("dims,prec,n_b,blocks,dilution,C,sigma", CASES)
@pytest.mark.parametrize("n_p", [1, 7])
def test_batched_blocks_equal_single_blocks(P, dims, prec, n_b, blocks, dilution, C, sigma, n_p):
    H = topi_csr(*dims, m=1.0, W=1.5, seed=5, dilution=dilution, dilution_seed=3)
    n, n_s = len(H[0]) - 1, n_b * blocks
    M = P.chebfd_matrix_build(*H, C=C, sigma=sigma, prec=prec)
    lo, hi = P.chebfd_bounds(M)
    al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, n_p)
    X = random_phase_block(n, n_s, 9)
    x = torch.from_numpy(np.ascontiguousarray(X.T)).cuda().T
    xb = P.chebfd_pack(M, x, n_b)
    single = xb.clone()
    eta, nu = P.chebfd_filter(M, al, be, gam, n_s, n_b, xb)
    for b in range(blocks):
        one = single[b].clone()
        e1, n1 = P.chebfd_filter(M, al, be, gam, n_b, n_b, one)
        single[b] = one
        assert torch.equal(e1[1:], eta[1:, b * n_b:(b + 1) * n_b]) and torch.equal(n1[1:], nu[1:, b * n_b:(b + 1) * n_b])
    assert torch.equal(xb, single)
    if n > 600:
        return
    u = 2.0 ** -53 if prec == 0 else 2.0 ** -24
    s = np.max(np.abs(np.linalg.eigvalsh(csr_to_dense(*H)) * al + be))
    tol = n_p * (int(np.max(np.diff(H[0]))) + 4) * u / np.sqrt(1.0 - s * s)
    Yr, er, nr = O.chebyshev_filter(H, al, be, gam, X, n_b)
    assert np.max(np.abs(P.chebfd_unpack(M, xb).cpu().numpy() - Yr)) <= max(np.sum(np.abs(gam)), 1.0) * tol
    tol_m = 2.0 * n * tol + n * 4 * u
    assert np.max(np.abs(eta.cpu().numpy()[1:] - er[1:])) <= tol_m
    assert np.max(np.abs(nu.cpu().numpy()[1:] - nr[1:].real)) <= tol_m
