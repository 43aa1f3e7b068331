"""Gathers that leave the window of the window step kernel, and its FP64 n_b = 16 instance.

The kernel loads such gathers one tile ahead, into the registers that the products read in
slot order.  The row orders below scatter a fortieth of the rows over the matrix, so that
rows with none, some and all of their entries outside the window occur in both sweep
directions, with uniform and ragged widths.
Tolerances as in test_gpu_window.py.
"""
import numpy as np
import pytest
import torch

import oracle as O
from topi import csr_to_dense, random_phase_block, topi_csr

pytestmark = pytest.mark.gpu

EPS = (2.0 ** -53, 2.0 ** -24)


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def _scattered(dims, seed):
    from paper_1803_02156_amd.ordering import lattice_row_order
    order = np.array(lattice_row_order(*dims, pencil=(4, 4)))
    rng = np.random.default_rng(seed)
    at = rng.choice(len(order), len(order) // 40, replace=False)
    order[at] = order[rng.permutation(at)]
    return order


@pytest.mark.parametrize("n_p", [5, 6])
@pytest.mark.parametrize("dims,dil,prec,n_b", [((8, 8, 8), 0.0, 0, 32), ((8, 8, 8), 0.0, 1, 64),
                                               ((8, 8, 9), 0.1, 0, 32), ((8, 8, 9), 0.1, 1, 64)])
def test_scattered_rows(P, dims, dil, prec, n_b, n_p):
    H = topi_csr(*dims, m=1.0, W=1.5, seed=11, dilution=dil, dilution_seed=2)
    n = len(H[0]) - 1
    M = P.chebfd_matrix_build(*H, C=32, sigma=1, prec=prec, order=_scattered(dims, 4))
    assert P.chebfd_step_kernel(M, n_b) == P.KERNEL_WINDOW
    X = random_phase_block(n, n_b, 17)
    lo, hi = P.chebfd_bounds(M)
    al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, n_p)
    xb = P.chebfd_pack(M, torch.from_numpy(np.ascontiguousarray(X.T)).cuda().T, n_b)
    eta, nu = P.chebfd_filter(M, al, be, gam, n_b, n_b, xb)
    Yr, etar, nur = O.chebyshev_filter(H, al, be, gam, X, n_b)
    s = np.max(np.abs(np.linalg.eigvalsh(csr_to_dense(*H)))) * al
    u = EPS[prec]
    tol_T = n_p * (int(np.max(np.diff(H[0]))) + 4) * u / np.sqrt(1.0 - s * s)
    tol_Y = max(np.sum(np.abs(gam)), 1.0) * tol_T
    assert np.max(np.abs(P.chebfd_unpack(M, xb).cpu().numpy() - Yr)) <= tol_Y
    tol_m = 2.0 * n * tol_T + n * 4 * u
    assert np.max(np.abs(eta.cpu().numpy()[1:] - etar[1:])) <= tol_m
    assert np.max(np.abs(nu.cpu().numpy()[1:] - nur[1:].real)) <= tol_m


@pytest.mark.parametrize("prec,n_b", [(0, 32), (1, 64)])
def test_infinite_entry_outside_the_window(P, prec, n_b):
    """An infinite entry gives what the LDS-staged kernel gives: infinities and NaN only
    where the sum has them."""
    dims = (8, 8, 8)
    rowptr, col, val = topi_csr(*dims, m=1.0, W=1.5, seed=11)
    n = len(rowptr) - 1
    order = _scattered(dims, 4)
    at = np.empty(n, np.int64)
    at[order] = np.arange(n)
    i = np.repeat(np.arange(n), np.diff(rowptr))
    k = int(np.flatnonzero(np.abs(at[i] - at[col]) > 512)[0])
    back = int(rowptr[col[k]] + np.flatnonzero(col[rowptr[col[k]]:rowptr[col[k] + 1]] == i[k])[0])
    val = val.copy()
    val[[k, back]] = np.inf
    M = P.chebfd_matrix_build(rowptr, col, val, C=32, sigma=1, prec=prec, order=order)
    assert P.chebfd_step_kernel(M, n_b) == P.KERNEL_WINDOW
    assert P.chebfd_step_kernel(M, n_b // 4) == P.KERNEL_LDS
    X = torch.from_numpy(np.ascontiguousarray(random_phase_block(n, n_b, 3).T)).cuda().T
    out = []
    for nb in (n_b, n_b // 4):
        y = [P.chebfd_unpack(M, P.chebfd_spmmv(M, 1.0, 0.0, P.chebfd_pack(M, X[:, c:c + nb], nb)))
             for c in range(0, n_b, nb)]
        out.append(torch.view_as_real(torch.cat(list(y), dim=1).contiguous()).cpu())
    assert not torch.isfinite(out[0]).all()
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(out[0]), f(out[1]))


@pytest.mark.parametrize("dims", [(64, 64, 32), (5, 5, 5405)])
def test_fp64_16_columns(P, dims):
    """n_b = 16 takes the window kernel from 32 tiles of 64 rows per CU; the same columns
    through n_b = 32 (tiles of 32 rows, or the LDS-staged kernel) agree to rounding."""
    from paper_1803_02156_amd.ordering import lattice_row_order
    H = topi_csr(*dims, m=1.0, W=1.0, seed=3)
    n = len(H[0]) - 1
    M = P.chebfd_matrix_build(*H, prec=0, order=lattice_row_order(*dims))
    assert P.chebfd_step_kernel(M, 16) == P.KERNEL_WINDOW
    lo, hi = P.chebfd_bounds(M)
    n_p = 8
    al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, n_p)
    X = torch.from_numpy(np.ascontiguousarray(random_phase_block(n, 32, 5).T)).cuda().T
    out = []
    for nb in (16, 32):
        xb = P.chebfd_pack(M, X, nb)
        eta, nu = P.chebfd_filter(M, al, be, gam, 32, nb, xb)
        out.append((P.chebfd_unpack(M, xb), eta, nu))
    # both sides within the bound of the oracle comparison; |alpha H + beta| <= 0.995
    tol_T = 2 * n_p * (13 + 4) * EPS[0] / np.sqrt(1.0 - 0.995 ** 2)
    tol_Y = max(np.sum(np.abs(gam)), 1.0) * tol_T
    assert float((out[0][0] - out[1][0]).abs().max()) <= tol_Y
    tol_m = 2.0 * n * tol_T + n * 4 * EPS[0]
    assert float((out[0][1][1:] - out[1][1][1:]).abs().max()) <= tol_m
    assert float((out[0][2][1:] - out[1][2][1:]).abs().max()) <= tol_m
