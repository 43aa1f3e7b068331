"""Layout conversion at the edges of its tiles (64 rows, up to 32 columns): exact
copies both ways, c64 entries rounded once, rows in the matrix's order."""
import numpy as np
import pytest
import torch

from topi import diag_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("n,n_b,blocks", [(1, 4, 1), (63, 1, 3), (64, 2, 2), (65, 4, 3), (127, 8, 1), (130, 16, 2),
                                          (200, 32, 2), (1000, 64, 1), (333, 128, 2)])
def test_pack_and_unpack(P, n, n_b, blocks, permuted, prec):
    rng = np.random.default_rng(n)
    order = rng.permutation(n).astype(np.int32) if permuted else None
    M = P.chebfd_matrix_build(*diag_csr(np.arange(1.0, n + 1)), prec=prec, order=order)
    m = n_b * blocks
    X = rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))
    x = torch.from_numpy(X).cuda().T
    xb = P.chebfd_pack(M, x, n_b)
    rows = np.arange(n) if order is None else order     # equal row lengths: the sigma sort keeps the order
    ref = X[:, rows].reshape(blocks, n_b, n).transpose(0, 2, 1).astype(np.complex128 if prec == 0 else np.complex64)
    assert np.array_equal(xb.cpu().numpy(), ref)
    y = P.chebfd_unpack(M, xb).cpu().numpy()
    back = X if prec == 0 else X.astype(np.complex64).astype(np.complex128)
    assert np.array_equal(y, back.T)
