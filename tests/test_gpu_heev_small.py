"""The one-launch eigensolver for matrices that fit in LDS, at its edges (odd sizes get
a dummy row, 64 is the last size, 65 the first of the launch-per-round path), for a
graded and a nearly diagonal matrix: eigenvalues to 50 m u ||A||, residuals and
orthonormality of the vectors to 100 m u (||A||)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


@pytest.mark.parametrize("kind", ["random", "graded", "near_diagonal", "zero", "pairs", "tiny"])
@pytest.mark.parametrize("m", [1, 2, 3, 8, 31, 32, 36, 63, 64, 65])
def test_heev_small_edges(P, m, kind):
    rng = np.random.default_rng(m)
    A = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    A = A + A.conj().T
    if kind == "graded":
        d = 10.0 ** -np.linspace(0, 6, m)
        A = d[:, None] * A * d[None, :]
    elif kind == "near_diagonal":
        A = np.diag(rng.standard_normal(m)) + 1e-9 * A
    elif kind == "pairs":       # exactly degenerate pairs: off-diagonals shrink to any size with equal diagonals
        h = (m + 1) // 2
        A = np.kron(np.eye(2), A[:h, :h])[:m, :m]
    elif kind == "tiny":        # the launch-per-round path does not scale (squares underflow)
        if m > 64:
            pytest.skip("entries below 1e-150 underflow in the launch-per-round path")
        A = A * 1e-200
    elif kind == "zero":
        A = np.zeros((m, m), dtype=complex)
    w, V, sweeps = P.chebfd_heev(torch.from_numpy(A).cuda())
    w, V = w.cpu().numpy(), V.cpu().numpy()
    nrm = np.linalg.norm(A, 2) if m > 1 else abs(A[0, 0])
    assert np.all(np.diff(w) >= 0)
    assert np.max(np.abs(w - np.linalg.eigvalsh(A))) <= 50 * m * U * nrm
    assert np.linalg.norm(A @ V - V * w, 2) <= 100 * m * U * nrm
    assert np.linalg.norm(V.conj().T @ V - np.eye(m), 2) <= 100 * m * U
    assert sweeps <= 15
