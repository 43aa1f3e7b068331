"""Gram and update products at the edges of their tiles: the Hermitian product's
diagonal tiles (at most 32 columns: rows quartered among the waves; 33 .. 64; several
tiles with a last one of few columns), narrow products, few rows.  Tolerances: 4 n u
relative to |A|^T |B| (Gram) and 4 u_z + 8 m u relative to |A| |M| (update)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS64 = 2.0 ** -53
EPS32 = 2.0 ** -24


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def _block(rng, n, m, n_b, dtype):
    blocks = -(-m // n_b)
    x = rng.standard_normal((blocks, n, n_b)) + 1j * rng.standard_normal((blocks, n, n_b))
    t = torch.from_numpy(x).to("cuda", dtype)
    a = t.cpu().numpy().astype(np.complex128).transpose(1, 0, 2).reshape(n, blocks * n_b)[:, :m]
    return t, a


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,n_b,m", [(1, 1, 1), (15, 4, 16), (300, 16, 17), (2000, 32, 32), (130, 32, 33), (777, 64, 64),
                                     (1000, 8, 65), (70000, 32, 100), (400, 32, 200), (5000, 32, 257)])
def test_hermitian_gram_and_update_edges(P, prec, n, n_b, m):
    rng = np.random.default_rng(n + m)
    a, A = _block(rng, n, m, n_b, P.vec_dtype(prec))
    S = P.chebfd_gram(a, a, m, m).cpu().numpy()
    scale = np.abs(A).T @ np.abs(A)
    assert np.max(np.abs(S - A.conj().T @ A) / scale) < 4 * n * EPS64
    assert np.array_equal(np.triu(S, 1), np.triu(S.conj().T, 1))
    c = min(m, 32)
    b, B = _block(rng, n, c, n_b, P.vec_dtype(prec))
    S = P.chebfd_gram(a, b, m, c).cpu().numpy()
    assert np.max(np.abs(S - A.conj().T @ B) / (np.abs(A).T @ np.abs(B))) < 4 * n * EPS64
    M = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    z = P.chebfd_update(a, torch.from_numpy(M).cuda())
    Z = z.cpu().numpy().astype(np.complex128).transpose(1, 0, 2).reshape(n, -1)[:, :m]
    u = EPS64 if prec == 0 else EPS32
    assert np.max(np.abs(Z - A @ M) / (np.abs(A) @ np.abs(M))) < 4 * u + 8 * m * EPS64
