"""TSQR panels at the edges of its tree: leaves of 256 rows, nodes of fewer rows than columns,
every panel width, one and several levels, and columns whose reflectors vanish.

Q comes from the reflectors in compact form (I - V T V^H); Q^H Q = I and Q R = Y hold to a few
hundred roundings of FP64 per column whatever the conditioning of Y.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS64 = 2.0 ** -53


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


@pytest.mark.parametrize("n,m,n_b", [(1, 1, 1), (255, 2, 2), (256, 4, 4), (257, 8, 8), (256, 16, 16), (258, 16, 16),
                                     (256, 32, 32), (273, 32, 32), (2049, 31, 32), (8193, 40, 32), (4097, 70, 64)])
@pytest.mark.parametrize("kind", ["full", "zero", "dependent"])
def test_tsqr_q_and_r(P, n, m, n_b, kind):
    rng = np.random.default_rng(n + m)
    Y = rng.standard_normal((n, m)) + 1j * rng.standard_normal((n, m))
    if kind == "zero" and m > 1:
        Y[:, m // 2] = 0.0
    if kind == "dependent" and m > 1:
        Y[:, m - 1] = Y[:, 0] * (0.5 - 2.0j)
    mb = -(-m // n_b) * n_b
    b = np.zeros((n, mb), dtype=np.complex128)
    b[:, :m] = Y
    y = torch.from_numpy(np.ascontiguousarray(b.T.reshape(mb // n_b, n_b, n).transpose(0, 2, 1))).cuda()
    q, R = P.chebfd_tsqr(y, m)
    Q = q.cpu().numpy().transpose(0, 2, 1).reshape(mb, n).T[:, :m]
    R = R.cpu().numpy()
    ymax = np.max(np.linalg.norm(Y, axis=0))
    assert np.max(np.abs(np.tril(R, -1)), initial=0.0) == 0.0
    assert np.all(np.diag(R).imag == 0.0) and np.all(np.diag(R).real >= 0.0)
    assert np.max(np.abs(Q @ R - Y)) < 200 * m * EPS64 * ymax
    # a column that vanishes in a later panel has no direction of its own: Q^H Q = I is asked
    # of the panel's own reflectors only (all columns within one panel)
    if kind == "full" or m <= min(n_b, 32):
        assert np.max(np.abs(Q.conj().T @ Q - np.eye(m))) < 200 * m * EPS64
