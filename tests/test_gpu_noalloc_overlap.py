"""chebfd_filter_noalloc on two streams at once: the static array that all calls of a
device share holds sums and progress words only, never blocks of the search space, so
filters without moments do not disturb each other, also where a matrix is small enough
for chebfd_filter to step several blocks per launch (240 rows, four and three blocks:
their U and W would fit the array).  Exact: the same kernels in the same order."""
import numpy as np
import pytest
import torch

from topi import topi_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


@pytest.mark.parametrize("prec,n_b", [(0, 32), (1, 16)])
def test_overlapping_filters_without_moments(P, prec, n_b):
    calls = []
    for seed, blocks in ((5, 4), (6, 3)):
        H = topi_csr(5, 4, 3, m=1.0, W=1.5, seed=seed)
        M = P.chebfd_matrix_build(*H, prec=prec)
        lo, hi = P.chebfd_bounds(M)
        al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, 60)
        x = P.chebfd_random_phase(M, blocks * n_b, n_b, seed)
        ref = x.clone()
        P.chebfd_filter(M, al, be, gam, blocks * n_b, n_b, ref, moments=False)
        u = torch.empty((M.n, n_b), dtype=x.dtype, device="cuda")
        calls.append((M, al, be, gam, blocks * n_b, x, ref, u, torch.empty_like(u), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(10):
        out = [c[5].clone() for c in calls]
        torch.cuda.synchronize()
        for (M, al, be, gam, n_s, _, _, u, w, s), y in zip(calls, out):
            with torch.cuda.stream(s):
                P.chebfd_filter_noalloc(M, al, be, gam, n_s, n_b, y, u, w, None, None)
        torch.cuda.synchronize()
        for c, y in zip(calls, out):
            assert torch.equal(y, c[6])
    assert np.isfinite(calls[0][6].abs().sum().item())
