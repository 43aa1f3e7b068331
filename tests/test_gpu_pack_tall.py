"""Layout conversion of more rows than a grid has room for (2^30 rows: one workgroup of
256 threads per 64 rows would be 2^32 work-items).  The handle holds sizes only: the
conversion reads nothing else of a matrix in natural order.  Exact (entries that c64
holds); about 130 GB of device memory."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N, NB = (1 << 30) + 77, 4


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def test_pack_and_unpack_of_a_billion_rows(P):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GiB of free device memory")
    some = torch.zeros(64, dtype=torch.uint8, device="cuda")
    h = P._abi.ChebfdMatrix()
    h.n, h.C, h.sigma, h.prec, h.identity_perm = N, 32, 256, P.PREC_MIXED, 1
    for f in ("chunk_off", "chunk_width", "col", "val", "perm", "iperm"):
        setattr(h, f, some.data_ptr())
    M = P.Matrix(h, some)
    x = torch.empty((NB, N), dtype=torch.complex128, device="cuda").T
    for c in range(NB):     # entry (i, c) = i + c 2^20 modulo 2^24, exact in c64; imaginary part c + 1
        re = torch.view_as_real(x[:, c])
        re[:, 0].copy_(torch.arange(c << 20, N + (c << 20), device="cuda").bitwise_and_((1 << 24) - 1))
        re[:, 1] = c + 1
    xb = P.chebfd_pack(M, x, NB)
    for c in range(NB):
        assert torch.equal(torch.view_as_real(xb[0, :, c]).double(), torch.view_as_real(x[:, c]))
    x.zero_()
    P.chebfd_unpack(M, xb, out=x)
    for c in range(NB):
        assert torch.equal(torch.view_as_real(xb[0, :, c]).double(), torch.view_as_real(x[:, c]))
    assert x[N - 1, NB - 1].real == (N - 1 + ((NB - 1) << 20)) & ((1 << 24) - 1)
    del x, xb
    torch.cuda.empty_cache()
