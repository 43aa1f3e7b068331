"""Gram products of more output tiles than the reduction's grid has room for (128
workgroups of 256 threads a tile, 64 where the second operand has at most 32 columns),
and of a size where the grid is just not looped.  One row, so S is the outer product
conj(a)^T b: within four roundings of its two-term sums.  Up to 20 GB of device memory."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


@pytest.mark.parametrize("m1,m2,n_b", [((131072 + 1) * 64 - 5, 33, 128), ((262144 + 1) * 64 - 5, 1, 1),
                                       (32768 * 64, 33, 128), (65536 * 64 + 1, 2, 2)])
def test_gram_of_many_tiles(P, m1, m2, n_b):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 30 << 30:
        pytest.skip("needs 30 GiB of free device memory")
    g = torch.Generator(device="cuda").manual_seed(m1)

    def block(m):
        v = torch.randn((-(-m // n_b), 1, n_b, 2), generator=g, dtype=torch.float64, device="cuda")
        return torch.view_as_complex(v)

    a, b = block(m1), block(m2)
    S = P.chebfd_gram(a, b, m1, m2)
    av, bv = a.reshape(-1)[:m1], b.reshape(-1)[:m2]
    for j in range(m2):
        ref = av.conj() * bv[j]
        err = (S[:, j] - ref).abs()
        assert bool((err <= 4 * 2.0 ** -53 * av.abs() * bv[j].abs()).all()), j
    del S
    torch.cuda.empty_cache()
