"""Workspace sizes of the filter on small matrices, where one launch can step several
blocks of the search space: chebfd_filter_query is what one block needs (the size that
decides whether chebfd_filter_noalloc takes a call), chebfd_filter_query_blocks adds the
room for the blocks that there are, and the results are the same bits with either."""
import ctypes

import pytest
import torch

from topi import topi_csr

pytestmark = pytest.mark.gpu

SCRATCH_BYTES = 4 << 20


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def test_work_buffers_without_whole_blocks(P):
    """The buffers of single steps: n_s need not be a multiple of n_b."""
    M = P.chebfd_matrix_build(*topi_csr(5, 4, 3, m=1.0, W=1.5, seed=5))
    for n_s in (0, 1, 31):
        w = P.FilterWork(M, 32, 4, n_s)
        assert w.nbytes == P.chebfd_filter_query(M, 32) and w.u.shape == (M.n, 32) and w.eta.shape == (5, n_s)
    assert P.FilterWork(M, 32, 4, 33 + 32).nbytes == P.chebfd_filter_query_blocks(M, 64, 32)
    for n_b in (0, 3):
        with pytest.raises(P.ChebfdError):
            P.FilterWork(M, n_b, 4, 12)


@pytest.mark.parametrize("dims,prec,n_b,blocks", [((16, 16, 8), 0, 32, 2), ((5, 4, 3), 0, 32, 11), ((7, 5, 3), 1, 8, 3)])
def test_one_block_and_batched_workspaces(P, dims, prec, n_b, blocks):
    M = P.chebfd_matrix_build(*topi_csr(*dims, m=1.0, W=1.5, seed=5), prec=prec)
    n_s, block = n_b * blocks, M.n * n_b * (16 if prec == 0 else 8)
    one = P.chebfd_filter_query(M, n_b)
    # sums of at most 1024 workgroups twice, and their progress words
    assert one <= 2 * 24 * n_b * 1024 + 8 * 1024 + 1024
    assert one <= SCRATCH_BYTES          # the call that needs it is taken below
    sizes = [P.chebfd_filter_query_blocks(M, n_b * k, n_b) for k in range(1, 13)]
    assert sizes[0] == one
    assert all(a <= b for a, b in zip(sizes, sizes[1:])) and sizes[1] >= one + 2 * block and sizes[11] == sizes[7]
    with pytest.raises(P.ChebfdError):
        P.chebfd_filter_query_blocks(M, n_b + 1 if n_b > 1 else 0, n_b)
    # calls of one block allocate nothing for the others
    assert P.FilterWork(M, n_b, 20, n_b).nbytes == one
    sz = ctypes.c_size_t()
    P.check(P.load().chebfd_filter_streamed_query(M.ref(), 20, n_b, ctypes.byref(sz)))
    assert sz.value <= 2 * (block + 256) + 24 * 21 * n_b + 512 + one

    lo, hi = P.chebfd_bounds(M)
    al, be, gam = P.chebfd_coefficients(lo, hi, -0.4, 0.3, 20)
    x = P.chebfd_random_phase(M, n_s, n_b, 7)
    work = P.FilterWork(M, n_b, 20, n_s)
    assert work.nbytes == P.chebfd_filter_query_blocks(M, n_s, n_b) > one
    y = x.clone()
    eta, nu = P.chebfd_filter(M, al, be, gam, n_s, n_b, y, work)
    for size in (one, work.nbytes - 1, P.chebfd_filter_query_blocks(M, n_s + n_b, n_b)):
        w2 = P.FilterWork(M, n_b, 20, n_s)
        w2.nbytes, w2.work = size, P.device_buffer(size)
        z = x.clone()
        e2, n2 = P.chebfd_filter(M, al, be, gam, n_s, n_b, z, w2)
        assert torch.equal(z, y) and torch.equal(e2[1:], eta[1:]) and torch.equal(n2[1:], nu[1:])
    w2 = P.FilterWork(M, n_b, 20, n_s)
    w2.nbytes = one - 1
    with pytest.raises(P.ChebfdError):
        P.chebfd_filter(M, al, be, gam, n_s, n_b, x.clone(), w2)
    z = x.clone()
    P.chebfd_filter_noalloc(M, al, be, gam, n_s, n_b, z, w2.u, w2.w, w2.eta, w2.nu)
    assert torch.equal(z, y) and torch.equal(w2.eta[1:], eta[1:])
