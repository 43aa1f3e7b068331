"""The LDS-staged step kernel, in all its modes: natural-order lattices and matrices of
up to 16 entries per row whose blocks exceed 210 MB (smaller ones take the small-matrix
kernel, which chebfd_step_kernel_small tells apart), with equal and ragged rows, in
FP64 and c64.

The filter (steps that add one, two and three terms, sweeps in both directions, with and
without moments) against the recurrence in 64 bits, and bit for bit against the chain of
single steps; the unfused filter's products and the moment calls against the same
recurrence.  Tolerances: p (nnzr + 4) u / sqrt(1 - s^2) for T_p x, times sum |gamma_p|
for Y, times 2 n for the dot products (u the unit roundoff of the vectors, s the
largest scaled eigenvalue)."""
import numpy as np
import pytest
import torch

from topi import topi_csr

pytestmark = pytest.mark.gpu

DEGREES = (2, 3, 4, 5, 6, 10)


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def _matchings(n, count, keep, seed):
    """Hermitian matrix of `count` random matchings and a diagonal: rows of 1 .. count + 1
    entries (a pair is kept with probability `keep`)."""
    rng = np.random.default_rng(seed)
    row, col, val = [np.arange(n)], [np.arange(n)], [rng.uniform(-1, 1, n) + 0j]
    for _ in range(count):
        p = rng.permutation(n)[:n // 2 * 2].reshape(-1, 2)
        p = p[rng.random(len(p)) < keep]
        v = rng.standard_normal(len(p)) + 1j * rng.standard_normal(len(p))
        row += [p[:, 0], p[:, 1]]
        col += [p[:, 1], p[:, 0]]
        val += [v, v.conj()]
    row, col, val = np.concatenate(row), np.concatenate(col), np.concatenate(val)
    at = np.argsort(row, kind="stable")
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))])
    return rowptr.astype(np.int64), col[at].astype(np.int32), val[at]


class _Rows:
    """alpha H + beta in 64 bits, rows padded to equal width."""

    def __init__(self, H, al, be):
        rowptr, col, val = H
        n, cnt = len(rowptr) - 1, np.diff(rowptr)
        r = np.repeat(np.arange(n), cnt)
        k = np.arange(len(col)) - rowptr[:-1][r]
        cols, vals = np.zeros((cnt.max(), n), dtype=np.int64), np.zeros((cnt.max(), n), dtype=np.complex128)
        cols[k, r], vals[k, r] = col, val
        self.cols, self.vals = torch.from_numpy(cols).cuda(), torch.from_numpy(vals).cuda()
        self.al, self.be = al, be

    def times(self, x):
        y = self.be * x
        for c, v in zip(self.cols, self.vals):
            y += (self.al * v)[:, None] * x[c]
        return y


# matrix, prec, n_b: every lane layout from 4 lanes per row on (two columns per lane in
# c64), chunks of 32 and of 8 rows, widths 13 (equal and ragged) and 16
CASES = [("lattice", (33, 33, 34), 0.0, 32, 0, 32), ("lattice", (33, 33, 34), 0.1, 32, 0, 32),
         ("lattice", (33, 33, 34), 0.0, 32, 1, 64), ("lattice", (33, 33, 34), 0.1, 32, 1, 64),
         ("lattice", (21, 21, 20), 0.1, 8, 0, 128), ("lattice", (26, 26, 27), 0.0, 32, 1, 128),
         ("lattice", (66, 65, 65), 0.0, 32, 0, 4), ("lattice", (52, 52, 51), 0.1, 32, 1, 16),
         ("lattice", (52, 52, 51), 0.1, 32, 0, 8),
         ("matchings", 140003, 0.7, 32, 0, 32), ("matchings", 140003, 1.0, 32, 1, 64), ("matchings", 70001, 0.7, 16, 0, 64)]


@pytest.mark.parametrize("kind,size,par,C,prec,n_b", CASES)
def test_lds_staged_kernel(P, kind, size, par, C, prec, n_b):
    H = topi_csr(*size, m=1.0, W=1.5, seed=5, dilution=par, dilution_seed=3) if kind == "lattice" \
        else _matchings(size, 15, par, 8)
    n, width = len(H[0]) - 1, int(np.max(np.diff(H[0])))
    M = P.chebfd_matrix_build(*H, C=C, sigma=256, prec=prec)
    assert P.chebfd_step_kernel(M, n_b) == P.KERNEL_LDS and not P.chebfd_step_kernel_small(M, n_b)
    lo, hi = P.chebfd_bounds(M)
    lo2, hi2 = lo - 0.08 * (hi - lo), hi + 0.03 * (hi - lo)
    al, be, _ = P.chebfd_coefficients(lo2, hi2, 0.1 * lo, 0.1 * hi, 2)
    s = max(abs(al * lo + be), abs(al * hi + be))
    u = 2.0 ** -53 if prec == 0 else 2.0 ** -24

    def tol(p):
        return p * (width + 4) * u / np.sqrt(1.0 - s * s)

    xb = P.chebfd_random_phase(M, n_b, n_b, 17)
    x = P.chebfd_unpack(M, xb)
    rows = _Rows(H, al, be)
    gam = {p: P.chebfd_coefficients(lo2, hi2, 0.1 * lo, 0.1 * hi, p)[2] for p in DEGREES}
    Y = {p: gam[p][0] * x for p in DEGREES}
    eta, nu = {}, {}
    prev, cur = x.contiguous(), rows.times(x.contiguous())
    for p in range(1, max(DEGREES) + 1):
        if p > 1:
            prev, cur = cur, 2.0 * rows.times(cur) - prev
        eta[p], nu[p] = (cur.conj() * prev).sum(0), (prev.real ** 2 + prev.imag ** 2).sum(0)
        for q in DEGREES:
            if p <= q:
                Y[q] += gam[q][p] * cur
    del prev, cur, rows
    for n_p in DEGREES:
        got = xb.clone()
        e, v = P.chebfd_filter(M, al, be, gam[n_p], n_b, n_b, got)
        tol_Y, tol_m = max(np.sum(np.abs(gam[n_p])), 1.0) * tol(n_p), 2.0 * n * tol(n_p) + n * 4 * u
        assert (P.chebfd_unpack(M, got) - Y[n_p]).abs().max().item() <= tol_Y
        for p in range(1, n_p + 1):
            assert (e[p] - eta[p]).abs().max().item() <= tol_m and (v[p] - nu[p]).abs().max().item() <= tol_m
        quiet = xb.clone()
        P.chebfd_filter(M, al, be, gam[n_p], n_b, n_b, quiet, moments=False)
        assert torch.equal(quiet, got)
        # the chain of single steps: the same fused multiply-adds in the same order
        chain = xb.clone()
        w2 = P.FilterWork(M, n_b, 2, n_b)
        P.chebfd_filter(M, al, be, gam[n_p][:3].copy(), n_b, n_b, chain, work=w2)   # w2.u = T_1 x, w2.w = T_2 x
        a, b = w2.w, w2.u
        for p in range(3, n_p + 1):
            P.chebfd_op(M, al, be, gam[n_p][p], n_b, a, b, chain, w2.work, w2.nbytes)
            a, b = b, a
        assert torch.equal(chain, got)
    got = xb.clone()
    e, v = P.chebfd_filter_unfused(M, al, be, gam[6], n_b, n_b, got)
    assert (P.chebfd_unpack(M, got) - Y[6]).abs().max().item() <= max(np.sum(np.abs(gam[6])), 1.0) * tol(6)
    assert (e[6] - eta[6]).abs().max().item() <= 2.0 * n * tol(6) + n * 4 * u
    if n_b <= 32:
        # the same columns in the moment call (blocks of min(R, 32)): no filtered block
        mu = P.chebfd_kpm_moments(M, al, be, 10, n_b, 17)
        ref = np.array([nu[1].sum().item(), eta[1].sum().real.item()])
        for k in range(1, 10):
            ref = np.append(ref, [2 * nu[k + 1].sum().item() - ref[0], 2 * eta[k + 1].sum().real.item() - ref[1]])
        assert np.max(np.abs(mu - ref / (n * n_b))) <= 2 * (2.0 * tol(10) + 4 * u) + (2.0 * tol(1) + 4 * u)
