// Dense kernels of the orthogonalisation and Rayleigh-Ritz steps (gfx950):
//  * tall-skinny Gram  S = A^H B  over the rows of two blocked block vectors
//    (FP64 MFMA, split over row ranges, deterministic fixed-order reduction);
//  * tall-skinny update  Z = A M  with a small FP64 complex matrix M (FP64 MFMA);
//  * a cyclic Jacobi eigensolver for small Hermitian matrices (one workgroup);
//  * column norms, scaled copies and the residual reduction.
//
// Block vectors use the filter's blocked layout: element (i, c) of an n x m
// block vector with block width nb is at ((c / nb) n + i) nb + c % nb, stored
// as c128 (prec FP64) or c64 (prec MIXED).  Small matrices are FP64 complex,
// column-major with leading dimension ld.
//
// MFMA: v_mfma_f64_16x16x4_f64 computes D(16x16) += A(16x4) B(4x16); lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[l / 16 + 4 r][l % 16] in its r-th accumulator (r = 0..3; measured on gfx950).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace chebfd {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int kT = 256;

// Keeps MFMA accumulators in accumulation registers across a loop's back edge:
// left alone the compiler carries them in vector registers in some instances and
// moves all of them there and back in every stage (128 moves per 64 products, and
// two waves per SIMD instead of three: update 524288 x 256 x 256 c64 4677 -> 4321 us).
template <int NY>
__device__ inline void hold_acc(d4v (&acc)[2][NY][2]) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
            for (int q = 0; q < 2; ++q) asm volatile("" : "+a"(acc[x][y][q]));
}

__device__ inline double2 load_c(const void *base, int prec, int64_t idx) {
    if (prec == CHEBFD_PREC_FP64) return static_cast<const double2 *>(base)[idx];
    const float2 f = static_cast<const float2 *>(base)[idx];
    double2 r;
    r.x = f.x;
    r.y = f.y;
    return r;
}

__device__ inline void store_c(void *base, int prec, int64_t idx, double2 v) {
    if (prec == CHEBFD_PREC_FP64) {
        static_cast<double2 *>(base)[idx] = v;
    } else {
        float2 f;
        f.x = static_cast<float>(v.x);
        f.y = static_cast<float>(v.y);
        static_cast<float2 *>(base)[idx] = f;
    }
}

// nb is a power of two (the launchers check): shifts instead of an integer division
__device__ inline int64_t blocked_index(int64_t n, int nb, int64_t i, int c) {
    const int lg = __ffs(nb) - 1;
    return ((int64_t)(c >> lg) * n + i) * nb + (c & (nb - 1));
}

// ---------------------------------------------------------------------------
// Gram: S(a, b) = sum_i conj(A(i, a)) B(i, b), 64 x 64 complex output tile per
// workgroup (4 waves, 32 x 32 each = 2 x 2 MFMA tiles x 4 real products), rows
// [r0, r1) of one split; partial tiles go to part[split][tile] and are summed
// in a fixed order by gram_reduce_kernel.  For the Hermitian product A^H A only
// the tiles on and above the diagonal are formed, by a launch of their own (DIAG)
// for those on it: each of these needs ten of its sixteen 16 x 16 products and
// one operand (at most 32 columns: three products, the rows quartered among the
// waves).  The reduction mirrors them.  Waves skip products of columns past the
// matrices.  Bound: FP64 matrix cores (a plain FP64 product of 8192^2 reaches 71
// TFLOP/s here).  Time of A^H A, every tile whole and 4096 tile-splits -> now:
// 524288 x 256 c64 2674 -> 2330 us, x 128 c128 1229 -> 698, x 32 c64 515 -> 81;
// 8192 x 32 c128 55 -> 17; 524288 x 256 x 32 c64 (BW = 32) 963 -> 588.
// ---------------------------------------------------------------------------
constexpr int kGT = 64;   // output tile edge
constexpr int kGK = 16;   // rows per LDS stage
constexpr int kGramPerCu = 3;   // resident workgroups per CU (registers); one more of the BW = 32 instances
constexpr int kGramRounds = 2;

// (row tile, column tile) of output tile t.  General product: column-major over all
// tiles.  Hermitian product: the tiles above the diagonal, column by column.
__device__ inline void gram_tile(int t, int tiles_a, bool herm, int *ta, int *tb) {
    if (!herm) {
        *ta = t % tiles_a;
        *tb = t / tiles_a;
        return;
    }
    int c = 1;
    while (c * (c + 1) / 2 <= t) ++c;
    *tb = c;
    *ta = t - c * (c - 1) / 2;
}

// Element types TA, TB of A and B (double: c128, float: c64) are template
// parameters: a storage precision chosen at run time made every element access
// a branch and kept the prefetch registers FP64 wide (two waves per SIMD
// instead of three; 287 -> 162 ms for a 33.5 M x 256 c64 product).  Stages stay
// in registers in the storage type until they go to LDS as FP64.
template <typename TA, typename TB, int BW, bool DIAG>
__global__ __launch_bounds__(kT) void gram_kernel(const void *A, int nb_a, const void *B, int nb_b, int64_t n,
                                                   int m1, int m2, int tiles_a, int herm, int64_t rows_per_split,
                                                   int ntiles, int nsplit, double *part) {
    // output tile 64 (columns of A) x BW (columns of B); BW = 32 for products of at
    // most 32 columns of B (Rayleigh-Ritz and TSQR panels), so no wave multiplies zeros
    constexpr int KG = kGK;
    constexpr int NY = BW / 32;                // 16-column MFMA tiles per wave
    using RA = typename std::conditional<std::is_same<TA, double>::value, double2, float2>::type;
    using RB = typename std::conditional<std::is_same<TB, double>::value, double2, float2>::type;
    __shared__ double2 sa[KG][kGT];
    __shared__ double2 sb[DIAG ? 1 : KG][BW];
    // all tiles of a split on one XCD (workgroup w runs on XCD w % 8): they read the same rows
    int tile, split;
    if (nsplit % 8 == 0) {
        const int k = blockIdx.x / 8;
        tile = k % ntiles;
        split = k / ntiles * 8 + blockIdx.x % 8;
    } else {
        tile = blockIdx.x % ntiles;
        split = blockIdx.x / ntiles;
    }
    int ta = tile, tb = tile;
    if constexpr (!DIAG) gram_tile(tile, tiles_a, herm != 0, &ta, &tb);
    const int a0 = ta * kGT, b0 = tb * BW;
    const int64_t r0 = (int64_t)split * rows_per_split;
    const int64_t r1 = r0 + rows_per_split < n ? r0 + rows_per_split : n;

    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int wa = (wv & 1) * 32, wb = (wv >> 1) * (BW / 2);  // wave's 32 x BW/2 sub-tile
    // whether the wave's products, and those of its second 16 columns of B, reach into the matrices
    const bool live = __builtin_amdgcn_readfirstlane(a0 + wa < m1 && b0 + wb < m2);
    const bool both = __builtin_amdgcn_readfirstlane(b0 + wb + 16 < m2);
    // DIAG: products (row, column) in units of 16: role 0 (0,0) (0,1) (1,1), role 1
    // (0,2) (0,3) (1,3), role 2 (1,2) (2,2), role 3 (2,3) (3,3); the roles of three
    // products alternate between the wave pairs (that is, between SIMDs)
    const int role = __builtin_amdgcn_readfirstlane((wv + 2 * (split & 1)) & 3);
    const bool quarter = DIAG && m1 <= 32;   // one tile of at most 2 x 2 products
    const int part_of = quarter ? 0 : role;
    const int np = part_of < 2 ? 3 : 2;
    int ro[3], co[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        ro[p] = 16 * (p == 2 ? 1 : part_of < 2 ? 0 : part_of - 1 + p);
        co[p] = 16 * (p == 2 ? 1 + 2 * part_of : part_of == 0 ? p : part_of == 1 ? 2 + p : part_of);
    }

    // two accumulators per 16 x 16 tile: real and imaginary part of the sum
    d4v acc[2][NY][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[x][y][q] = d4v{0.0, 0.0, 0.0, 0.0};

    // Stages of KG rows x 64 columns of A and KG rows x BW columns of B (zero
    // outside the matrices): the next stage's global loads are issued before the
    // current stage's products, so their latency hides behind the matrix-core work.
    constexpr int kPerA = KG * kGT / kT, kPerB = DIAG ? 0 : KG * BW / kT;   // elements per thread
    RA ra[kPerA];
    RB rb2[kPerB > 0 ? kPerB : 1];
    auto fetch = [&](int64_t rbase) {
#pragma unroll
        for (int q = 0; q < kPerA; ++q) {
            const int t = threadIdx.x + q * kT;
            const int rr = t / kGT, cc = t % kGT;
            const int64_t i = rbase + rr;
            RA va{};
            if (i < r1 && a0 + cc < m1) va = static_cast<const RA *>(A)[blocked_index(n, nb_a, i, a0 + cc)];
            ra[q] = va;
        }
#pragma unroll
        for (int q = 0; q < kPerB; ++q) {
            const int t = threadIdx.x + q * kT;
            const int rr = t / BW, cc = t % BW;
            const int64_t i = rbase + rr;
            RB vb{};
            if (i < r1 && b0 + cc < m2) vb = static_cast<const RB *>(B)[blocked_index(n, nb_b, i, b0 + cc)];
            rb2[q] = vb;
        }
    };
    if (r0 < r1) fetch(r0);
    hold_acc<NY>(acc);
    for (int64_t rb = r0; rb < r1; rb += KG) {
#pragma unroll
        for (int q = 0; q < kPerA; ++q) {
            const int t = threadIdx.x + q * kT;
            sa[t / kGT][t % kGT] = double2{(double)ra[q].x, (double)ra[q].y};
        }
#pragma unroll
        for (int q = 0; q < kPerB; ++q) {
            const int t = threadIdx.x + q * kT;
            sb[t / BW][t % BW] = double2{(double)rb2[q].x, (double)rb2[q].y};
        }
        __syncthreads();
        if (rb + KG < r1) fetch(rb + KG);
        // conj(a) b = (ar br + ai bi) + i (ar bi - ai br)
        auto product = [&](const double2 av, const double2 bv, d4v *c) {
            c[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.x, c[0], 0, 0, 0);
            c[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, bv.y, c[0], 0, 0, 0);
            c[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.y, c[1], 0, 0, 0);
            c[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av.y, bv.x, c[1], 0, 0, 0);
        };
        if constexpr (DIAG) {
            // at most 32 columns: every wave takes role 0 for a quarter of the rows
#pragma unroll
            for (int k0 = 0; k0 < KG; k0 += 4) {
                if (quarter && k0 != 4 * role) continue;
                const int kk = k0 + lane / 16;
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    product(sa[kk][ro[p] + lane % 16], sa[kk][co[p] + lane % 16], acc[0][p % NY]);
                if (np > 2) product(sa[kk][ro[2] + lane % 16], sa[kk][co[2] + lane % 16], acc[1][0]);
            }
        } else if (live) {
#pragma unroll
            for (int k0 = 0; k0 < KG; k0 += 4) {
                const int kk = k0 + lane / 16;
                double2 av[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) av[x] = sa[kk][wa + 16 * x + lane % 16];
#pragma unroll
                for (int y = 0; y < NY; ++y) {
                    if (y > 0 && !both) continue;
                    const double2 bv = sb[kk][wb + 16 * y + lane % 16];
#pragma unroll
                    for (int x = 0; x < 2; ++x) product(av[x], bv, acc[x][y]);
                }
            }
        }
        hold_acc<NY>(acc);
        __syncthreads();
    }
    if constexpr (DIAG) {
        if (quarter) {
            // the four quarters' sums, in order, through the (idle) stage buffer
            double2 *sw = &sa[0][0];
            for (int v = 1; v < 4; ++v) {
                if (role == v) {
#pragma unroll
                    for (int p = 0; p < 3; ++p)
#pragma unroll
                        for (int r = 0; r < 4; ++r) sw[(p * 4 + r) * 64 + lane] = double2{acc[p / 2][p % 2][0][r], acc[p / 2][p % 2][1][r]};
                }
                __syncthreads();
                if (role == 0) {
#pragma unroll
                    for (int p = 0; p < 3; ++p)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const double2 t = sw[(p * 4 + r) * 64 + lane];
                            acc[p / 2][p % 2][0][r] += t.x;
                            acc[p / 2][p % 2][1][r] += t.y;
                        }
                }
                __syncthreads();
            }
            if (role != 0) return;
        }
    }
    // write the partial tile into a 64 x 64 slot (column-major inside the slot;
    // a BW = 32 tile fills its first 32 columns, the reduction reads no others)
    double2 *out = reinterpret_cast<double2 *>(part) + ((int64_t)split * ntiles + tile) * (kGT * kGT);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y) {
            const int p = x * NY + y;
            if (DIAG && p >= np) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ra = (DIAG ? ro[p % 3] : wa + 16 * x) + lane / 16 + 4 * r;  // row of S (column of A)
                const int cb = (DIAG ? co[p % 3] : wb + 16 * y) + lane % 16;            // column of S within the tile
                double2 v;
                v.x = acc[x][y][0][r];
                v.y = acc[x][y][1][r];
                out[(int64_t)cb * kGT + ra] = v;
            }
        }
}

// S = sum over splits of the partial tiles; S column-major, ld.  A workgroup sums
// kRE neighbouring entries of a tile, each with kRS threads that take every
// kRS-th split and are then added in order.  (One thread per entry, walking all
// splits one after the other, left a product of few tiles with a few workgroups
// and took longer than the product itself: 524288 x 64 x 32, 2 tiles, 1024
// splits: 288 of the 424 us that the whole product took, now 179.)
// Hermitian product: the tiles on the diagonal first (nsplit_d splits each), then
// the ntiles - tiles_a above it; entries above the diagonal also give their mirror
// image S(b, a) = conj S(a, b).
// per_tile workgroups a tile (its first columns, where it is narrow); more than
// kReduceMaxGrid (32768 tiles) go through the loop, since a grid holds at most 2^32 - 1
// work-items.
constexpr int kRE = 32, kRS = kT / kRE;
constexpr int64_t kReduceMaxGrid = 1 << 22;
__global__ __launch_bounds__(kT) void gram_reduce_kernel(const double *part, int nsplit, int nsplit_d, int ntiles,
                                                         int per_tile, int tiles_a, int herm, int m1, int m2,
                                                         double *S, int ld) {
    __shared__ double2 sred[kRS][kRE];
    const int el = threadIdx.x % kRE, sl = threadIdx.x / kRE;
    const int64_t total = (int64_t)ntiles * per_tile;
    for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {
        const double2 *p = reinterpret_cast<const double2 *>(part);
        int tile = static_cast<int>(w / per_tile), set = ntiles, splits = nsplit;
        const int e = static_cast<int>(w % per_tile) * kRE + el;
        int ta = tile, tb = tile;
        if (!herm) {
            gram_tile(tile, tiles_a, false, &ta, &tb);
        } else if (tile < tiles_a) {
            set = tiles_a;
            splits = nsplit_d;
        } else {
            tile -= tiles_a;
            set = ntiles - tiles_a;
            p += (int64_t)nsplit_d * tiles_a * (kGT * kGT);
            gram_tile(tile, tiles_a, true, &ta, &tb);
        }
        double sr = 0.0, si = 0.0;
#pragma unroll 8
        for (int s = sl; s < splits; s += kRS) {
            const double2 v = p[((int64_t)s * set + tile) * (kGT * kGT) + e];
            sr += v.x;
            si += v.y;
        }
        sred[sl][el] = double2{sr, si};
        __syncthreads();
        if (sl == 0) {
            for (int q = 1; q < kRS; ++q) {
                sr += sred[q][el].x;
                si += sred[q][el].y;
            }
            const int a = ta * kGT + e % kGT, b = tb * kGT + e / kGT;
            if (a < m1 && b < m2 && !(herm && a > b)) {
                reinterpret_cast<double2 *>(S)[(int64_t)b * ld + a] = double2{sr, si};
                if (herm && a != b) reinterpret_cast<double2 *>(S)[(int64_t)a * ld + b] = double2{sr, -si};
            }
        }
        if (w + gridDim.x < total) __syncthreads();   // sred is written again
    }
}

// ---------------------------------------------------------------------------
// Update: Z(i, c) = sum_k A(i, k) M(k, c), M FP64 complex column-major (ld).
// 64 rows x 64 columns of Z per workgroup; k staged 16 at a time.
// ---------------------------------------------------------------------------
// Element types TA of A and TZ of Z (double: c128, float: c64) are template
// parameters, as for the Gram product.
// Z = A M, or Z = S - A M when TS (the storage type of S, blocked width nb_s) is
// not void; S may be Z itself (each entry is read by the thread that writes it).
template <typename TA, typename TZ, int BW, typename TS = void>
__global__ __launch_bounds__(kT) void update_kernel(const void *A, int nb_a, const double *M, int ldm, void *Z,
                                                    int nb_z, int64_t n, int m1, int m2, const void *S = nullptr,
                                                    int nb_s = 1) {
    // output tile 64 rows x BW columns of Z (BW = 32 when Z has at most 32 columns)
    constexpr int NY = BW / 32;                // 16-column MFMA tiles per wave
    using RA = typename std::conditional<std::is_same<TA, double>::value, double2, float2>::type;
    using RZ = typename std::conditional<std::is_same<TZ, double>::value, double2, float2>::type;
    __shared__ double2 sa[kGT][kGK + 1];
    __shared__ double2 sm[kGK][BW];
    const int64_t i0 = (int64_t)blockIdx.x * kGT;
    const int c0 = blockIdx.y * BW;
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int wi = (wv & 1) * 32, wc = (wv >> 1) * (BW / 2);
    const double2 *Mc = reinterpret_cast<const double2 *>(M);
    const bool live = __builtin_amdgcn_readfirstlane(c0 + wc < m2);
    const bool both = __builtin_amdgcn_readfirstlane(c0 + wc + 16 < m2);

    // two accumulators per 16 x 16 tile: real and imaginary part of the sum
    d4v acc[2][NY][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[x][y][q] = d4v{0.0, 0.0, 0.0, 0.0};

    // stages of kGK columns of A (64 rows) and kGK rows of M (BW columns): the next
    // stage's global loads are issued before the current stage's products
    constexpr int kPerA = kGT * kGK / kT, kPerM = BW * kGK / kT;   // elements per thread
    RA pa[kPerA];
    double2 pm[kPerM];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < kPerA; ++q) {
            const int t = threadIdx.x + q * kT;
            const int rr = t / kGK, kk = t % kGK;
            const int64_t i = i0 + rr;
            RA va{};
            if (i < n && k0 + kk < m1) va = static_cast<const RA *>(A)[blocked_index(n, nb_a, i, k0 + kk)];
            pa[q] = va;
        }
#pragma unroll
        for (int q = 0; q < kPerM; ++q) {
            const int t = threadIdx.x + q * kT;
            const int km = t / BW, cc = t % BW;
            double2 vm{0.0, 0.0};
            if (k0 + km < m1 && c0 + cc < m2) vm = Mc[(int64_t)(c0 + cc) * ldm + k0 + km];
            pm[q] = vm;
        }
    };
    fetch(0);
    hold_acc<NY>(acc);
    for (int k0 = 0; k0 < m1; k0 += kGK) {
#pragma unroll
        for (int q = 0; q < kPerA; ++q) {
            const int t = threadIdx.x + q * kT;
            sa[t / kGK][t % kGK] = double2{(double)pa[q].x, (double)pa[q].y};
        }
#pragma unroll
        for (int q = 0; q < kPerM; ++q) {
            const int t = threadIdx.x + q * kT;
            sm[t / BW][t % BW] = pm[q];
        }
        __syncthreads();
        if (k0 + kGK < m1) fetch(k0 + kGK);
        // a m = (ar mr - ai mi) + i (ar mi + ai mr)
        auto product = [&](const double2 av, const double2 mv, d4v *c) {
            c[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, mv.x, c[0], 0, 0, 0);
            c[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av.y, mv.y, c[0], 0, 0, 0);
            c[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, mv.y, c[1], 0, 0, 0);
            c[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, mv.x, c[1], 0, 0, 0);
        };
        if (live) {
#pragma unroll
            for (int kb = 0; kb < kGK; kb += 4) {
                const int kk = kb + lane / 16;
                double2 av[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) av[x] = sa[wi + 16 * x + lane % 16][kk];
#pragma unroll
                for (int y = 0; y < NY; ++y) {
                    if (y > 0 && !both) continue;
                    const double2 mv = sm[kk][wc + 16 * y + lane % 16];
#pragma unroll
                    for (int x = 0; x < 2; ++x) product(av[x], mv, acc[x][y]);
                }
            }
        }
        hold_acc<NY>(acc);
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i = i0 + wi + 16 * x + lane / 16 + 4 * r;
                const int c = c0 + wc + 16 * y + lane % 16;
                if (i < n && c < m2) {
                    double vx = acc[x][y][0][r], vy = acc[x][y][1][r];
                    if constexpr (!std::is_void<TS>::value) {
                        using RS = typename std::conditional<std::is_same<TS, double>::value, double2, float2>::type;
                        const RS sv = static_cast<const RS *>(S)[blocked_index(n, nb_s, i, c)];
                        vx = static_cast<double>(sv.x) - vx;
                        vy = static_cast<double>(sv.y) - vy;
                    }
                    RZ v;
                    v.x = static_cast<TZ>(vx);
                    v.y = static_cast<TZ>(vy);
                    static_cast<RZ *>(Z)[blocked_index(n, nb_z, i, c)] = v;
                }
            }
}

// ---------------------------------------------------------------------------
// Cyclic Jacobi eigensolver for a Hermitian m x m FP64 complex matrix.
// A sweep is me - 1 rounds (me = m rounded up to even) of the round-robin
// ordering; a round rotates me/2 disjoint (p, q) pairs.  For the pair block
// [[a, b], [conj(b), d]], b = |b| e^{i phi}, the rotation is
// J = diag(1, e^{-i phi}) [[c, s], [-s, c]] with t = s / c the smaller root of
// t^2 + 2 zeta t - 1 = 0, zeta = (d - a) / (2 |b|); A <- J^H A J, V <- V J.
//
// One launch per round, one workgroup per pair: the workgroup first applies the
// previous round's row rotations (A <- J^H A, every pair) to its own two
// columns -- each column belongs to exactly one pair of every round, so every
// column receives them -- then forms its rotation from the updated columns and
// applies the column rotation to A and V.  The last round of a sweep is closed
// by a launch that applies its row rotations to all columns.  The rotated pair's
// off-diagonal entries are stored as exact zeros and its diagonal as real.
// ---------------------------------------------------------------------------
constexpr int kMaxM = 512;
constexpr int kJW = 256;       // threads per Jacobi workgroup
constexpr int kJNormG = 64;    // workgroups of the norm reduction

__device__ inline int rr_player(int m, int r, int k) {
    // round r, seat k of the circle method over players 0..m-1 (m even):
    // seat 0 holds player 0, the other seats rotate over 1..m-1
    const int x = k - 1 + r;   // r < m - 1, k < m
    return k == 0 ? 0 : (x >= m - 1 ? x - (m - 1) : x) + 1;
}

struct JacobiRound {
    int *p, *q;           // [2][kMaxM / 2] pair indices (p < q; q >= m: no rotation)
    double *c, *sr, *si;  // [2][kMaxM / 2] c and s e^{-i phi}
};

// rows p, q of column `col` <- J^H (rows p, q) for the rotation in slot `slot`, pair kk
__device__ inline void jacobi_row_rotate(double2 *Ac, int lda, const JacobiRound &jr, int slot, int kk, int col,
                                         int m) {
    const int h = slot * (kMaxM / 2) + kk;
    const int p = jr.p[h], q = jr.q[h];
    if (q >= m) return;
    const double c = jr.c[h], sr = jr.sr[h], si = -jr.si[h];  // s e^{+i phi}
    const double s = sqrt(sr * sr + si * si);
    const double er = s > 0.0 ? sr / s : 1.0, ei = s > 0.0 ? si / s : 0.0;
    const double2 x = Ac[(int64_t)col * lda + p], y = Ac[(int64_t)col * lda + q];
    double2 np, nq;
    np.x = c * x.x - (sr * y.x - si * y.y);
    np.y = c * x.y - (sr * y.y + si * y.x);
    nq.x = s * x.x + c * (er * y.x - ei * y.y);
    nq.y = s * x.y + c * (er * y.y + ei * y.x);
    if (col == q) np = double2{0.0, 0.0};
    if (col == p) {
        nq = double2{0.0, 0.0};
        np.y = 0.0;
    }
    if (col == q) nq.y = 0.0;
    Ac[(int64_t)col * lda + p] = np;
    Ac[(int64_t)col * lda + q] = nq;
}

__global__ __launch_bounds__(kJW) void jacobi_round_kernel(int m, int me, int r, int has_prev, double *A, int lda,
                                                           double *V, int ldv, JacobiRound jr) {
    __shared__ double s_par[3];
    double2 *Ac = reinterpret_cast<double2 *>(A);
    double2 *Vc = reinterpret_cast<double2 *>(V);
    const int half = me / 2, k = blockIdx.x, tid = threadIdx.x;
    int p = rr_player(me, r, k), q = rr_player(me, r, me - 1 - k);
    if (p > q) { const int tmp = p; p = q; q = tmp; }
    const int cur = r & 1, prv = cur ^ 1;
    // (a) the previous round's row rotations on columns p and q
    if (has_prev) {
        for (int t = tid; t < 2 * half; t += kJW) {
            const int col = t < half ? p : q;
            if (col < m) jacobi_row_rotate(Ac, lda, jr, prv, t % half, col, m);
        }
    }
    __syncthreads();
    // (b) this round's rotation from the updated columns
    if (tid == 0) {
        double c = 1.0, sr = 0.0, si = 0.0;
        if (q < m) {
            const double a = Ac[(int64_t)p * lda + p].x;
            const double d = Ac[(int64_t)q * lda + q].x;
            const double2 b = Ac[(int64_t)q * lda + p];  // A[p][q]
            const double ab = sqrt(b.x * b.x + b.y * b.y);
            if (ab > 0.0) {
                const double zeta = (d - a) / (2.0 * ab);
                const double t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
                c = 1.0 / sqrt(1.0 + t * t);
                const double sn = t * c;
                sr = sn * b.x / ab;   // s e^{-i phi} = s conj(b) / |b|
                si = -sn * b.y / ab;
            }
        }
        const int h = cur * (kMaxM / 2) + k;
        jr.p[h] = p;
        jr.q[h] = q;
        jr.c[h] = c;
        jr.sr[h] = sr;
        jr.si[h] = si;
        s_par[0] = c;
        s_par[1] = sr;
        s_par[2] = si;
    }
    __syncthreads();
    if (q >= m) return;
    // (c) columns: A(:,p) <- c A(:,p) - s e^{-i phi} A(:,q); A(:,q) <- s A(:,p) + c e^{-i phi} A(:,q); same for V
    const double c = s_par[0], sr = s_par[1], si = s_par[2];
    const double s = sqrt(sr * sr + si * si);
    const double er = s > 0.0 ? sr / s : 1.0, ei = s > 0.0 ? si / s : 0.0;
    for (int t = tid; t < 2 * m; t += kJW) {
        const int which = t / m, row = t % m;
        double2 *M = which ? Vc : Ac;
        const int ld = which ? ldv : lda;
        const double2 x = M[(int64_t)p * ld + row], y = M[(int64_t)q * ld + row];
        double2 np, nq;
        np.x = c * x.x - (sr * y.x - si * y.y);
        np.y = c * x.y - (sr * y.y + si * y.x);
        nq.x = s * x.x + c * (er * y.x - ei * y.y);
        nq.y = s * x.y + c * (er * y.y + ei * y.x);
        M[(int64_t)p * ld + row] = np;
        M[(int64_t)q * ld + row] = nq;
    }
}

// the row rotations of round slot `slot` on every column (closes a sweep)
__global__ __launch_bounds__(kJW) void jacobi_rows_kernel(int m, int me, int slot, double *A, int lda,
                                                          JacobiRound jr) {
    double2 *Ac = reinterpret_cast<double2 *>(A);
    const int half = me / 2;
    for (int col = blockIdx.x; col < m; col += gridDim.x)
        for (int t = threadIdx.x; t < half; t += kJW) jacobi_row_rotate(Ac, lda, jr, slot, t, col, m);
}

// The same sweeps for a matrix that fits in the LDS of one CU with its eigenvectors
// (m <= kJSmall), all of them in one launch of one workgroup.
// Bound: the chain of a round (pair entries -> rotation -> barrier -> update ->
// barrier), about 0.8 us at m = 32; a launch per round took about 6 us each with its
// gap, plus a host synchronisation per sweep.  m = 32: about 1.1 ms -> 0.21 ms.  Larger
// matrices (2 m (m + 1) entries in 160 KB of LDS) keep a launch per round.
// With delta = d - a, h = sqrt(delta^2 + 4 |b|^2), r = |delta| + h the smaller rotation is
// c = r g, s = 2 |b| g (sign of delta), g = 1 / sqrt(2 h r): one root and one inverse
// root in a row instead of four roots and five divisions.  Columns are rotated as
// (x, y) <- (c x - sigma y, conj(sigma) x + c y), sigma = s e^{-i phi}, which leaves out
// the factor e^{-i phi} of the second column; a second wave keeps the product of
// these factors per column, and the eigenvectors get it at the end, so they carry
// the phases of the rotations above.  The matrix is scaled by a power of two.
constexpr int kJSmall = 64;
// |b|^2 at or below this (of a matrix with entries of order 1) is set to zero without a
// rotation: nearer the smallest normal number c and sigma lose their digits, and with
// equal diagonal entries the rotation would not be unitary
constexpr double kJTiny2 = 1e-280;
struct __align__(16) JacobiPair {
    double c, sr, si;   // c, sigma
    int p, q;
};

__device__ inline void jacobi_rotate(double c, double sr, double si, double2 &x, double2 &y) {
    const double2 nx{c * x.x - (sr * y.x - si * y.y), c * x.y - (sr * y.y + si * y.x)};
    const double2 ny{c * y.x + (sr * x.x + si * x.y), c * y.y + (sr * x.y - si * x.x)};
    x = nx;
    y = ny;
}

constexpr size_t jacobi_small_lds(int me) {
    return (size_t)2 * me * (me + 1) * 16 + (size_t)(me / 2) * sizeof(JacobiPair) + (size_t)me * 16 +
           16 * sizeof(double);
}

__global__ __launch_bounds__(1024) void jacobi_small_kernel(int m, int me, const double *A, int lda, double *V, int ldv,
                                                            double *w, int max_sweeps, double tol, int *status) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int ld = me + 1;
    double2 *sa = reinterpret_cast<double2 *>(smem);     // column c at sa + c ld
    double2 *sv = sa + me * ld;
    JacobiPair *pr = reinterpret_cast<JacobiPair *>(sv + me * ld);
    double2 *ph = reinterpret_cast<double2 *>(pr + me / 2);   // left-out phase of every column
    double *sred = reinterpret_cast<double *>(ph + me);
    const int tid = threadIdx.x, nt = blockDim.x, half = me / 2;
    const int lane = tid & 63, wv = tid >> 6, waves = nt >> 6;
    const double2 *Ac = reinterpret_cast<const double2 *>(A);
    double amax = 0.0;
    for (int t = tid; t < me * me; t += nt) {
        const int r = t % me, c = t / me;
        const double2 v = r < m && c < m ? Ac[(int64_t)c * lda + r] : double2{0.0, 0.0};
        sa[c * ld + r] = v;
        sv[c * ld + r] = double2{r == c ? 1.0 : 0.0, 0.0};
        amax = fmax(amax, fmax(fabs(v.x), fabs(v.y)));
    }
    for (int t = tid; t < me; t += nt) ph[t] = double2{1.0, 0.0};
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) amax = fmax(amax, __shfl_xor(amax, k));
    if (lane == 0) sred[wv] = amax;
    __syncthreads();
    for (int k = 0; k < waves; ++k) amax = fmax(amax, sred[k]);
    // a power of two brings the largest entry to [1, 2): no square over- or underflows
    const int ex = amax > 0.0 && amax < INFINITY ? ilogb(amax) : 0;
    for (int t = tid; t < me * me; t += nt) {
        const int at = t / me * ld + t % me;
        sa[at] = double2{ldexp(sa[at].x, -ex), ldexp(sa[at].y, -ex)};
    }
    __syncthreads();
    // squared Frobenius norm, off-diagonal entries only if `off` (every thread gets it)
    auto norm2 = [&](bool off) {
        double acc = 0.0;
        for (int t = tid; t < me * me; t += nt) {
            const int r = t % me, c = t / me;
            if (off && r == c) continue;
            const double2 v = sa[c * ld + r];
            acc += v.x * v.x + v.y * v.y;
        }
#pragma unroll
        for (int k = 32; k >= 1; k >>= 1) acc += __shfl_xor(acc, k);
        if (lane == 0) sred[wv] = acc;
        __syncthreads();
        acc = 0.0;
        for (int k = 0; k < waves; ++k) acc += sred[k];
        __syncthreads();
        return acc;
    };
    // this thread's items of every round: 2 x 2 blocks of A (k1, k2), then pairs of V (row, k2)
    constexpr int IT = (kJSmall / 2 * (kJSmall / 2) + kJSmall / 2 * kJSmall) / 1024;
    const int nb2 = half * half, items = nb2 + half * me;
    int i1[IT], i2[IT];
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        const int t = tid + u * nt;
        i1[u] = t < nb2 ? t % half : (t - nb2) % me;
        i2[u] = t < nb2 ? t / half : (t - nb2) / me;
    }
    const double limit = tol * tol * norm2(false);
    bool done = norm2(true) <= limit;
    int sweep = 0;
    for (; sweep < max_sweeps && !done; ++sweep) {
        for (int r = 0; r < me - 1; ++r) {
            // wave 0: rotations; wave 1: phases
            if (lane < half && wv < 2) {
                int p = rr_player(me, r, lane), q = rr_player(me, r, me - 1 - lane);
                if (p > q) { const int tmp = p; p = q; q = tmp; }
                const double2 b = sa[q * ld + p];
                const double b2 = b.x * b.x + b.y * b.y;
                if (wv == 0) {
                    const double d = sa[q * ld + q].x - sa[p * ld + p].x;
                    JacobiPair j{1.0, 0.0, 0.0, p, q};
                    if (b2 > kJTiny2) {
                        const double h = sqrt(fma(d, d, 4.0 * b2)), rr = fabs(d) + h;
                        const double g = 1.0 / sqrt(2.0 * h * rr), g2 = d >= 0.0 ? 2.0 * g : -2.0 * g;
                        j.c = rr * g;
                        j.sr = g2 * b.x;
                        j.si = -g2 * b.y;
                    }
                    pr[lane] = j;
                } else if (b2 > kJTiny2) {
                    const double2 u = ph[p];
                    const double f = sa[q * ld + q].x >= sa[p * ld + p].x ? rsqrt(b2) : -rsqrt(b2);
                    const double er = f * b.x, ei = -f * b.y;   // e^{-i phi}, with the sign of s
                    ph[q] = double2{er * u.x - ei * u.y, er * u.y + ei * u.x};
                }
            }
            __syncthreads();
            // A <- J^H A J in 2 x 2 blocks (rows of pair k1, columns of pair k2), V <- V J
#pragma unroll
            for (int u = 0; u < IT; ++u) {
                const int t = tid + u * nt;
                if (t < nb2) {
                    const int k1 = i1[u], k2 = i2[u];
                    const JacobiPair r1 = pr[k1], c2 = pr[k2];
                    double2 *pp = sa + c2.p * ld + r1.p, *qp = sa + c2.p * ld + r1.q;   // row p, q of column p
                    double2 *pq = sa + c2.q * ld + r1.p, *qq = sa + c2.q * ld + r1.q;   // row p, q of column q
                    double2 a00 = *pp, a10 = *qp, a01 = *pq, a11 = *qq;
                    jacobi_rotate(c2.c, c2.sr, c2.si, a00, a01);
                    jacobi_rotate(c2.c, c2.sr, c2.si, a10, a11);
                    jacobi_rotate(r1.c, r1.sr, -r1.si, a00, a10);
                    jacobi_rotate(r1.c, r1.sr, -r1.si, a01, a11);
                    if (k1 == k2) {
                        a01 = a10 = double2{0.0, 0.0};
                        a00.y = a11.y = 0.0;
                    }
                    *pp = a00;
                    *qp = a10;
                    *pq = a01;
                    *qq = a11;
                } else if (t < items) {
                    const int row = i1[u];
                    const JacobiPair c2 = pr[i2[u]];
                    jacobi_rotate(c2.c, c2.sr, c2.si, sv[c2.p * ld + row], sv[c2.q * ld + row]);
                }
            }
            __syncthreads();
        }
        done = norm2(true) <= limit;
    }
    // eigenvalues ascending (ties by index), eigenvectors permuted alike
    double2 *Vc = reinterpret_cast<double2 *>(V);
    int *rank_of = reinterpret_cast<int *>(pr);
    if (tid < m) {
        const double d = sa[tid * ld + tid].x;
        int rank = 0;
        for (int u = 0; u < m; ++u) {
            const double e = sa[u * ld + u].x;
            rank += (e < d || (e == d && u < tid)) ? 1 : 0;
        }
        w[rank] = ldexp(d, ex);
        rank_of[tid] = rank;
        const double2 f = ph[tid];
        const double n = 1.0 / sqrt(f.x * f.x + f.y * f.y);   // rounding of the product only
        ph[tid] = double2{f.x * n, f.y * n};
    }
    __syncthreads();
    for (int t = tid; t < m * m; t += nt) {
        const int r = t % m, c = t / m;
        const double2 v = sv[c * ld + r], f = ph[c];
        Vc[(int64_t)rank_of[c] * ldv + r] = double2{v.x * f.x - v.y * f.y, v.x * f.y + v.y * f.x};
    }
    if (tid == 0) {
        status[0] = sweep;
        status[1] = done ? 1 : 0;
    }
}

// partial sums of |A_ij|^2 (off-diagonal only if `off`), one per workgroup, fixed order
__global__ __launch_bounds__(kJW) void jacobi_norm_kernel(int m, const double *A, int lda, int off,
                                                          double *part) {
    __shared__ double sred[kJW];
    const double2 *Ac = reinterpret_cast<const double2 *>(A);
    double acc = 0.0;
    for (int t = blockIdx.x * kJW + threadIdx.x; t < m * m; t += gridDim.x * kJW) {
        const int r = t % m, c = t / m;
        if (off && r == c) continue;
        const double2 v = Ac[(int64_t)c * lda + r];
        acc += v.x * v.x + v.y * v.y;
    }
    sred[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kJW / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) sred[threadIdx.x] += sred[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sred[0];
}

__global__ __launch_bounds__(kJW) void jacobi_init_kernel(int m, double *V, int ldv) {
    double2 *Vc = reinterpret_cast<double2 *>(V);
    for (int t = blockIdx.x * kJW + threadIdx.x; t < m * m; t += gridDim.x * kJW) {
        const int r = t % m, c = t / m;
        Vc[(int64_t)c * ldv + r] = double2{r == c ? 1.0 : 0.0, 0.0};
    }
}

// eigenvalues ascending (ties by index) into w, eigenvectors permuted alike (one workgroup)
__global__ __launch_bounds__(kJW) void jacobi_sort_kernel(int m, double *A, int lda, double *V, int ldv,
                                                          double *w, double *scratch) {
    double2 *Ac = reinterpret_cast<double2 *>(A);
    double2 *Vc = reinterpret_cast<double2 *>(V);
    int *rank_of = reinterpret_cast<int *>(scratch + m);
    const int tid = threadIdx.x;
    for (int t = tid; t < m; t += kJW) scratch[t] = Ac[(int64_t)t * lda + t].x;
    __syncthreads();
    for (int t = tid; t < m; t += kJW) {
        const double d = scratch[t];
        int rank = 0;
        for (int u = 0; u < m; ++u) {
            const double e = scratch[u];
            rank += (e < d || (e == d && u < t)) ? 1 : 0;
        }
        w[rank] = d;
        rank_of[t] = rank;
    }
    __syncthreads();
    // permuted copy of V through A's storage (A is no longer needed)
    for (int t = tid; t < m * m; t += kJW) {
        const int r = t % m, c = t / m;
        Ac[(int64_t)rank_of[c] * lda + r] = Vc[(int64_t)c * ldv + r];
    }
    __syncthreads();
    for (int t = tid; t < m * m; t += kJW) {
        const int r = t % m, c = t / m;
        Vc[(int64_t)c * ldv + r] = Ac[(int64_t)c * lda + r];
    }
}

// ---------------------------------------------------------------------------
// small helpers of the SVQB / Rayleigh-Ritz / residual steps
// ---------------------------------------------------------------------------

// d_i = diag(S)_ii^{-1/2} (1 for non-positive entries); S <- D S D
__global__ __launch_bounds__(kT) void svqb_scale_kernel(int m, double *S, int ld, double *d) {
    double2 *Sc = reinterpret_cast<double2 *>(S);
    __shared__ double sd[kMaxM];
    for (int t = threadIdx.x; t < m; t += kT) {
        const double v = Sc[(int64_t)t * ld + t].x;
        sd[t] = v > 0.0 ? 1.0 / sqrt(v) : 1.0;
        d[t] = sd[t];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < m * m; t += kT) {
        const int r = t % m, c = t / m;
        double2 v = Sc[(int64_t)c * ld + r];
        const double f = sd[r] * sd[c];
        v.x *= f;
        v.y *= f;
        Sc[(int64_t)c * ld + r] = v;
    }
}

// T(:, c) = D V(:, first + c) / sqrt(w[first + c]), c < k (the kept directions)
__global__ __launch_bounds__(kT) void svqb_transform_kernel(int m, int k, int first, const double *d,
                                                            const double *V, int ldv, const double *w,
                                                            double *T, int ldt) {
    const double2 *Vc = reinterpret_cast<const double2 *>(V);
    double2 *Tc = reinterpret_cast<double2 *>(T);
    for (int t = blockIdx.x * kT + threadIdx.x; t < m * k; t += gridDim.x * kT) {
        const int r = t % m, c = t / m;
        const double f = d[r] / sqrt(w[first + c]);
        double2 v = Vc[(int64_t)(first + c) * ldv + r];
        v.x *= f;
        v.y *= f;
        Tc[(int64_t)c * ldt + r] = v;
    }
}

// G <- (G + G^H) / 2
__global__ __launch_bounds__(kT) void hermitise_kernel(int m, double *G, int ld) {
    double2 *Gc = reinterpret_cast<double2 *>(G);
    for (int t = blockIdx.x * kT + threadIdx.x; t < m * m; t += gridDim.x * kT) {
        const int r = t % m, c = t / m;
        if (r > c) continue;
        const double2 a = Gc[(int64_t)c * ld + r], b = Gc[(int64_t)r * ld + c];
        const double2 u = double2{0.5 * (a.x + b.x), 0.5 * (a.y - b.y)};
        Gc[(int64_t)c * ld + r] = u;
        Gc[(int64_t)r * ld + c] = double2{u.x, -u.y};
    }
}

// Per column c of one n x nb block (blocked storage, precision prec): partial
// sums over the rows of this workgroup of |HZ - theta_c Z|^2 and |Z|^2, written
// to part[(2 c + q) * G + w]; reduced in order by colsum_reduce_kernel.
__global__ __launch_bounds__(kT) void resid_partial_kernel(const void *HZ, const void *Z, int prec,
                                                           int64_t n, int nb, const double *theta,
                                                           double *part) {
    __shared__ double s0[kT], s1[kT];
    const int cpt = nb < kT ? nb : kT;           // columns handled in parallel
    const int rows = kT / cpt;
    const int c = threadIdx.x % cpt, rr = threadIdx.x / cpt;
    for (int cb = 0; cb < nb; cb += cpt) {
        const int cc = cb + c;
        double a = 0.0, b = 0.0;
        const double th = theta ? theta[cc] : 0.0;
        for (int64_t i = (int64_t)blockIdx.x * rows + rr; i < n; i += (int64_t)gridDim.x * rows) {
            const int64_t e = i * nb + cc;
            const double2 h = load_c(HZ, prec, e), z = load_c(Z, prec, e);
            const double rx = h.x - th * z.x, ry = h.y - th * z.y;
            a += rx * rx + ry * ry;
            b += z.x * z.x + z.y * z.y;
        }
        s0[threadIdx.x] = a;
        s1[threadIdx.x] = b;
        __syncthreads();
        if (rr == 0) {
            double sa = 0.0, sb = 0.0;
            for (int q = 0; q < rows; ++q) {
                sa += s0[q * cpt + c];
                sb += s1[q * cpt + c];
            }
            part[(int64_t)(2 * cc) * gridDim.x + blockIdx.x] = sa;
            part[(int64_t)(2 * cc + 1) * gridDim.x + blockIdx.x] = sb;
        }
        __syncthreads();
    }
}

// out[q] = sum_g part[q * G + g], q < count (fixed order)
__global__ __launch_bounds__(kT) void colsum_reduce_kernel(const double *part, int G, int count,
                                                           double *out) {
    __shared__ double s[kT];
    for (int q = blockIdx.x; q < count; q += gridDim.x) {
        double a = 0.0;
        for (int g = threadIdx.x; g < G; g += kT) a += part[(int64_t)q * G + g];
        s[threadIdx.x] = a;
        __syncthreads();
        for (int h = kT / 2; h > 0; h >>= 1) {
            if (threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[q] = s[0];
        __syncthreads();
    }
}

// T(:, c) = S(:, order[c]) for c < m (FP64 complex, column-major)
__global__ __launch_bounds__(kT) void permute_columns_kernel(int rows, int m, const double *S, int lds,
                                                             const int *order, double *T, int ldt) {
    const double2 *Sc = reinterpret_cast<const double2 *>(S);
    double2 *Tc = reinterpret_cast<double2 *>(T);
    for (int t = blockIdx.x * kT + threadIdx.x; t < rows * m; t += gridDim.x * kT) {
        const int r = t % rows, c = t / rows;
        Tc[(int64_t)c * ldt + r] = Sc[(int64_t)order[c] * lds + r];
    }
}

// Precision conversion of a blocked block vector (count complex entries).
__global__ __launch_bounds__(kT) void convert_kernel(const void *src, int prec_src, void *dst,
                                                     int prec_dst, int64_t count) {
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < count; t += (int64_t)gridDim.x * kT)
        store_c(dst, prec_dst, t, load_c(src, prec_src, t));
}

// SplitMix64 output function (Steele, Lea and Flood, OOPSLA 2014).
__device__ inline uint64_t splitmix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Random-phase columns c in [c_begin, c_end) of a blocked block vector:
// entry (i, c) = exp(2 pi i u), u = top 53 bits of splitmix64(k ^ i) / 2^53,
// k = splitmix64(splitmix64(seed) ^ (col0 + c - c_begin)).
__global__ __launch_bounds__(kT) void random_phase_kernel(void *X, int prec, int64_t n, int nb,
                                                          int c_begin, int c_end, uint64_t seed,
                                                          uint64_t col0, const int32_t *perm) {
    const uint64_t base = splitmix64(seed);
    const int64_t cols = c_end - c_begin;
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < n * cols;
         t += (int64_t)gridDim.x * kT) {
        const int64_t cc = t / n, i = t % n;
        const uint64_t kj = splitmix64(base ^ (col0 + (uint64_t)cc));
        const uint64_t row = perm ? (uint64_t)perm[i] : (uint64_t)i;  // the row's original index
        const double u = (double)(splitmix64(kj ^ row) >> 11) * 0x1.0p-53;
        double sn, cs;
        sincospi(2.0 * u, &sn, &cs);
        store_c(X, prec, blocked_index(n, nb, i, c_begin + static_cast<int>(cc)), double2{cs, sn});
    }
}

// Per column: index of the largest-modulus entry (ties: smallest row) and the
// unit phase conj(z)/|z| that makes it real positive; then scale the column.
__global__ __launch_bounds__(kT) void phase_argmax_kernel(const void *Z, int prec, int64_t n, int nb,
                                                          int m, double *phase) {
    __shared__ double sv[kT];
    __shared__ int64_t si[kT];
    for (int c = blockIdx.x; c < m; c += gridDim.x) {
        double best = -1.0;
        int64_t bi = 0;
        for (int64_t i = threadIdx.x; i < n; i += kT) {
            const double2 z = load_c(Z, prec, blocked_index(n, nb, i, c));
            const double a = z.x * z.x + z.y * z.y;
            if (a > best) { best = a; bi = i; }
        }
        sv[threadIdx.x] = best;
        si[threadIdx.x] = bi;
        __syncthreads();
        for (int h = kT / 2; h > 0; h >>= 1) {
            if (threadIdx.x < h) {
                const double o = sv[threadIdx.x + h];
                const int64_t oi = si[threadIdx.x + h];
                if (o > sv[threadIdx.x] || (o == sv[threadIdx.x] && oi < si[threadIdx.x])) {
                    sv[threadIdx.x] = o;
                    si[threadIdx.x] = oi;
                }
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const double2 z = load_c(Z, prec, blocked_index(n, nb, si[0], c));
            const double a = sqrt(z.x * z.x + z.y * z.y);
            phase[2 * c] = a > 0.0 ? z.x / a : 1.0;
            phase[2 * c + 1] = a > 0.0 ? -z.y / a : 0.0;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kT) void scale_columns_kernel(void *Z, int prec, int64_t n, int nb, int m,
                                                           const double *phase) {
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < n * m; t += (int64_t)gridDim.x * kT) {
        const int c = static_cast<int>(t / n);
        const int64_t i = t % n;
        const int64_t e = blocked_index(n, nb, i, c);
        const double2 z = load_c(Z, prec, e);
        const double pr = phase[2 * c], pi = phase[2 * c + 1];
        store_c(Z, prec, e, double2{z.x * pr - z.y * pi, z.x * pi + z.y * pr});
    }
}

}  // namespace

static bool pow2(int v) { return v >= 1 && (v & (v - 1)) == 0; }

int launch_gram(const void *A, int prec_a, int nb_a, const void *B, int prec_b, int nb_b, int64_t n,
                int m1, int m2, double *part, int nsplit, double *S, int ld, hipStream_t s) {
    if (!pow2(nb_a) || !pow2(nb_b)) CHEBFD_FAIL(CHEBFD_EINVAL, "block widths %d, %d must be powers of two", nb_a, nb_b);
    const int ta = (m1 + kGT - 1) / kGT, tb = (m2 + kGT - 1) / kGT;
    // A^H A: Hermitian, only the tiles on and above the diagonal
    const int herm = (A == B && prec_a == prec_b && nb_a == nb_b && m1 == m2) ? 1 : 0;
    const bool a64 = prec_a == CHEBFD_PREC_FP64, b64 = prec_b == CHEBFD_PREC_FP64;
    // at most 32 columns of B: 64 x 32 output tiles (the slots and the reduction stay 64 x 64)
    const bool narrow = !herm && m2 <= 32;
    DeviceProps d;
    int rc = device_props(&d);
    if (rc) return rc;
    // splits of a launch of `tiles` tiles: at most nsplit (the workspace), whole
    // rounds of the resident workgroups where there is more than one (2560 workgroups
    // for 768 places leave the last round a third full, and each split costs a 64 KB
    // slot written and read; two and three rounds measure alike), a multiple of 8
    // (one XCD per split)
    auto splits = [&](int tiles, int per_cu) {
        const int resident = per_cu * d.num_cus;
        const int rounds = std::min<int64_t>(kGramRounds, (int64_t)tiles * nsplit / resident);
        int k = rounds >= 1 ? std::max(1, rounds * resident / tiles) : nsplit;
        if (k >= 8) k -= k % 8;
        return k;
    };
    auto rows = [&](int k) { return ((n + k - 1) / k + kGK - 1) / kGK * kGK; };
    const int ntiles = herm ? ta * (ta - 1) / 2 : ta * tb;      // of the general kernel
    const int ks = ntiles > 0 ? splits(ntiles, narrow ? kGramPerCu + 1 : kGramPerCu) : 0;
    const int kd = herm ? splits(ta, kGramPerCu) : 0;
#define CHEBFD_GRAM_ONE(TA_, TB_, BW_, DIAG_, TILES_, K_, PART_)                                                 \
    hipLaunchKernelGGL((gram_kernel<TA_, TB_, BW_, DIAG_>), dim3((TILES_) * (K_)), dim3(kT), 0, s, A, nb_a, B,   \
                       nb_b, n, m1, m2, ta, herm, rows(K_), TILES_, K_, PART_)
#define CHEBFD_GRAM(TA_, TB_)                                                     \
    do {                                                                          \
        if (narrow)                                                               \
            CHEBFD_GRAM_ONE(TA_, TB_, 32, false, ntiles, ks, part);               \
        else                                                                      \
            CHEBFD_GRAM_ONE(TA_, TB_, 64, false, ntiles, ks, part);               \
    } while (0)
    if (herm) {
        if (a64)
            CHEBFD_GRAM_ONE(double, double, 64, true, ta, kd, part);
        else
            CHEBFD_GRAM_ONE(float, float, 64, true, ta, kd, part);
        CHEBFD_HIP(hipGetLastError());
        double *above = part + (size_t)kd * ta * kGT * kGT * 2;
        if (ntiles > 0) {
            if (a64)
                CHEBFD_GRAM_ONE(double, double, 64, false, ntiles, ks, above);
            else
                CHEBFD_GRAM_ONE(float, float, 64, false, ntiles, ks, above);
        }
    } else if (a64 && b64) {
        CHEBFD_GRAM(double, double);
    } else if (a64) {
        CHEBFD_GRAM(double, float);
    } else if (b64) {
        CHEBFD_GRAM(float, double);
    } else {
        CHEBFD_GRAM(float, float);
    }
#undef CHEBFD_GRAM
#undef CHEBFD_GRAM_ONE
    CHEBFD_HIP(hipGetLastError());
    const int all = herm ? ta + ntiles : ntiles;
    const int per_tile = kGT * (narrow ? 32 : kGT) / kRE;
    const unsigned G = static_cast<unsigned>(std::min((int64_t)all * per_tile, kReduceMaxGrid));
    hipLaunchKernelGGL(gram_reduce_kernel, dim3(G), dim3(kT), 0, s, part, ks, kd, all, per_tile, ta, herm, m1, m2, S,
                       ld);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

size_t gram_part_bytes(int m1, int m2, int nsplit) {
    const size_t ta = (m1 + kGT - 1) / kGT, tb = (m2 + kGT - 1) / kGT;
    return ta * tb * (size_t)nsplit * kGT * kGT * 16;
}

int launch_update(const void *A, int prec_a, int nb_a, const double *M, int ldm, void *Z, int prec_z,
                  int nb_z, int64_t n, int m1, int m2, hipStream_t s) {
    if (!pow2(nb_a) || !pow2(nb_z)) CHEBFD_FAIL(CHEBFD_EINVAL, "block widths %d, %d must be powers of two", nb_a, nb_z);
    // at most 32 columns of Z: 64 x 32 output tiles
    const int bw = m2 <= 32 ? 32 : kGT;
    const dim3 grid(static_cast<unsigned>((n + kGT - 1) / kGT), (m2 + bw - 1) / bw);
    const bool a64 = prec_a == CHEBFD_PREC_FP64, z64 = prec_z == CHEBFD_PREC_FP64;
#define CHEBFD_UPD(TA_, TZ_)                                                                                     \
    do {                                                                                                         \
        if (bw == 32)                                                                                            \
            hipLaunchKernelGGL((update_kernel<TA_, TZ_, 32>), grid, dim3(kT), 0, s, A, nb_a, M, ldm, Z, nb_z, n, \
                               m1, m2);                                                                          \
        else                                                                                                     \
            hipLaunchKernelGGL((update_kernel<TA_, TZ_, 64>), grid, dim3(kT), 0, s, A, nb_a, M, ldm, Z, nb_z, n, \
                               m1, m2);                                                                          \
    } while (0)
    if (a64 && z64)
        CHEBFD_UPD(double, double);
    else if (a64)
        CHEBFD_UPD(double, float);
    else if (z64)
        CHEBFD_UPD(float, double);
    else
        CHEBFD_UPD(float, float);
#undef CHEBFD_UPD
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_update_sub(const void *A, int prec_a, int nb_a, const double *M, int ldm, const void *S, int prec_s,
                      int nb_s, double *Z, int nb_z, int64_t n, int m1, int m2, hipStream_t s) {
    if (!pow2(nb_a) || !pow2(nb_z) || !pow2(nb_s))
        CHEBFD_FAIL(CHEBFD_EINVAL, "block widths %d, %d, %d must be powers of two", nb_a, nb_s, nb_z);
    if (m2 > 32) CHEBFD_FAIL(CHEBFD_EINVAL, "Z = S - A M takes at most 32 columns (%d)", m2);
    const dim3 grid(static_cast<unsigned>((n + kGT - 1) / kGT), 1);
    const bool a64 = prec_a == CHEBFD_PREC_FP64, s64 = prec_s == CHEBFD_PREC_FP64;
#define CHEBFD_UPDS(TA_, TS_)                                                                                  \
    hipLaunchKernelGGL((update_kernel<TA_, double, 32, TS_>), grid, dim3(kT), 0, s, A, nb_a, M, ldm,          \
                       static_cast<void *>(Z), nb_z, n, m1, m2, S, nb_s)
    if (a64 && s64)
        CHEBFD_UPDS(double, double);
    else if (a64)
        CHEBFD_UPDS(double, float);
    else if (s64)
        CHEBFD_UPDS(float, double);
    else
        CHEBFD_UPDS(float, float);
#undef CHEBFD_UPDS
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

size_t jacobi_scratch_bytes(int m) {
    (void)m;
    // params [2][kMaxM/2] x (2 ints + 3 doubles), norm partials, sort scratch (2 kMaxM doubles)
    return round_up(2 * (kMaxM / 2) * (2 * sizeof(int) + 3 * sizeof(double)), 256) +
           round_up(kJNormG * sizeof(double), 256) + round_up(2 * kMaxM * sizeof(double), 256);
}

int launch_jacobi(int m, double *A, int lda, double *V, int ldv, double *w, int max_sweeps, double tol,
                  void *scratch, int *sweeps, int *converged, hipStream_t s) {
    if (m < 1 || m > kMaxM) CHEBFD_FAIL(CHEBFD_EINVAL, "eigensolver size %d not in [1, %d]", m, kMaxM);
    char *base = static_cast<char *>(scratch);
    const int H2 = 2 * (kMaxM / 2);
    JacobiRound jr;
    jr.p = reinterpret_cast<int *>(base);
    jr.q = jr.p + H2;
    jr.c = reinterpret_cast<double *>(base + round_up(2 * H2 * sizeof(int), 16));
    jr.sr = jr.c + H2;
    jr.si = jr.sr + H2;
    double *part = reinterpret_cast<double *>(base + round_up(2 * (kMaxM / 2) * (2 * sizeof(int) + 3 * sizeof(double)), 256));
    double *sortw = part + round_up(kJNormG * sizeof(double), 256) / sizeof(double);
    const int me = m + (m & 1), half = me / 2;
    if (m <= kJSmall) {
        const size_t lds = jacobi_small_lds(me);
        CHEBFD_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(jacobi_small_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(jacobi_small_lds(kJSmall))));
        const int items = half * half + half * me;   // 2 x 2 blocks of A and rotated pairs of V per round
        const int nt = std::max(128, std::min(1024, (items + 63) / 64 * 64));   // at least two waves
        int *d_status = jr.p, h_status[2];
        hipLaunchKernelGGL(jacobi_small_kernel, dim3(1), dim3(nt), lds, s, m, me, A, lda, V, ldv, w, max_sweeps, tol,
                           d_status);
        CHEBFD_HIP(hipGetLastError());
        CHEBFD_HIP(hipMemcpyAsync(h_status, d_status, sizeof(h_status), hipMemcpyDeviceToHost, s));
        CHEBFD_HIP(hipStreamSynchronize(s));
        *sweeps = h_status[0];
        *converged = h_status[1];
        return CHEBFD_OK;
    }
    const int G = std::min(kJNormG, std::max(1, (m * m + kJW - 1) / kJW));
    double hp[kJNormG];
    auto norm2 = [&](int off, double *out) -> int {
        hipLaunchKernelGGL(jacobi_norm_kernel, dim3(G), dim3(kJW), 0, s, m, A, lda, off, part);
        CHEBFD_HIP(hipGetLastError());
        CHEBFD_HIP(hipMemcpyAsync(hp, part, sizeof(double) * G, hipMemcpyDeviceToHost, s));
        CHEBFD_HIP(hipStreamSynchronize(s));
        double acc = 0.0;
        for (int g = 0; g < G; ++g) acc += hp[g];
        *out = acc;
        return CHEBFD_OK;
    };
    int rc;
    hipLaunchKernelGGL(jacobi_init_kernel, dim3(std::min(1024, (m * m + kJW - 1) / kJW)), dim3(kJW), 0, s, m, V,
                       ldv);
    CHEBFD_HIP(hipGetLastError());
    double fro2 = 0.0, off2 = 0.0;
    if ((rc = norm2(0, &fro2))) return rc;
    if ((rc = norm2(1, &off2))) return rc;
    *converged = off2 <= tol * tol * fro2 ? 1 : 0;
    int sweep = 0;
    for (; sweep < max_sweeps && !*converged; ++sweep) {
        for (int r = 0; r < me - 1; ++r) {
            hipLaunchKernelGGL(jacobi_round_kernel, dim3(half), dim3(kJW), 0, s, m, me, r, r > 0 ? 1 : 0, A, lda, V,
                               ldv, jr);
            CHEBFD_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(jacobi_rows_kernel, dim3(std::min(m, 256)), dim3(kJW), 0, s, m, me, (me - 2) & 1, A, lda,
                           jr);
        CHEBFD_HIP(hipGetLastError());
        if ((rc = norm2(1, &off2))) return rc;
        *converged = off2 <= tol * tol * fro2 ? 1 : 0;
    }
    *sweeps = sweep;
    hipLaunchKernelGGL(jacobi_sort_kernel, dim3(1), dim3(kJW), 0, s, m, A, lda, V, ldv, w, sortw);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

static int grid_cap(int64_t work, int cap = 8192) {
    int64_t g = (work + kT - 1) / kT;
    if (g > cap) g = cap;
    return static_cast<int>(g < 1 ? 1 : g);
}

int launch_svqb_scale(int m, double *S, int ld, double *d, hipStream_t s) {
    if (m > kMaxM) CHEBFD_FAIL(CHEBFD_EINVAL, "SVQB size %d > %d", m, kMaxM);
    hipLaunchKernelGGL(svqb_scale_kernel, dim3(1), dim3(kT), 0, s, m, S, ld, d);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_svqb_transform(int m, int k, int first, const double *d, const double *V, int ldv,
                          const double *w, double *T, int ldt, hipStream_t s) {
    hipLaunchKernelGGL(svqb_transform_kernel, dim3(grid_cap((int64_t)m * k)), dim3(kT), 0, s, m, k,
                       first, d, V, ldv, w, T, ldt);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_hermitise(int m, double *G, int ld, hipStream_t s) {
    hipLaunchKernelGGL(hermitise_kernel, dim3(grid_cap((int64_t)m * m)), dim3(kT), 0, s, m, G, ld);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int resid_grid(int64_t n) { return grid_cap(n, 1024); }

int launch_resid(const void *HZ, const void *Z, int prec, int64_t n, int nb, const double *theta,
                 double *part, int G, double *out, hipStream_t s) {
    hipLaunchKernelGGL(resid_partial_kernel, dim3(G), dim3(kT), 0, s, HZ, Z, prec, n, nb, theta, part);
    CHEBFD_HIP(hipGetLastError());
    hipLaunchKernelGGL(colsum_reduce_kernel, dim3(2 * nb), dim3(kT), 0, s, part, G, 2 * nb, out);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_permute_columns(int rows, int m, const double *S, int lds, const int *order, double *T,
                           int ldt, hipStream_t s) {
    hipLaunchKernelGGL(permute_columns_kernel, dim3(grid_cap((int64_t)rows * m)), dim3(kT), 0, s, rows, m, S,
                       lds, order, T, ldt);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_convert(const void *src, int prec_src, void *dst, int prec_dst, int64_t count,
                   hipStream_t s) {
    hipLaunchKernelGGL(convert_kernel, dim3(grid_cap(count, 65536)), dim3(kT), 0, s, src, prec_src, dst,
                       prec_dst, count);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_random_phase(void *X, int prec, int64_t n, int nb, int c_begin, int c_end, uint64_t seed,
                        uint64_t col0, const int32_t *perm, hipStream_t s) {
    if (c_end <= c_begin) return CHEBFD_OK;
    if (!pow2(nb)) CHEBFD_FAIL(CHEBFD_EINVAL, "block width %d must be a power of two", nb);
    hipLaunchKernelGGL(random_phase_kernel, dim3(grid_cap(n * (c_end - c_begin), 65536)), dim3(kT), 0, s,
                       X, prec, n, nb, c_begin, c_end, seed, col0, perm);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_fix_phases(void *Z, int prec, int64_t n, int nb, int m, double *phase, hipStream_t s) {
    if (!pow2(nb)) CHEBFD_FAIL(CHEBFD_EINVAL, "block width %d must be a power of two", nb);
    hipLaunchKernelGGL(phase_argmax_kernel, dim3(m < 1024 ? m : 1024), dim3(kT), 0, s, Z, prec, n, nb, m,
                       phase);
    CHEBFD_HIP(hipGetLastError());
    hipLaunchKernelGGL(scale_columns_kernel, dim3(grid_cap(n * m, 65536)), dim3(kT), 0, s, Z, prec, n, nb,
                       m, phase);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

}  // namespace chebfd
