// Fused Chebyshev step with the gathered block staged in LDS (gfx950).
//
// Same computation as the other step kernels (the recurrence step of Alg. 1 of
// the ChebFD paper, and its two start launches): per row i and block column j,
// W_ij <- 2 ((aH + bI) U)_ij - W_ij, the filtered-block update and the
// per-column dot products.
//
// The sparse product gathers whole row segments of U (NB complex numbers) at
// the matrix's column indices.  After a locality-preserving row order most of
// those columns lie close to the row, so one workgroup per CU sweeps a
// contiguous range of tiles and keeps a window of U in LDS: a ring of blocks of
// TR rows (TR = rows of one tile, 16 KB per block).  While tile t (rows
// [t TR, t TR + TR)) is processed the ring holds blocks t - h .. t + h
// (h = win_halo(TR): 3 tiles of 32 rows, 1 tile of 64) and receives the next
// block in the direction of the sweep, which is loaded from HBM once and read by
// the next 2 h + 1 tiles.  Gathers inside the window are LDS reads; columns
// outside it are gathered from global memory (L2, while the ranges of an XCD
// advance together).  W and Y are non-temporal streams; the matrix slots are
// staged in LDS per tile.
//
// What bounds it: memory.  A step has to move U, W in and out, the matrix, and
// every third step Y in and out; what it fetches beyond that are gathers that
// miss L2 (FP64 n_b = 32 on the 64x64x32 lattice: about 810 MB against 673 MB).
// To stay near the rate of a large copy (6 TB/s) a tile must not wait for its own
// loads:
//  - The gathers that leave the window are issued one tile ahead, into the
//    registers that the products read them from (their columns are known: the
//    slots arrive two tiles ahead, in three LDS buffers), and so are the W rows.
//    The gathers inside the window go to the registers of the same array, so the
//    products stay in slot order.
//  - Y rows (and the W rows of the c64 instance that reads both) are loaded when
//    the tile starts: held a tile longer they do not fit the 128 registers that
//    sixteen wavefronts leave each lane.
//  - The slots are resolved when they are deposited: an LDS offset, or the
//    complement of a column outside the window.
//  - The loops over the slots run to the row width, a scalar, also where every
//    chunk has kWinWidth of them: the branches keep the compiler from moving all
//    loads of a row to the front, which spills.
// us per step over a degree-30 filter, before (gathers, W and Y loaded by their
// own tile) and after; lattice, 4 orbitals:
//              rows      131072        524288        2097152
//   FP64 n_b = 32      68 -> 62     233 -> 216     928 -> 901
//   c64  n_b = 64      71 -> 66     233 -> 216     924 -> 896
//   c64  n_b = 32         -         128 -> 117     473 -> 452
//   FP64 n_b = 16         -         141 -> 118     574 -> 476 (LDS-staged kernel before, sweeps
//                                                              in one direction)
//
// Lanes: TR = 1024 * 16 / (bytes of a row) rows per tile; lane t works on the
// 16-byte vector t % LPR of row t / LPR of the tile.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "step_io.h"

namespace chebfd {
namespace {

using namespace step_io;

constexpr int kWinThreads = 1024;
constexpr int kXcdCount = 8;
constexpr int kWinLdsLimit = 160 * 1024;
// Lead control (see the kernel): every kWinCheckEvery tiles the first wave of a
// workgroup publishes its progress and reads that of the other workgroups of its
// XCD; more than kWinMaxLead tiles ahead of the slowest, it waits for it,
// polling at most kWinMaxPolls times.
constexpr int kWinCheckEvery = 32;
constexpr int kWinMaxLead = 4;
constexpr int kWinMaxPolls = 200;

template <typename T, int NB>
struct WinShape {
    static constexpr int CV = 8 / sizeof(T);           // complex numbers per 16-byte vector
    static constexpr int RB = NB * 2 * sizeof(T);      // bytes of one row of U
    static constexpr int LPR = RB / 16;                // lanes per row
    static constexpr int TR = kWinThreads / LPR;       // rows per tile (one per lane group)
    static constexpr int HALO = win_halo(TR);          // window: tiles t - HALO .. t + HALO
    static constexpr int BLOCKS = TR >= 64 ? 4 : 8;    // ring blocks: the window and the incoming block
    static constexpr int RING_ROWS = BLOCKS * TR;      // power of two
    static_assert(2 * HALO + 2 <= BLOCKS, "the window and the incoming block fit the ring");
    static constexpr int CPT = TR / 32;                // SELL chunks (C = 32) per tile
};

// Matrix slots of one tile in LDS: values, and for each slot the byte offset of its row of U in
// the ring or the complement of its column, if that lies outside the window.
template <typename T, int MAXW, int TR>
struct WinMatBuf {
    using VT = typename V2<T>::type;
    static constexpr int SLOTS = TR * MAXW;
    static constexpr int CPT = TR / 32;
    static constexpr int O_VALS = 0;
    static constexpr int O_OFFS = O_VALS + SLOTS * static_cast<int>(sizeof(VT));
    static constexpr int O_COFF = O_OFFS + 4 * SLOTS;
    static constexpr int O_CW = O_COFF + 4 * CPT;
    static constexpr int BYTES = (O_CW + 4 * CPT + 15) & ~15;
};
constexpr int kMatBufs = 3;   // tile t computes, tile t + 1 names its gathers, tile t + 2 arrives

template <typename T, int NB, int MAXW>
constexpr int win_lds_bytes() {
    using S = WinShape<T, NB>;
    return S::RING_ROWS * S::RB + kMatBufs * WinMatBuf<T, MAXW, S::TR>::BYTES;
}

template <typename T, int NB>
constexpr bool win_supported() {
    using S = WinShape<T, NB>;
    return S::TR >= 32 && S::TR % 32 == 0 && S::LPR >= 8 && S::LPR <= 32 &&
           win_lds_bytes<T, NB, kWinWidth>() <= kWinLdsLimit;
}

// partials of the previous launch (3 NB columns of G_prev values), fixed order
template <int NB>
__device__ void win_reduce_prev(const StepArgs &a, double *sred) {
    const int tid = threadIdx.x;
    for (int q = blockIdx.x; q < 3 * NB; q += gridDim.x) {
        const double *src = a.part_in + (int64_t)q * a.G_prev;
        double s = 0.0;
        for (int g = tid; g < a.G_prev; g += kWinThreads) s += src[g];
        sred[tid] = s;
        __syncthreads();
        for (int hh = kWinThreads / 2; hh > 0; hh >>= 1) {
            if (tid < hh) sred[tid] += sred[tid + hh];
            __syncthreads();
        }
        if (tid == 0) {
            const int comp = q / NB, jj = q % NB;
            if (comp < 2)
                a.red_eta[2 * jj + comp] = sred[0];
            else
                a.red_nu[jj] = sred[0];
        }
        __syncthreads();
    }
}

}  // namespace

// LDS layout (dynamic): ring[RING_ROWS][RB] | kMatBufs x WinMatBuf.
// The ring area also serves the reductions before the first and after the last tile.
template <typename T, int NB, int MODE, int MAXW, bool UNI>
__global__ __launch_bounds__(kWinThreads) void cheb_win_kernel(StepArgs a, int64_t ntiles) {
    using S = WinShape<T, NB>;
    using MB = WinMatBuf<T, MAXW, S::TR>;
    using VT = typename V2<T>::type;
    constexpr int CV = S::CV, LPR = S::LPR, TR = S::TR, RB = S::RB, CPT = S::CPT, HALO = S::HALO;
    constexpr int O_MAT = S::RING_ROWS * RB;
    using PK = Pack<T, CV>;
    // W rows one tile ahead, unless the registers do not suffice (with them 226 against 216 us
    // per step, c64 n_b = 64, 524288 rows)
    constexpr bool kAheadW = !(sizeof(T) == 4 && MODE == kModeStep);
    static_assert(win_supported<T, NB>(), "tile shape does not fit the window kernel");

    extern __shared__ __align__(16) unsigned char smem[];
    double *sred = reinterpret_cast<double *>(smem);
#define CHEBFD_WV(b) reinterpret_cast<VT *>(smem + O_MAT + (b) * MB::BYTES + MB::O_VALS)
#define CHEBFD_WO(b) reinterpret_cast<int32_t *>(smem + O_MAT + (b) * MB::BYTES + MB::O_OFFS)
#define CHEBFD_WCOFF(b) reinterpret_cast<int32_t *>(smem + O_MAT + (b) * MB::BYTES + MB::O_COFF)
#define CHEBFD_WCW(b) reinterpret_cast<int32_t *>(smem + O_MAT + (b) * MB::BYTES + MB::O_CW)

    const int tid = threadIdx.x, lane = tid & 63;
    const int rr = tid / LPR;                  // row within the tile
    const int lane_off = (tid % LPR) * 16;     // this lane's vector within a row

    if (a.part_in != nullptr) win_reduce_prev<NB>(a, sred);

    const char *const P = static_cast<const char *>(a.P);
    const char *const O = static_cast<const char *>(a.O);
    const char *const Y = static_cast<const char *>(a.Y);
    const VT *__restrict__ gval = static_cast<const VT *>(a.val);
    const int32_t *__restrict__ gcol = a.col;
    const T alpha = static_cast<T>(a.alpha), beta = static_cast<T>(a.beta);
    const T g0 = static_cast<T>(a.g0), g1 = static_cast<T>(a.g1), g2 = static_cast<T>(a.g2);
    // row and tile indices fit 32 bits (n < 2^31): scalar loop control stays in SGPRs
    const int n32 = static_cast<int>(a.n);
    const int nch = static_cast<int>(a.n_chunks);
    const int nblk = (n32 + TR - 1) / TR;

    double e_re[CV], e_im[CV], nu[CV];
#pragma unroll
    for (int c = 0; c < CV; ++c) e_re[c] = e_im[c] = nu[c] = 0.0;

    // contiguous tile range of this workgroup; each XCD sweeps one eighth
    const int G = gridDim.x, w = blockIdx.x;
    int tb, te;
    if (G % kXcdCount == 0) {
        const int x = w % kXcdCount, k = w / kXcdCount, per = G / kXcdCount;
        const int64_t xb = ntiles * x / kXcdCount, xe = ntiles * (x + 1) / kXcdCount;
        tb = static_cast<int>(xb + (xe - xb) * k / per);
        te = static_cast<int>(xb + (xe - xb) * (k + 1) / per);
    } else {
        tb = static_cast<int>(ntiles * w / G);
        te = static_cast<int>(ntiles * (w + 1) / G);
    }
    // sweep direction: tiles ts, ts + dir, ... of [tb, te)
    const int dir = a.reverse ? -1 : 1, ts = a.reverse ? te - 1 : tb;
    auto clamp_tile = [&](int tile) { return tile < tb ? tb : tile < te ? tile : te - 1; };
    // Rows of tile or block `blk` (uniform, inside the matrix) of a block vector: a
    // uniform base address and this lane's 32-bit offset, its row held to the matrix.
    auto block_base = [&](const char *x, int blk) { return x + (int64_t)blk * (TR * RB); };
    auto row_off = [&](int blk) {
        const int last = n32 - 1 - blk * TR;   // last row of the block that exists
        return static_cast<uint32_t>((rr < last ? rr : last) * RB + lane_off);
    };

    // matrix slots of one tile: registers, then LDS.  Threads past the slots repeat the
    // last one, so that the loads of all tiles are the same instructions and the
    // compiler can count them.
    constexpr int MQ = (MB::SLOTS + kWinThreads - 1) / kWinThreads;
    VT pv[MQ];
    int32_t pc[MQ];
    int64_t pf_s0 = 0;
    auto fetch_mat = [&](int tile) {
        const int c0 = tile * CPT, c1 = c0 + CPT < nch ? c0 + CPT : nch;
        int ns;
        if constexpr (UNI) {
            pf_s0 = (int64_t)c0 * 32 * MAXW;
            ns = (c1 - c0) * 32 * MAXW;
        } else {
            pf_s0 = a.chunk_off[c0];
            ns = static_cast<int>(a.chunk_off[c1] - pf_s0);
        }
        const VT *const gv = gval + pf_s0;
        const int32_t *const gc = gcol + pf_s0;
#pragma unroll
        for (int q = 0; q < MQ; ++q) {
            const int s = tid + q * kWinThreads;
            const uint32_t sl = s < ns ? s : (ns > 0 ? ns - 1 : 0);
            // non-temporal: each slot is read once, and keeping the slots out of L2
            // leaves room for the U rows that neighbouring workgroups gather a few
            // tiles after they were loaded (the gathers that leave the window)
            pv[q] = ld_nt(gv + sl);
            pc[q] = __builtin_nontemporal_load(gc + sl);
        }
    };
    auto deposit_mat = [&](int tile, int b) {
        const int wlo = (tile - HALO) * TR;   // window [wlo, wlo + (2 HALO + 1) TR)
#pragma unroll
        for (int q = 0; q < MQ; ++q) {
            const int s = tid + q * kWinThreads;
            if (s < MB::SLOTS) {
                const bool in = static_cast<unsigned>(pc[q] - wlo) < static_cast<unsigned>((2 * HALO + 1) * TR);
                CHEBFD_WV(b)[s] = pv[q];
                CHEBFD_WO(b)[s] = in ? (pc[q] & (S::RING_ROWS - 1)) * RB : ~pc[q];
            }
        }
        if constexpr (!UNI) {
            if (tid < CPT) {
                const int c = tile * CPT + tid;
                CHEBFD_WCOFF(b)[tid] = c < nch ? static_cast<int32_t>(a.chunk_off[c] - pf_s0) : 0;
                CHEBFD_WCW(b)[tid] = c < nch ? a.chunk_width[c] : 0;
            }
        }
    };
    // one block of U rows (blocks outside the matrix: its first or last one, never referenced)
    auto ring_load = [&](int blk, PK &x) {
        const int bc = blk < 0 ? 0 : blk < nblk ? blk : nblk - 1;
        const char *const base = block_base(P, bc);
        const uint32_t off = row_off(bc);
        x = load_pack<T, CV, false>(reinterpret_cast<const T *>(base + off));
    };
    auto ring_store = [&](int blk, const PK &x) {
        unsigned char *dst = smem + ((blk * TR + rr) & (S::RING_ROWS - 1)) * RB + lane_off;
        store_pack<T, CV>(reinterpret_cast<T *>(dst), x);
    };

    // What a tile finds in registers, loaded while the tile before it ran: its W row, its
    // resolved slots (LDS byte offset, or ~column outside the window) and the rows of U
    // outside the window, in the array that the products read.
    PK o, yv, u[MAXW];
    int so[MAXW];
    int base = 0, wdt = UNI ? a.uniform_width : 0;   // first slot and width of the row
#pragma unroll
    for (int c = 0; c < CV; ++c) o.re[c] = o.im[c] = yv.re[c] = yv.im[c] = T(0);
    auto load_row = [&](const char *x, int tile) {
        return load_pack<T, CV, true>(reinterpret_cast<const T *>(block_base(x, tile) + row_off(tile)));
    };
    auto issue_ahead = [&](int tile, int b) {
        const int cl = rr >> 5;
        if constexpr (UNI) {
            base = cl * 32 * MAXW + (rr & 31);
        } else {
            // the rows of a wavefront lie in one chunk
            base = CHEBFD_WCOFF(b)[cl] + (rr & 31);
            wdt = __builtin_amdgcn_readfirstlane(CHEBFD_WCW(b)[cl]);
        }
#pragma unroll
        for (int k = 0; k < MAXW; ++k) so[k] = k < wdt ? CHEBFD_WO(b)[base + k * 32] : 0;
#pragma unroll
        for (int k = 0; k < MAXW; ++k)
            if (so[k] < 0) {
                const char *const row = P + ((int64_t)~so[k] * RB + lane_off);
                u[k] = load_pack<T, CV, false>(reinterpret_cast<const T *>(row));
            }
        if constexpr (!mode_first(MODE) && kAheadW) o = load_row(O, tile);
    };

    // (the reduction above ends with a barrier: the ring area is free)
    int buf = 0;                               // matrix buffer of the current tile
    if (tb < te) {
        // prologue: the window of the first tile, the matrix slots of the first two
        PK pro[2 * HALO + 1];
#pragma unroll
        for (int q = 0; q < 2 * HALO + 1; ++q) ring_load(ts - HALO + q, pro[q]);
        fetch_mat(ts);
#pragma unroll
        for (int q = 0; q < 2 * HALO + 1; ++q) ring_store(ts - HALO + q, pro[q]);
        deposit_mat(ts, 0);
        fetch_mat(clamp_tile(ts + dir));
        deposit_mat(clamp_tile(ts + dir), 1);
        __syncthreads();
        issue_ahead(ts, 0);
    }

    // One tile.  FULL: every row of the tile exists (all tiles but a ragged last one).
    auto tile_body = [&](int tile, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        const bool live = FULL || tile * TR + rr < n32;
        const int b1 = buf + 1 < kMatBufs ? buf + 1 : 0, b2 = b1 + 1 < kMatBufs ? b1 + 1 : 0;
        const VT *sv = CHEBFD_WV(buf);
        // the block entering the window and the matrix slots of the tile after the next
        const int blk_in = tile + dir * (HALO + 1);
        PK rf;
        ring_load(blk_in, rf);
        fetch_mat(clamp_tile(tile + 2 * dir));

        if constexpr (MODE == kModeStep) yv = load_row(Y, tile);
        if constexpr (!mode_first(MODE) && !kAheadW) o = load_row(O, tile);
        auto lds_vec = [&](int off) {
            return load_pack<T, CV, false>(reinterpret_cast<const T *>(smem + off + lane_off));
        };
        const PK up = lds_vec(((tile * TR + rr) & (S::RING_ROWS - 1)) * RB);
#pragma unroll
        for (int k = 0; k < MAXW; ++k)
            if (so[k] >= 0) u[k] = lds_vec(so[k]);
        T acc_re[CV], acc_im[CV];
#pragma unroll
        for (int c = 0; c < CV; ++c) acc_re[c] = acc_im[c] = T(0);
#pragma unroll
        for (int k = 0; k < MAXW; ++k) {
            if (k >= wdt) break;
            const VT h = sv[base + k * 32];
#pragma unroll
            for (int c = 0; c < CV; ++c) {
                acc_re[c] = fma(h.x, u[k].re[c], acc_re[c]);
                acc_re[c] = fma(-h.y, u[k].im[c], acc_re[c]);
                acc_im[c] = fma(h.x, u[k].im[c], acc_im[c]);
                acc_im[c] = fma(h.y, u[k].re[c], acc_im[c]);
            }
        }
        PK nw, yo;
#pragma unroll
        for (int c = 0; c < CV; ++c) {
            const T hu_re = fma(alpha, acc_re[c], beta * up.re[c]);
            const T hu_im = fma(alpha, acc_im[c], beta * up.im[c]);
            if constexpr (mode_first(MODE)) {
                nw.re[c] = hu_re;
                nw.im[c] = hu_im;
            } else {
                nw.re[c] = fma(T(2), hu_re, -o.re[c]);
                nw.im[c] = fma(T(2), hu_im, -o.im[c]);
            }
            if constexpr (MODE == kModeSecond) {
                yo.re[c] = fma(g0, o.re[c], fma(g1, up.re[c], g2 * nw.re[c]));
                yo.im[c] = fma(g0, o.im[c], fma(g1, up.im[c], g2 * nw.im[c]));
            } else if constexpr (MODE == kModeStep) {
                yo.re[c] = add_terms(a.y_terms, g0, o.re[c], g1, up.re[c], g2, nw.re[c], yv.re[c]);
                yo.im[c] = add_terms(a.y_terms, g0, o.im[c], g1, up.im[c], g2, nw.im[c], yv.im[c]);
            }
        }
        if (mode_dots(MODE) && live) {
#pragma unroll
            for (int c = 0; c < CV; ++c) {
                const double nr = nw.re[c], ni = nw.im[c], ur = up.re[c], ui = up.im[c];
                e_re[c] = fma(nr, ur, fma(ni, ui, e_re[c]));
                e_im[c] = fma(nr, ui, fma(-ni, ur, e_im[c]));
                nu[c] = fma(ur, ur, fma(ui, ui, nu[c]));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // the next tile's loads (its matrix slots were deposited one tile ago); the last
        // tile of the range repeats its own
        const int next = clamp_tile(tile + dir);
        issue_ahead(next, next != tile ? b1 : buf);
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
            auto out = [&](void *x) {
                return reinterpret_cast<T *>(static_cast<char *>(x) + (int64_t)tile * (TR * RB) + (rr * RB + lane_off));
            };
            store_pack_nt<T, CV>(out(mode_first(MODE) || MODE == kModeSecond ? a.N : a.O), nw);
            // Second: Y aliases O, whose row is read only here (one tile ago)
            if constexpr (MODE == kModeSecond || MODE == kModeStep) store_pack_nt<T, CV>(out(a.Y), yo);
        }
        // the block entering the window replaces one that has left it (the ring holds at least
        // 2 HALO + 2 blocks); the matrix slots go to the buffer that the tile before this one
        // used.  The stores stay in flight across the barrier (it orders LDS only; no other
        // row reads this row's W or Y).
        ring_store(blk_in, rf);
        deposit_mat(clamp_tile(tile + 2 * dir), b2);
        __syncthreads();
        buf = b1;
    };
    // Lead control between the sweep ranges of one XCD.  The row order deals
    // neighbouring pencils of the lattice to the ranges of one XCD at equal
    // offsets, so the gathers that leave the window read rows that another
    // range has just loaded into the shared L2 -- as long as the ranges advance
    // together; left alone they drift apart by far more than the few tiles the
    // L2 holds.  Every kWinCheckEvery tiles the first wave publishes
    // (launch tag, tiles done) in prog[x per + k] (workgroup w = x + 8 k on XCD
    // x) and, while the workgroup is more than kWinMaxLead tiles ahead of the
    // slowest range of its XCD that has started this launch, polls again (a
    // bounded wait: it only costs time).  Only the first wave touches the
    // counters (a wave-uniform branch); the others wait at the tile's barrier.
    const int per = G / kXcdCount;
    const bool lead = a.prog != nullptr && G % kXcdCount == 0 && per <= 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t *const my_prog = lead ? a.prog + (w % kXcdCount) * per + w / kXcdCount : nullptr;
    const int64_t *const xcd_prog = lead ? a.prog + (w % kXcdCount) * per : nullptr;
    const int64_t tag = static_cast<int64_t>(a.epoch) << 32;
    auto check = [&](int done) {
        __hip_atomic_store(my_prog, tag | static_cast<uint32_t>(done), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int k = (tid & 63) % per;
        for (int poll = 0; poll < kWinMaxPolls; ++poll) {
            const int64_t v = __hip_atomic_load(xcd_prog + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // a range that has not started this launch (older tag) holds no one back
            int d = static_cast<int32_t>(v >> 32) == a.epoch ? static_cast<int>(v & 0xffffffff) : INT_MAX;
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) d = min(d, __shfl_xor(d, m));
            if (done - d <= kWinMaxLead) break;
            __builtin_amdgcn_s_sleep(16);
        }
    };

    // full tiles, and the ragged last tile of the matrix (if it is in this range) after or before them
    const int te_full = te < n32 / TR ? te : (n32 / TR > tb ? n32 / TR : tb);
    if (dir < 0)
        for (int tile = te - 1; tile >= te_full; --tile) tile_body(tile, std::false_type{});
    const int full = te_full - tb;
    int tile = dir > 0 ? tb : te_full - 1;
    for (int k = 0; k < full; ++k, tile += dir) {
        if (lead && wave == 0 && k % kWinCheckEvery == 0) check(k);
        tile_body(tile, std::true_type{});
    }
    if (dir > 0)
        for (; tile < te; ++tile) tile_body(tile, std::false_type{});
    if (lead && wave == 0)
        __hip_atomic_store(my_prog, tag | static_cast<uint32_t>(te - tb), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    if constexpr (!mode_dots(MODE)) return;
    if (a.part_out == nullptr) return;
    // sums of a column: over the rows of a wavefront by lane exchanges, then over the
    // wavefronts through LDS (over the ring: every wave has passed the last barrier)
#pragma unroll
    for (int c = 0; c < CV; ++c) {
#pragma unroll
        for (int m = LPR; m < 64; m <<= 1) {
            e_re[c] += __shfl_xor(e_re[c], m);
            e_im[c] += __shfl_xor(e_im[c], m);
            nu[c] += __shfl_xor(nu[c], m);
        }
        if (lane < LPR) {
            double *const sw = sred + (tid >> 6) * (3 * NB) + lane * CV + c;
            sw[0] = e_re[c];
            sw[NB] = e_im[c];
            sw[2 * NB] = nu[c];
        }
    }
    __syncthreads();
    for (int q = tid; q < 3 * NB; q += kWinThreads) {
        double s = 0.0;
#pragma unroll
        for (int x = 0; x < kWinThreads / 64; ++x) s += sred[x * (3 * NB) + q];
        a.part_out[(int64_t)q * G + w] = s;
    }
}
#undef CHEBFD_WV
#undef CHEBFD_WO
#undef CHEBFD_WCOFF
#undef CHEBFD_WCW

namespace {

template <typename T, int NB, int MODE, int MAXW, bool UNI>
int launch_win_one(const StepArgs &a, const WinGeometry &g, hipStream_t s) {
    constexpr int lds = win_lds_bytes<T, NB, MAXW>();
    hipLaunchKernelGGL((cheb_win_kernel<T, NB, MODE, MAXW, UNI>), dim3(g.G), dim3(kWinThreads), lds, s, a, g.ntiles);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

template <typename T, int NB, int MAXW, bool UNI>
int launch_win_mode(int mode, const StepArgs &a, const WinGeometry &g, hipStream_t s) {
    switch (mode) {
        case kModeFirst: return launch_win_one<T, NB, kModeFirst, MAXW, UNI>(a, g, s);
        case kModeSecond: return launch_win_one<T, NB, kModeSecond, MAXW, UNI>(a, g, s);
        case kModeStep: return launch_win_one<T, NB, kModeStep, MAXW, UNI>(a, g, s);
        case kModeKpm: return launch_win_one<T, NB, kModeKpm, MAXW, UNI>(a, g, s);
        case kModeSpmv: return launch_win_one<T, NB, kModeSpmv, MAXW, UNI>(a, g, s);
        case kModeSpmvRec: return launch_win_one<T, NB, kModeSpmvRec, MAXW, UNI>(a, g, s);
    }
    CHEBFD_FAIL(CHEBFD_EINVAL, "bad step mode %d", mode);
}

template <typename T, int NB>
int launch_win_w(int mode, const StepArgs &a, const WinGeometry &g, hipStream_t s) {
    if (g.uniform) return launch_win_mode<T, NB, kWinWidth, true>(mode, a, g, s);
    return launch_win_mode<T, NB, kWinWidth, false>(mode, a, g, s);
}

template <typename T, int NB, int MAXW, bool UNI>
bool set_win_attr() {
    const int bytes = win_lds_bytes<T, NB, MAXW>();
    bool ok = true;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeFirst, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeSecond, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeStep, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeKpm, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeSpmv, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    ok &= hipFuncSetAttribute(reinterpret_cast<const void *>(cheb_win_kernel<T, NB, kModeSpmvRec, MAXW, UNI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    return ok;
}

}  // namespace

bool win_geometry(const chebfd_matrix *H, int prec, int nb, int num_cus, WinGeometry *g) {
    if (H->C != 32 || H->max_width > kWinWidth) return false;
    int tr;
    // instances where the window beats the kernels that would take the matrix otherwise
    // (measured): FP64 n_b = 32, c64 n_b = 64, and rows of 256 bytes (FP64 n_b = 16 and
    // c64 n_b = 32) from 32 tiles of 64 rows per CU, 524288 rows.  us per step of a
    // degree-30 filter with moments, other kernel against window:
    //          rows      131072    262144    294912    393216     524288    1048576
    //   FP64 n_b = 16   31 | 37   59 | 62   77 | 71  102 | 91  136 | 110  277 | 227
    //   c64  n_b = 32   30 | 37   54 | 61   76 | 71   98 | 89  131 | 109  265 | 220
    // The times cross where U, W and Y leave the memory-side cache and the small-matrix
    // kernel ends (210 MB, 273 thousand rows); the line lies above that.
    if (prec == CHEBFD_PREC_FP64 && nb == 32)
        tr = WinShape<double, 32>::TR;
    else if (prec == CHEBFD_PREC_MIXED && nb == 64)
        tr = WinShape<float, 64>::TR;
    else if (prec == CHEBFD_PREC_MIXED && nb == 32 && H->n >= (int64_t)kWinNarrowTiles * num_cus * 64)
        tr = WinShape<float, 32>::TR;
    else if (prec == CHEBFD_PREC_FP64 && nb == 16 && H->n >= (int64_t)kWinNarrowTiles * num_cus * 64)
        tr = WinShape<double, 16>::TR;
    else
        return false;
    const int local = H->window_local[tr == 32 ? 0 : 1];
    if (local < kWinMinLocal) return false;
    g->tr = tr;
    // every chunk exactly kWinWidth slots wide (lattice Hamiltonians of 4 orbitals): no chunk tables
    g->uniform = H->uniform_width == kWinWidth ? 1 : 0;
    g->ntiles = (H->n + tr - 1) / tr;
    // one workgroup per CU, at least two tiles each (the window needs a sweep to pay off)
    int64_t G = num_cus;
    while (G > kXcdCount && g->ntiles < 2 * G) G /= 2;
    if (g->ntiles < 2 * G) return false;
    static bool attr_ok =
        set_win_attr<double, 32, kWinWidth, true>() && set_win_attr<double, 32, kWinWidth, false>() &&
        set_win_attr<float, 64, kWinWidth, true>() && set_win_attr<float, 64, kWinWidth, false>() &&
        set_win_attr<float, 32, kWinWidth, true>() && set_win_attr<float, 32, kWinWidth, false>() &&
        set_win_attr<double, 16, kWinWidth, true>() && set_win_attr<double, 16, kWinWidth, false>();
    if (!attr_ok) return false;
    g->G = static_cast<int>(G);
    return true;
}

int launch_win_step(int prec, int nb, int mode, const StepArgs &a, const WinGeometry &g, hipStream_t s) {
    if (prec == CHEBFD_PREC_FP64 && nb == 32) return launch_win_w<double, 32>(mode, a, g, s);
    if (prec == CHEBFD_PREC_MIXED && nb == 64) return launch_win_w<float, 64>(mode, a, g, s);
    if (prec == CHEBFD_PREC_MIXED && nb == 32) return launch_win_w<float, 32>(mode, a, g, s);
    if (prec == CHEBFD_PREC_FP64 && nb == 16) return launch_win_w<double, 16>(mode, a, g, s);
    CHEBFD_FAIL(CHEBFD_EINVAL, "window kernel has no instance for prec %d, n_b = %d", prec, nb);
}

}  // namespace chebfd
