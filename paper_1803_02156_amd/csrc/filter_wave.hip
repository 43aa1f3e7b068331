// Fused Chebyshev step for small matrices (gfx950).
//
// Same computation as the other step kernels (the recurrence step of Alg. 1 of
// the ChebFD paper, and its two start launches), with the same fused
// multiply-adds per entry in the same order as the LDS-staged kernel.
//
// A step on a small matrix is bound by its chain of dependent memory accesses
// (slots, gathers, sums), by the address unit (17 accesses of 16 bytes per lane)
// and by the launch itself (about 1.7 us between dependent launches), not by HBM:
// the blocks stay in the 256 MB memory-side cache.  The LDS-staged kernel gives a
// workgroup a tile of at least 32 rows, which it steps in several passes one
// after the other behind a workgroup-wide staging of the tile's slots, sums the
// previous launch's partials before its own rows, and leaves a 16x16x8 lattice
// (8192 rows) with one workgroup per CU.  Here
//  * a workgroup takes 256 / (lanes per row) rows, one pass where the grid allows,
//    and every wavefront stages the slots of its own rows in LDS, without a
//    workgroup barrier (with one lane per row it reads them directly);
//  * the previous launch's sums are formed by extra workgroups beside the steps;
//  * a column's sum over a wavefront's rows goes through lane exchanges;
//  * W and Y use plain loads and stores (the next launch reads them from cache);
//  * one launch steps several blocks of the search space (blockIdx.y) while a
//    single one does not fill the device.
// Per step, LDS-staged -> this kernel (FP64, with moments): 2048 rows n_b = 1
// 10.5 -> 4.7 us, n_b = 128 24.6 -> 8.5; 8192 rows n_b = 16 7.7 -> 5.8, n_b = 32
// 9.2 -> 8.6 (two blocks per launch: 5.3 per block); 36864 rows n_b = 32
// 23.4 -> 19.5; 131072 rows n_b = 32 73.8 -> 64.0; c64, 131072 rows n_b = 64
// 74 -> 61.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "common.h"
#include "kernels.h"
#include "step_io.h"

namespace chebfd {
namespace {

using namespace step_io;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kXcds = 8;

template <typename T, int NB>
struct WaveShape {
    static constexpr int CPL = cols_per_lane<T, NB>();
    static constexpr int LPR = NB / CPL;                    // lanes per row
    static constexpr int LPW = LPR < 64 ? LPR : 64;         // of them in one wavefront
    static constexpr int RPW = 64 / LPW;                    // rows per wavefront
    static constexpr int WPR = LPR / LPW;                   // wavefronts per row (1 or 2)
    static constexpr int ROWS = kThreads / LPR;             // rows per workgroup pass
    static constexpr bool STAGED = RPW < 64;                // one lane per row reads its own slots
};

// The partial sums of a launch are stored workgroup by workgroup, part[w][3 NB]
// (one contiguous run per workgroup).  They are summed by workgroups of their
// own, kRedCols columns each, that come first in the next launch's grid and run
// beside its steps; their number is a multiple of 8, which keeps the step
// workgroups' XCD mapping.
constexpr int kRedCols = 4;
constexpr int reduce_wgs(int nb) { return (3 * nb + kRedCols * kXcds - 1) / (kRedCols * kXcds) * kXcds; }

// columns [kRedCols blockIdx.x, ...) of batch entry blockIdx.y, fixed order
template <int NB>
__device__ void reduce_prev(const StepArgs &a, double *sred) {
    constexpr int LANES = kThreads / kRedCols;   // workgroups summed side by side
    constexpr int UNR = 8;
    const int tid = threadIdx.x;
    const int q = blockIdx.x * kRedCols + tid % kRedCols;
    if (blockIdx.x * kRedCols >= 3 * NB) return;
    double t = 0.0;
    if (q < 3 * NB) {
        const double *src = a.part_in + (int64_t)blockIdx.y * 3 * NB * a.G_prev + q;
        double s[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) s[u] = 0.0;
        int g = tid / kRedCols;
        for (; g + (UNR - 1) * LANES < a.G_prev; g += UNR * LANES) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) s[u] += src[(int64_t)(g + u * LANES) * (3 * NB)];
        }
        for (; g < a.G_prev; g += LANES) s[0] += src[(int64_t)g * (3 * NB)];
        t = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
#pragma unroll
    for (int m = kRedCols; m < 64; m <<= 1) t += __shfl_xor(t, m);
    if ((tid & 63) < kRedCols) sred[(tid >> 6) * kRedCols + tid % kRedCols] = t;
    __syncthreads();
    if (tid < kRedCols && q < 3 * NB) {
        double r = 0.0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) r += sred[v * kRedCols + tid];
        const int comp = q / NB, jj = q % NB + blockIdx.y * NB;
        if (comp < 2)
            a.red_eta[2 * jj + comp] = r;
        else
            a.red_nu[jj] = r;
    }
}

}  // namespace

template <typename T, int NB, int MODE, int MAXW>
__global__ __launch_bounds__(kThreads) void cheb_wave_kernel(StepArgs a, int red) {
    using S = WaveShape<T, NB>;
    using VT = typename V2<T>::type;
    constexpr int CPL = S::CPL, LPR = S::LPR, LPW = S::LPW, RPW = S::RPW, WPR = S::WPR, ROWS = S::ROWS;
    using PK = Pack<T, CPL>;
    constexpr int SLOTS = S::STAGED ? RPW * MAXW : 1;       // matrix slots of a wavefront's rows
    constexpr int KSTEP = 64 / RPW;                         // slots per row that one staging load covers
    constexpr int NS = (MAXW + KSTEP - 1) / KSTEP;          // staging loads per lane
    __shared__ VT sval[kWaves][SLOTS];
    __shared__ int32_t scol[kWaves][SLOTS];
    __shared__ double sred[3 * CPL * kThreads];

    if (static_cast<int>(blockIdx.x) < red) {
        reduce_prev<NB>(a, sred);
        return;
    }
    // this block of the batch: the first at P, O, N, Y, the others one after another
    // from P1, O1, N1, Y1 on
    const int64_t bofs = ((int64_t)blockIdx.y - 1) * a.n * NB * 2;
    auto block = [&](const void *first, const void *rest) {
        return blockIdx.y == 0 ? static_cast<const T *>(first) : static_cast<const T *>(rest) + bofs;
    };
    const int w = blockIdx.x - red, G = gridDim.x - red;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rr = lane / LPW;                              // row within the wavefront
    const int jc = ((wv % WPR) * LPW + lane % LPW) * CPL;   // first column of this lane

    const T *__restrict__ P = block(a.P, a.P1);
    T *const O = const_cast<T *>(block(a.O, a.O1));
    T *const N = const_cast<T *>(block(a.N, a.N1));
    T *const Y = const_cast<T *>(block(a.Y, a.Y1));   // Second: the same block as O
    const VT *__restrict__ gval = static_cast<const VT *>(a.val);
    const int32_t *__restrict__ gcol = a.col;
    const T alpha = static_cast<T>(a.alpha), beta = static_cast<T>(a.beta);
    const T g0 = static_cast<T>(a.g0), g1 = static_cast<T>(a.g1), g2 = static_cast<T>(a.g2);

    double e_re[CPL], e_im[CPL], nu[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) e_re[c] = e_im[c] = nu[c] = 0.0;

    // each XCD takes one contiguous eighth of the passes
    int64_t begin, end, stride;
    if (G % kXcds == 0 && a.npass >= G) {
        const int x = w % kXcds, k = w / kXcds;
        begin = a.npass * x / kXcds + k;
        end = a.npass * (x + 1) / kXcds;
        stride = G / kXcds;
    } else {
        begin = w;
        end = a.npass;
        stride = G;
    }
    // slots per row that are loaded at all: max over rows when chunks differ
    const int uw = a.uniform_width;
    auto locate = [&](int64_t row, int64_t &off, int &wdt) {
        const int64_t c = row >> a.log2C;
        const int r = static_cast<int>(row & (a.C - 1));
        if (uw > 0) {
            wdt = uw;
            off = c * a.C * uw + r;
        } else {
            wdt = a.chunk_width[c];
            off = a.chunk_off[c] + r;
        }
    };

    for (int64_t pass = begin; pass < end; pass += stride) {
        const int64_t row0 = pass * ROWS + (wv / WPR) * RPW;    // first row of this wavefront
        const int64_t i = row0 + rr;
        const bool live = i < a.n;
        const int64_t e = 2 * (i * NB + jc);
        // the rows' matrix slots: a coalesced load per KSTEP slots of the
        // wavefront's rows (slots past a row's width: the row itself, coefficient 0)
        VT h[MAXW];
        int32_t cc[MAXW];
        const int64_t srow = S::STAGED ? row0 + lane % RPW : i;
        const bool shave = srow < a.n;
        int64_t off = 0;
        int wdt = 0;
        if (shave) locate(srow, off, wdt);
        if constexpr (S::STAGED) {
            VT pv[NS];
            int32_t pc[NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int k = lane / RPW + q * KSTEP;
                pv[q] = VT{T(0), T(0)};
                pc[q] = static_cast<int32_t>(shave ? srow : 0);
                if (shave && k < wdt) {
                    pv[q] = gval[off + (int64_t)k * a.C];
                    pc[q] = gcol[off + (int64_t)k * a.C];
                }
            }
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int k = lane / RPW + q * KSTEP;
                if (k < MAXW) {
                    sval[wv][k * RPW + lane % RPW] = pv[q];
                    scol[wv][k * RPW + lane % RPW] = pc[q];
                }
            }
            // written and read by the same wavefront, whose LDS accesses complete in order
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < MAXW; ++k) cc[k] = scol[wv][k * RPW + rr];
        } else {
#pragma unroll
            for (int k = 0; k < MAXW; ++k) {
                h[k] = VT{T(0), T(0)};
                cc[k] = static_cast<int32_t>(live ? i : 0);
                if (live && k < wdt) {
                    h[k] = gval[off + (int64_t)k * a.C];
                    cc[k] = gcol[off + (int64_t)k * a.C];
                }
            }
        }
        if (live) {
            PK u[MAXW];
#pragma unroll
            for (int k = 0; k < MAXW; ++k) u[k] = load_pack<T, CPL, false>(P + 2 * ((int64_t)cc[k] * NB + jc));
            const PK up = load_pack<T, CPL, false>(P + e);
            PK o, yv;
#pragma unroll
            for (int c = 0; c < CPL; ++c) o.re[c] = o.im[c] = yv.re[c] = yv.im[c] = T(0);
            if constexpr (!mode_first(MODE)) o = load_pack<T, CPL, false>(O + e);
            if constexpr (MODE == kModeStep) yv = load_pack<T, CPL, false>(Y + e);
            if constexpr (S::STAGED) {
#pragma unroll
                for (int k = 0; k < MAXW; ++k) h[k] = sval[wv][k * RPW + rr];
            }
            T acc_re[CPL], acc_im[CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc_re[c] = acc_im[c] = T(0);
#pragma unroll
            for (int k = 0; k < MAXW; ++k) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    acc_re[c] = fma(h[k].x, u[k].re[c], acc_re[c]);
                    acc_re[c] = fma(-h[k].y, u[k].im[c], acc_re[c]);
                    acc_im[c] = fma(h[k].x, u[k].im[c], acc_im[c]);
                    acc_im[c] = fma(h[k].y, u[k].re[c], acc_im[c]);
                }
            }
            PK nw;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const T hu_re = fma(alpha, acc_re[c], beta * up.re[c]);
                const T hu_im = fma(alpha, acc_im[c], beta * up.im[c]);
                if constexpr (mode_first(MODE)) {
                    nw.re[c] = hu_re;
                    nw.im[c] = hu_im;
                } else {
                    nw.re[c] = fma(T(2), hu_re, -o.re[c]);
                    nw.im[c] = fma(T(2), hu_im, -o.im[c]);
                }
            }
            if constexpr (mode_first(MODE) || MODE == kModeSecond)
                store_pack<T, CPL>(N + e, nw);
            else
                store_pack<T, CPL>(O + e, nw);
            if constexpr (MODE == kModeSecond || MODE == kModeStep) {
                PK y;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    if constexpr (MODE == kModeSecond) {
                        y.re[c] = fma(g0, o.re[c], fma(g1, up.re[c], g2 * nw.re[c]));
                        y.im[c] = fma(g0, o.im[c], fma(g1, up.im[c], g2 * nw.im[c]));
                    } else {
                        y.re[c] = add_terms(a.y_terms, g0, o.re[c], g1, up.re[c], g2, nw.re[c], yv.re[c]);
                        y.im[c] = add_terms(a.y_terms, g0, o.im[c], g1, up.im[c], g2, nw.im[c], yv.im[c]);
                    }
                }
                store_pack<T, CPL>(Y + e, y);   // Second: Y aliases O, read only here
            }
            if constexpr (mode_dots(MODE)) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const double nr = nw.re[c], ni = nw.im[c], ur = up.re[c], ui = up.im[c];
                    e_re[c] = fma(nr, ur, fma(ni, ui, e_re[c]));
                    e_im[c] = fma(nr, ui, fma(-ni, ur, e_im[c]));
                    nu[c] = fma(ur, ur, fma(ui, ui, nu[c]));
                }
            }
        }
    }

    if constexpr (!mode_dots(MODE)) return;
    if (a.part_out == nullptr) return;
    // sums of a column: over the rows of a wavefront by lane exchanges, then over
    // the wavefronts through LDS, fixed order
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
#pragma unroll
        for (int m = LPW; m < 64; m <<= 1) {
            e_re[c] += __shfl_xor(e_re[c], m);
            e_im[c] += __shfl_xor(e_im[c], m);
            nu[c] += __shfl_xor(nu[c], m);
        }
        if (lane < LPW) {
            sred[(0 * CPL + c) * kThreads + tid] = e_re[c];
            sred[(1 * CPL + c) * kThreads + tid] = e_im[c];
            sred[(2 * CPL + c) * kThreads + tid] = nu[c];
        }
    }
    __syncthreads();
    double *part = a.part_out + ((int64_t)blockIdx.y * G + w) * (3 * NB);
    for (int q = tid; q < 3 * NB; q += kThreads) {
        const int comp = q / NB, col = q % NB, l = col / CPL, c = col % CPL;
        double s = 0.0;
#pragma unroll
        for (int v = l / LPW; v < kWaves; v += WPR) s += sred[(comp * CPL + c) * kThreads + v * 64 + l % LPW];
        part[q] = s;
    }
}

// the sums of the last launch (no step follows)
template <int NB>
__global__ __launch_bounds__(kThreads) void cheb_wave_reduce_kernel(StepArgs a) {
    __shared__ double sred[kWaves * kRedCols];
    reduce_prev<NB>(a, sred);
}

namespace {

template <typename T, int NB, int MODE, int MAXW>
int launch_wave_one(const StepArgs &a, const WaveGeometry &g, hipStream_t s) {
    const int red = mode_dots(MODE) && a.part_in != nullptr ? reduce_wgs(NB) : 0;
    hipLaunchKernelGGL((cheb_wave_kernel<T, NB, MODE, MAXW>), dim3(g.G + red, a.batch), dim3(kThreads), 0, s, a, red);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

template <typename T, int NB, int MAXW>
int launch_wave_mode(int mode, const StepArgs &a, const WaveGeometry &g, hipStream_t s) {
    switch (mode) {
        case kModeFirst: return launch_wave_one<T, NB, kModeFirst, MAXW>(a, g, s);
        case kModeSecond: return launch_wave_one<T, NB, kModeSecond, MAXW>(a, g, s);
        case kModeStep: return launch_wave_one<T, NB, kModeStep, MAXW>(a, g, s);
        case kModeKpm: return launch_wave_one<T, NB, kModeKpm, MAXW>(a, g, s);
        case kModeSpmv: return launch_wave_one<T, NB, kModeSpmv, MAXW>(a, g, s);
        case kModeSpmvRec: return launch_wave_one<T, NB, kModeSpmvRec, MAXW>(a, g, s);
    }
    CHEBFD_FAIL(CHEBFD_EINVAL, "bad step mode %d", mode);
}

template <typename T, int NB>
int launch_wave_w(int mode, const StepArgs &a, const WaveGeometry &g, hipStream_t s) {
    if (g.maxw == 13) return launch_wave_mode<T, NB, 13>(mode, a, g, s);
    return launch_wave_mode<T, NB, kWaveMaxWidth>(mode, a, g, s);
}

template <typename T>
int launch_wave_nb(int nb, int mode, const StepArgs &a, const WaveGeometry &g, hipStream_t s) {
    switch (nb) {
        case 1: return launch_wave_w<T, 1>(mode, a, g, s);
        case 2: return launch_wave_w<T, 2>(mode, a, g, s);
        case 4: return launch_wave_w<T, 4>(mode, a, g, s);
        case 8: return launch_wave_w<T, 8>(mode, a, g, s);
        case 16: return launch_wave_w<T, 16>(mode, a, g, s);
        case 32: return launch_wave_w<T, 32>(mode, a, g, s);
        case 64: return launch_wave_w<T, 64>(mode, a, g, s);
        case 128: return launch_wave_w<T, 128>(mode, a, g, s);
    }
    CHEBFD_FAIL(CHEBFD_EINVAL, "n_b = %d not supported", nb);
}

}  // namespace

bool wave_geometry(const chebfd_matrix *H, int prec, int nb, WaveGeometry *g) {
    if (H->max_width > kWaveMaxWidth || H->C > 32) return false;   // the LDS-staged kernel's shapes
    const int64_t block = (int64_t)vec_elem_bytes(prec) * H->n * nb;
    if (nb > 1 && 3 * block > kWaveMaxBytes) return false;
    const int cpl = (prec == CHEBFD_PREC_MIXED && nb >= 2) ? 2 : 1;   // cols_per_lane<T, NB>()
    const int rows = kThreads * cpl / nb;
    g->maxw = H->max_width <= 13 ? 13 : kWaveMaxWidth;
    g->npass = (H->n + rows - 1) / rows;
    int64_t G = std::min<int64_t>(g->npass, std::min(kWaveMaxGrid, kWaveMaxPartials / nb));
    if (G >= kXcds) G -= G % kXcds;
    g->G = static_cast<int>(G < 1 ? 1 : G);
    g->batch = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(kWaveMaxBatch, kWaveBatchPasses / g->npass)));
    return true;
}

int launch_wave_reduce(int nb, const StepArgs &a, hipStream_t s) {
    const dim3 grid(reduce_wgs(nb), a.batch);
#define CHEBFD_WRED(NB_)                                                                           \
    case NB_:                                                                                      \
        hipLaunchKernelGGL((cheb_wave_reduce_kernel<NB_>), grid, dim3(kThreads), 0, s, a);        \
        break
    switch (nb) {
        CHEBFD_WRED(1);
        CHEBFD_WRED(2);
        CHEBFD_WRED(4);
        CHEBFD_WRED(8);
        CHEBFD_WRED(16);
        CHEBFD_WRED(32);
        CHEBFD_WRED(64);
        CHEBFD_WRED(128);
        default: CHEBFD_FAIL(CHEBFD_EINVAL, "n_b = %d not supported", nb);
    }
#undef CHEBFD_WRED
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_wave_step(int prec, int nb, int mode, const StepArgs &a, const WaveGeometry &g, hipStream_t s) {
    if (prec == CHEBFD_PREC_FP64) return launch_wave_nb<double>(nb, mode, a, g, s);
    return launch_wave_nb<float>(nb, mode, a, g, s);
}

}  // namespace chebfd
