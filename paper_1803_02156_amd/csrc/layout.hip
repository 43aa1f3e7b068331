// Support kernels: layout conversion between the caller's column-major c128
// block and the filter's blocked row-major layout, a blocked axpby, the
// Gershgorin bound reduction and the HBM stream probe.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace chebfd {

constexpr int kT = 256;

// Blocked element (b, i, j) <-> column-major element (row perm[i], column b*nb + j).
// One thread per blocked element, for narrow blocks (nb <= 2): rows are then next to
// each other on both sides.
template <typename T, bool UNPACK>
__global__ __launch_bounds__(kT) void pack_kernel(const int32_t *__restrict__ perm, int64_t n,
                                                  int m, int nb, const void *src, void *dst) {
    const int64_t total = n * m;
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * kT) {
        const int64_t b = t / (n * nb);
        const int64_t rem = t - b * n * nb;
        const int64_t i = rem / nb;
        const int j = static_cast<int>(rem - i * nb);
        const int64_t row = perm ? perm[i] : i;
        const int64_t cm = (b * nb + j) * n + row;  // column-major index
        if constexpr (!UNPACK) {
            const double2 v = static_cast<const double2 *>(src)[cm];
            if constexpr (sizeof(T) == 8) {
                static_cast<double2 *>(dst)[t] = v;
            } else {
                float2 f;
                f.x = static_cast<float>(v.x);
                f.y = static_cast<float>(v.y);
                static_cast<float2 *>(dst)[t] = f;
            }
        } else {
            double2 v;
            if constexpr (sizeof(T) == 8) {
                v = static_cast<const double2 *>(src)[t];
            } else {
                const float2 f = static_cast<const float2 *>(src)[t];
                v.x = f.x;
                v.y = f.y;
            }
            static_cast<double2 *>(dst)[cm] = v;
        }
    }
}

// The same for nb >= 4: a tile of kPackRows rows x CB columns goes through LDS, so that
// both sides move in runs (CB entries of a row in the blocked layout, the rows of a
// column -- consecutive as far as the row order keeps them -- in the other).
// Bound: HBM.  524288 x 64 c64 unpack: 859 -> 153 us, pack 396 -> 192 (element by
// element the column-major side was touched 16 bytes at a time with stride n).
constexpr int kPackRows = 64;
// Row tiles per launch column; more rows (67 million) go through the loop, since a grid
// holds at most 2^32 - 1 work-items in x.
constexpr int64_t kPackMaxGrid = 1 << 20;
template <typename T, bool UNPACK, int CB>
__global__ __launch_bounds__(kT) void pack_tile_kernel(const int32_t *__restrict__ perm, int64_t n, int nb,
                                                       const void *src, void *dst) {
    using VT = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
    __shared__ VT tile[kPackRows][CB + 1];
    const int64_t c0 = (int64_t)blockIdx.y * CB;                 // first column
    const int64_t bbase = c0 / nb * n * nb + c0 % nb;            // blocked index of (row 0, column c0)
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int RPP = kT / CB;                                 // rows per pass, blocked side
    const int c = threadIdx.x % CB, r0 = threadIdx.x / CB;
    const int64_t stride = (int64_t)gridDim.x * kPackRows;
    for (int64_t i0 = (int64_t)blockIdx.x * kPackRows; i0 < n; i0 += stride) {
        const int64_t il = i0 + lane;
        const int64_t row = il < n ? (perm ? perm[il] : il) : 0;     // this lane's row, column-major side
        if constexpr (UNPACK) {
#pragma unroll
            for (int r = r0; r < kPackRows; r += RPP)
                if (i0 + r < n) tile[r][c] = static_cast<const VT *>(src)[bbase + (i0 + r) * nb + c];
            __syncthreads();
            for (int k = wv; k < CB; k += kT / 64)
                if (il < n) {
                    const VT v = tile[lane][k];
                    static_cast<double2 *>(dst)[(c0 + k) * n + row] = double2{(double)v.x, (double)v.y};
                }
        } else {
            for (int k = wv; k < CB; k += kT / 64)
                if (il < n) {
                    const double2 v = static_cast<const double2 *>(src)[(c0 + k) * n + row];
                    VT f;
                    f.x = static_cast<T>(v.x);
                    f.y = static_cast<T>(v.y);
                    tile[lane][k] = f;
                }
            __syncthreads();
#pragma unroll
            for (int r = r0; r < kPackRows; r += RPP)
                if (i0 + r < n) static_cast<VT *>(dst)[bbase + (i0 + r) * nb + c] = tile[r][c];
        }
        if (i0 + stride < n) __syncthreads();   // the tile is written again
    }
}

template <typename T, bool UNPACK>
static void launch_pack_tile(const int32_t *perm, int64_t n, int m, int nb, const void *src, void *dst,
                             hipStream_t s) {
    const int cb = nb < 32 ? nb : 32;
    const dim3 grid(static_cast<unsigned>(std::min((n + kPackRows - 1) / kPackRows, kPackMaxGrid)), m / cb);
    switch (cb) {
        case 4: hipLaunchKernelGGL((pack_tile_kernel<T, UNPACK, 4>), grid, dim3(kT), 0, s, perm, n, nb, src, dst); break;
        case 8: hipLaunchKernelGGL((pack_tile_kernel<T, UNPACK, 8>), grid, dim3(kT), 0, s, perm, n, nb, src, dst); break;
        case 16: hipLaunchKernelGGL((pack_tile_kernel<T, UNPACK, 16>), grid, dim3(kT), 0, s, perm, n, nb, src, dst); break;
        default: hipLaunchKernelGGL((pack_tile_kernel<T, UNPACK, 32>), grid, dim3(kT), 0, s, perm, n, nb, src, dst); break;
    }
}

static int grid_for(int64_t work, int cap = 65536) {
    int64_t g = (work + kT - 1) / kT;
    if (g > cap) g = cap;
    return static_cast<int>(g < 1 ? 1 : g);
}

int launch_pack(const int32_t *perm, int64_t n, int m, int nb, int prec, const void *src,
                void *dst, bool unpack, hipStream_t s) {
    const int G = grid_for(n * m);
    if (nb >= 4 && m / 4 <= 65535) {   // (the grid's second dimension)
        if (prec == CHEBFD_PREC_FP64) {
            if (unpack)
                launch_pack_tile<double, true>(perm, n, m, nb, src, dst, s);
            else
                launch_pack_tile<double, false>(perm, n, m, nb, src, dst, s);
        } else {
            if (unpack)
                launch_pack_tile<float, true>(perm, n, m, nb, src, dst, s);
            else
                launch_pack_tile<float, false>(perm, n, m, nb, src, dst, s);
        }
        CHEBFD_HIP(hipGetLastError());
        return CHEBFD_OK;
    }
    if (prec == CHEBFD_PREC_FP64) {
        if (unpack)
            hipLaunchKernelGGL((pack_kernel<double, true>), dim3(G), dim3(kT), 0, s, perm, n, m, nb, src, dst);
        else
            hipLaunchKernelGGL((pack_kernel<double, false>), dim3(G), dim3(kT), 0, s, perm, n, m, nb, src, dst);
    } else {
        if (unpack)
            hipLaunchKernelGGL((pack_kernel<float, true>), dim3(G), dim3(kT), 0, s, perm, n, m, nb, src, dst);
        else
            hipLaunchKernelGGL((pack_kernel<float, false>), dim3(G), dim3(kT), 0, s, perm, n, m, nb, src, dst);
    }
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

// y <- a*y + b*x elementwise over `count` complex entries (degree 0 and 1 filters)
template <typename T>
__global__ __launch_bounds__(kT) void axpby_kernel(int64_t count, double a, T *y, double b,
                                                   const T *x) {
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < 2 * count;
         t += (int64_t)gridDim.x * kT) {
        const double xv = x ? static_cast<double>(x[t]) : 0.0;
        y[t] = static_cast<T>(a * static_cast<double>(y[t]) + b * xv);
    }
}

int launch_axpby_blocked(int prec, int64_t count, double a, void *y, double b, const void *x,
                         hipStream_t s) {
    const int G = grid_for(2 * count);
    if (prec == CHEBFD_PREC_FP64)
        hipLaunchKernelGGL((axpby_kernel<double>), dim3(G), dim3(kT), 0, s, count, a,
                           static_cast<double *>(y), b, static_cast<const double *>(x));
    else
        hipLaunchKernelGGL((axpby_kernel<float>), dim3(G), dim3(kT), 0, s, count, a,
                           static_cast<float *>(y), b, static_cast<const float *>(x));
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

// Gershgorin: per row c = Re(diagonal), r = sum of |off-diagonal|; per
// workgroup min(c - r) and max(c + r) -> part[2*w], part[2*w + 1].
template <typename T>
__global__ __launch_bounds__(kT) void bounds_kernel(const int64_t *__restrict__ chunk_off,
                                                    const int32_t *__restrict__ chunk_width,
                                                    const int32_t *__restrict__ col,
                                                    const T *__restrict__ val, int64_t n, int C,
                                                    int log2C, double *part) {
    __shared__ double slo[kT], shi[kT];
    double lo = 1.0 / 0.0, hi = -1.0 / 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
        const int64_t c = i >> log2C;
        const int64_t off = chunk_off[c] + (i & (C - 1));
        const int wdt = chunk_width[c];
        double d = 0.0, r = 0.0;
        for (int k = 0; k < wdt; ++k) {
            const int64_t sidx = off + (int64_t)k * C;
            const double re = static_cast<double>(val[2 * sidx]);
            const double im = static_cast<double>(val[2 * sidx + 1]);
            if (col[sidx] == i)
                d += re;
            else
                r += sqrt(re * re + im * im);
        }
        lo = fmin(lo, d - r);
        hi = fmax(hi, d + r);
    }
    slo[threadIdx.x] = lo;
    shi[threadIdx.x] = hi;
    __syncthreads();
    for (int h = kT / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            slo[threadIdx.x] = fmin(slo[threadIdx.x], slo[threadIdx.x + h]);
            shi[threadIdx.x] = fmax(shi[threadIdx.x], shi[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = slo[0];
        part[2 * blockIdx.x + 1] = shi[0];
    }
}

__global__ __launch_bounds__(kT) void bounds_final_kernel(const double *part, int G, double *out) {
    __shared__ double slo[kT], shi[kT];
    double lo = 1.0 / 0.0, hi = -1.0 / 0.0;
    for (int g = threadIdx.x; g < G; g += kT) {
        lo = fmin(lo, part[2 * g]);
        hi = fmax(hi, part[2 * g + 1]);
    }
    slo[threadIdx.x] = lo;
    shi[threadIdx.x] = hi;
    __syncthreads();
    for (int h = kT / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            slo[threadIdx.x] = fmin(slo[threadIdx.x], slo[threadIdx.x + h]);
            shi[threadIdx.x] = fmax(shi[threadIdx.x], shi[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = slo[0];
        out[1] = shi[0];
    }
}

int launch_bounds(const int64_t *chunk_off, const int32_t *chunk_width, const int32_t *col,
                  const void *val, int prec, int64_t n, int C, int log2C, double *part, int G,
                  hipStream_t s) {
    if (prec == CHEBFD_PREC_FP64)
        hipLaunchKernelGGL((bounds_kernel<double>), dim3(G), dim3(kT), 0, s, chunk_off, chunk_width,
                           col, static_cast<const double *>(val), n, C, log2C, part);
    else
        hipLaunchKernelGGL((bounds_kernel<float>), dim3(G), dim3(kT), 0, s, chunk_off, chunk_width,
                           col, static_cast<const float *>(val), n, C, log2C, part);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int launch_bounds_final(const double *part, int G, double *out2, hipStream_t s) {
    hipLaunchKernelGGL(bounds_final_kernel, dim3(1), dim3(kT), 0, s, part, G, out2);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

// STREAM-style probe over doubles, 16-byte vector accesses, grid-stride.
__global__ __launch_bounds__(kT) void copy_kernel(int64_t n2, const double2 *__restrict__ b,
                                                  double2 *__restrict__ a) {
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < n2; t += (int64_t)gridDim.x * kT)
        a[t] = b[t];
}

__global__ __launch_bounds__(kT) void triad_kernel(int64_t n2, const double2 *__restrict__ b,
                                                   const double2 *__restrict__ c, double s,
                                                   double2 *__restrict__ a) {
    for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < n2;
         t += (int64_t)gridDim.x * kT) {
        const double2 x = b[t], y = c[t];
        double2 r;
        r.x = fma(s, y.x, x.x);
        r.y = fma(s, y.y, x.y);
        a[t] = r;
    }
}

// Copy with non-temporal loads and stores, kU 16-byte elements per thread
// (consecutive threads take consecutive elements within each of the kU rounds).
constexpr int kU = 4;
typedef double dv2p __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(kT) void copy_nt_kernel(int64_t n2, const dv2p *__restrict__ b, dv2p *__restrict__ a) {
    const int64_t base = (int64_t)blockIdx.x * kT * kU + threadIdx.x;
    dv2p v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int64_t t = base + (int64_t)u * kT;
        if (t < n2) v[u] = __builtin_nontemporal_load(b + t);
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int64_t t = base + (int64_t)u * kT;
        if (t < n2) __builtin_nontemporal_store(v[u], a + t);
    }
}

// Read-only stream: per-workgroup sums of b (written to a[blockIdx.x]).
__global__ __launch_bounds__(kT) void read_kernel(int64_t n2, const dv2p *__restrict__ b, double *a) {
    __shared__ double sh[kT];
    const int64_t base = (int64_t)blockIdx.x * kT * kU + threadIdx.x;
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int64_t t = base + (int64_t)u * kT;
        if (t < n2) {
            const dv2p v = __builtin_nontemporal_load(b + t);
            acc += v.x + v.y;
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kT / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) a[blockIdx.x] = sh[0];
}

int launch_stream_probe(int kind, int64_t count, const double *b, const double *c, double sc,
                        double *a, int num_cus, hipStream_t s) {
    const int64_t n2 = count / 2;
    (void)num_cus;
    if (kind == 2 || kind == 3) {
        int64_t G = (n2 + (int64_t)kT * kU - 1) / ((int64_t)kT * kU);
        if (G > 0x7fffffff) G = 0x7fffffff;
        if (kind == 2)
            hipLaunchKernelGGL(copy_nt_kernel, dim3(G), dim3(kT), 0, s, n2, reinterpret_cast<const dv2p *>(b),
                               reinterpret_cast<dv2p *>(a));
        else
            hipLaunchKernelGGL(read_kernel, dim3(G), dim3(kT), 0, s, n2, reinterpret_cast<const dv2p *>(b), a);
        CHEBFD_HIP(hipGetLastError());
        return CHEBFD_OK;
    }
    // one 16-byte element per thread over a flat grid: the launch shape that
    // reaches the highest streaming rate of the plain copy on this device (a
    // persistent grid-stride loop of the same copy stays well below it)
    int64_t G = (n2 + kT - 1) / kT;
    if (G > 0x7fffffff) G = 0x7fffffff;
    if (G < 1) G = 1;
    if (kind == 0)
        hipLaunchKernelGGL(copy_kernel, dim3(G), dim3(kT), 0, s, n2,
                           reinterpret_cast<const double2 *>(b), reinterpret_cast<double2 *>(a));
    else
        hipLaunchKernelGGL(triad_kernel, dim3(G), dim3(kT), 0, s, n2,
                           reinterpret_cast<const double2 *>(b), reinterpret_cast<const double2 *>(c),
                           sc, reinterpret_cast<double2 *>(a));
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

}  // namespace chebfd
