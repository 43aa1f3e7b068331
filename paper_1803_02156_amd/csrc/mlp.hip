// Parameter predictor: a small FP32 multilayer perceptron from KPM moment
// features to (n_p, n_s), with forward pass, loss gradient and Adam update on
// the device.  The moments it reads are those of the filter's dot products
// (Sect. 2: KPM moments and the eigenvalue count come out of Alg. 1); the
// predictor replaces the hand-tuned choice of n_p and n_s (Sect. 2, Sect. 2.1).
//
// Network: x (258) -> relu(W1 x + b1) (128) -> relu(W2 h1 + b2) (128) -> W3 h2 + b3 (2).
// Parameters: one flat FP32 vector W1, b1, W2, b2, W3, b3 (weights row-major,
// output index slowest).  Batches are row-major (batch x features).
//
// The layers are small (258 x 128, 128 x 128, 128 x 2; the corpus has 125
// instances): the work is a few microseconds and launches, barriers and serial
// sums are what counts.  Forward: one launch for the whole network.  Gradient: one
// launch for the rows (network, loss, pre-activation gradients) and one for all
// weight gradients and the loss.  Batches past kRowsMax run the forward pass as
// three 64 x 64 LDS-tiled FP32 GEMMs.  Every output is accumulated in a fixed
// order, so results are bit-reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "common.h"

namespace chebfd {
namespace {

constexpr int kIn = CHEBFD_MLP_IN, kHid = CHEBFD_MLP_HIDDEN, kOut = CHEBFD_MLP_OUT;
constexpr int64_t kOffW1 = 0;
constexpr int64_t kOffB1 = kOffW1 + (int64_t)kHid * kIn;
constexpr int64_t kOffW2 = kOffB1 + kHid;
constexpr int64_t kOffB2 = kOffW2 + (int64_t)kHid * kHid;
constexpr int64_t kOffW3 = kOffB2 + kHid;
constexpr int64_t kOffB3 = kOffW3 + (int64_t)kOut * kHid;
constexpr int64_t kParams = kOffB3 + kOut;
static_assert(kParams == CHEBFD_MLP_PARAMS, "parameter count");

constexpr int kTile = 64, kKT = 16, kThreads = 256;

// C[i][j] = epi( sum_k A[i lda + k] B[j ldb + k] ),  epi: + bias[j], relu.
__global__ __launch_bounds__(kThreads) void gemm_kernel(int M, int N, int K, const float *__restrict__ A, int lda,
                                                        const float *__restrict__ B, int ldb, float *__restrict__ C,
                                                        int ldc, const float *__restrict__ bias, int relu) {
    __shared__ float sa[kKT][kTile + 1];
    __shared__ float sb[kKT][kTile + 1];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
    float acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = 0.0f;

    for (int k0 = 0; k0 < K; k0 += kKT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + kThreads * q;  // 0 .. 1023
            const int row = e / kKT, kk = e % kKT;
            const int i = i0 + row, j = j0 + row, k = k0 + kk;
            float v = 0.0f, w = 0.0f;
            if (i < M && k < K) v = A[(int64_t)i * lda + k];
            if (j < N && k < K) w = B[(int64_t)j * ldb + k];
            sa[kk][row] = v;
            sb[kk][row] = w;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kKT; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = sa[kk][ty + 16 * r];
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = sb[kk][tx + 16 * c];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(a[r], b[c], acc[r][c]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + ty + 16 * r;
        if (i >= M) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = j0 + tx + 16 * c;
            if (j >= N) continue;
            float v = acc[r][c];
            v += bias[j];
            if (relu) v = fmaxf(v, 0.0f);
            C[(int64_t)i * ldc + j] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// Rows kernel: the whole network (and, GRAD, the backward pass down to the
// pre-activation gradients) for R batch rows at a time in one workgroup.
// The weights are read once per workgroup into registers (unit j by 8 lanes, each
// every eighth pair or quad of its inputs), so a row costs LDS broadcasts and
// multiply-adds.  One workgroup fills a CU; a batch that gives every row a CU takes
// one row at a time, a larger one four per barrier.  Bound: latency of the chain
// load -> layer 1 -> layer 2 -> output up to about 1000 rows, then LDS reads (0.3 us
// per row and CU).  Time per call before (layer-wise 64 x 64 GEMMs, two or fewer
// workgroups per layer and 22 us each) -> now: batch 1 59 -> 12 us, 2000 78 -> 13;
// with the gradient batch 125 225 -> 16, 2000 1939 -> 87 (its sums over the
// batch were one thread's serial loop).
// ---------------------------------------------------------------------------
// pairs and quads at any float address (parameters and features carry no alignment)
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRowT = 1024;
constexpr int kX2 = kIn / 2;                    // float2 of a feature row
constexpr int kW1Regs = (kX2 + 7) / 8;          // of them per lane
constexpr int kGrp = kRowT / kHid;              // threads per hidden unit
static_assert(kIn % 2 == 0 && kGrp == 8 && kHid % (4 * kGrp) == 0, "layout of the rows kernel");

// sum over the 8 lanes of a hidden unit (every lane gets it)
__device__ inline float sum8(float v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    return v;
}

struct MlpRows {
    const float *P, *X, *T;
    float *Y;                                   // forward: outputs
    float *h1, *h2, *dz2, *dz1, *dy, *lossrow;  // GRAD
    float inv_b;
    int batch;
};

template <int R, bool GRAD>
__global__ __launch_bounds__(kRowT) void mlp_rows_kernel(MlpRows a) {
    __shared__ __align__(16) float sx[R][kIn + 2];
    __shared__ __align__(16) float sh1[R][kHid];
    __shared__ __align__(16) float sh2[R][kHid];
    __shared__ float sdz2[GRAD ? R : 1][kHid];
    __shared__ float sw3[kOut * kHid];
    __shared__ float sred[GRAD ? kGrp * R * kHid : 1];
    __shared__ float sdy[R][kOut], sd2[R][kOut];
    const int tid = threadIdx.x, j = tid / kGrp, l = tid % kGrp;
    const int wv = tid >> 6, lane = tid & 63;
    const float *__restrict__ P = a.P;

    // this lane's share of the weights: unit j, every eighth pair (layer 1) or quad
    // (layer 2) of inputs; GRAD: column tid % 128 of W2, rows 16 (tid / 128) + q
    f2u w1[kW1Regs];
#pragma unroll
    for (int q = 0; q < kW1Regs; ++q) {
        const int k2 = l + kGrp * q;
        w1[q] = k2 < kX2 ? reinterpret_cast<const f2u *>(P + kOffW1 + (int64_t)j * kIn)[k2] : f2u{0.0f, 0.0f};
    }
    constexpr int kW2Regs = kHid / (4 * kGrp);
    f4u w2[kW2Regs];
#pragma unroll
    for (int q = 0; q < kW2Regs; ++q)
        w2[q] = reinterpret_cast<const f4u *>(P + kOffW2 + (int64_t)j * kHid)[l + kGrp * q];
    float w2t[GRAD ? kHid / kGrp : 1];
    if constexpr (GRAD) {
#pragma unroll
        for (int q = 0; q < kHid / kGrp; ++q)
            w2t[q] = P[kOffW2 + (int64_t)((tid / kHid) * (kHid / kGrp) + q) * kHid + tid % kHid];
    }
    const float b1 = P[kOffB1 + j], b2 = P[kOffB2 + j];
    if (tid < kOut * kHid) sw3[tid] = P[kOffW3 + tid];
    if (tid < R) sx[tid][kIn] = sx[tid][kIn + 1] = 0.0f;   // read with the weights 0 past the row

    for (int base = blockIdx.x * R; base < a.batch; base += gridDim.x * R) {
        const int rows = a.batch - base < R ? a.batch - base : R;
        for (int t = tid; t < R * kX2; t += kRowT) {
            const int r = t / kX2, k2 = t % kX2;
            f2u v{0.0f, 0.0f};
            if (r < rows) v = reinterpret_cast<const f2u *>(a.X + (int64_t)(base + r) * kIn)[k2];
            reinterpret_cast<float2 *>(sx[r])[k2] = float2{v.x, v.y};
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int q = 0; q < kW1Regs; ++q) {
                const int k2 = l + kGrp * q;
                const float2 x = reinterpret_cast<const float2 *>(sx[r])[k2 < kX2 ? k2 : kX2];
                s0 = fmaf(w1[q].x, x.x, s0);
                s1 = fmaf(w1[q].y, x.y, s1);
            }
            const float h = fmaxf(sum8(s0 + s1) + b1, 0.0f);
            if (l == 0) {
                sh1[r][j] = h;
                if (GRAD && r < rows) a.h1[(int64_t)(base + r) * kHid + j] = h;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int q = 0; q < kW2Regs; ++q) {
                const float4 x = reinterpret_cast<const float4 *>(sh1[r])[l + kGrp * q];
                s0 = fmaf(w2[q].x, x.x, s0);
                s1 = fmaf(w2[q].y, x.y, s1);
                s0 = fmaf(w2[q].z, x.z, s0);
                s1 = fmaf(w2[q].w, x.w, s1);
            }
            const float h = fmaxf(sum8(s0 + s1) + b2, 0.0f);
            if (l == 0) {
                sh2[r][j] = h;
                if (GRAD && r < rows) a.h2[(int64_t)(base + r) * kHid + j] = h;
            }
        }
        __syncthreads();
        // output o of row r: one wave
        if (wv < R * kOut) {
            const int r = wv / kOut, o = wv % kOut;
            float s = sw3[o * kHid + lane] * sh2[r][lane];
            s = fmaf(sw3[o * kHid + 64 + lane], sh2[r][64 + lane], s);
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
            if (lane == 0 && r < rows) {
                const float y = s + P[kOffB3 + o];
                const int64_t e = (int64_t)(base + r) * kOut + o;
                if constexpr (GRAD) {
                    const float d = y - a.T[e], dy = d * a.inv_b;
                    a.dy[e] = dy;
                    sdy[r][o] = dy;
                    sd2[r][o] = d * d;
                } else {
                    a.Y[e] = y;
                }
            }
        }
        if constexpr (GRAD) {
            __syncthreads();
            // dZ2 = (dY W3) * [H2 > 0]
            for (int t = tid; t < R * kHid; t += kRowT) {
                const int r = t / kHid, c = t % kHid;
                float v = 0.0f;
                if (r < rows) {
                    v = fmaf(sdy[r][1], sw3[kHid + c], sdy[r][0] * sw3[c]);
                    v = sh2[r][c] > 0.0f ? v : 0.0f;
                    a.dz2[(int64_t)(base + r) * kHid + c] = v;
                }
                sdz2[r][c] = v;
            }
            if (tid < rows) a.lossrow[base + tid] = sd2[tid][0] + sd2[tid][1];
            __syncthreads();
            // dZ1 = (dZ2 W2) * [H1 > 0]
            const int c = tid % kHid, g = tid / kHid;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float s = 0.0f;
#pragma unroll
                for (int q = 0; q < kHid / kGrp; ++q) s = fmaf(sdz2[r][g * (kHid / kGrp) + q], w2t[q], s);
                sred[(g * R + r) * kHid + c] = s;
            }
            __syncthreads();
            for (int t = tid; t < R * kHid; t += kRowT) {
                const int r = t / kHid, cc = t % kHid;
                float s = 0.0f;
#pragma unroll
                for (int q = 0; q < kGrp; ++q) s += sred[(q * R + r) * kHid + cc];
                if (r < rows) a.dz1[(int64_t)(base + r) * kHid + cc] = sh1[r][cc] > 0.0f ? s : 0.0f;
            }
        }
        __syncthreads();
    }
}

// Gradients of all weights and biases from the pre-activation gradients D and the
// layer inputs A of every row: g[i][k] = sum_b D[b][i] A[b][k], the bias as the
// column k = K with A = 1.  A workgroup forms a 32 x 32 tile, its 16 waves every
// sixteenth batch row each (4 x 4 entries per lane), summed in wave order; one more
// workgroup sums the loss.  `first`: index of the launch's first workgroup (the loss can
// go ahead of the gradients in a launch of its own).
constexpr int kWT = 32, kWWaves = kRowT / 64;
constexpr int kWk1 = (kIn + 1 + kWT - 1) / kWT, kWk2 = (kHid + 1 + kWT - 1) / kWT, kWi = kHid / kWT;
constexpr int kWTiles1 = kWi * kWk1, kWTiles2 = kWi * kWk2, kWTiles = kWTiles1 + kWTiles2 + kWk2;

__global__ __launch_bounds__(kRowT) void mlp_wgrad_kernel(MlpRows a, float *__restrict__ G, float *__restrict__ loss, int first) {
    __shared__ float sred[kWWaves][kWT][kWT + 1];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int t = static_cast<int>(blockIdx.x) + first;
    if (t == kWTiles) {
        float s = 0.0f;
        for (int b = tid; b < a.batch; b += kRowT) s += a.lossrow[b];
        float *f = &sred[0][0][0];
        f[tid] = s;
        __syncthreads();
        for (int w = kRowT / 2; w > 0; w /= 2) {
            if (tid < w) f[tid] += f[tid + w];
            __syncthreads();
        }
        if (tid == 0) loss[0] = 0.5f * f[0] * a.inv_b;
        return;
    }
    const float *D, *A;
    float *gw, *gb;
    int ldd, lda, N, K, it, kt;
    if (t < kWTiles1) {
        D = a.dz1; A = a.X; ldd = kHid; lda = kIn; N = kHid; K = kIn;
        gw = G + kOffW1; gb = G + kOffB1; it = t / kWk1; kt = t % kWk1;
    } else if (t < kWTiles1 + kWTiles2) {
        D = a.dz2; A = a.h1; ldd = kHid; lda = kHid; N = kHid; K = kHid;
        gw = G + kOffW2; gb = G + kOffB2; it = (t - kWTiles1) / kWk2; kt = (t - kWTiles1) % kWk2;
    } else {
        D = a.dy; A = a.h2; ldd = kOut; lda = kHid; N = kOut; K = kHid;
        gw = G + kOffW3; gb = G + kOffB3; it = 0; kt = t - kWTiles1 - kWTiles2;
    }
    const int i0 = it * kWT + lane / 8 * 4, k0 = kt * kWT + lane % 8 * 4;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][k] = 0.0f;
    if (N == kHid && kt * kWT + kWT <= K) {
        // whole tile (rows of D are 16-byte aligned)
#pragma unroll 8
        for (int b = wv; b < a.batch; b += kWWaves) {
            const float4 d = *reinterpret_cast<const float4 *>(D + (int64_t)b * ldd + i0);
            const f2u x0 = *reinterpret_cast<const f2u *>(A + (int64_t)b * lda + k0);
            const f2u x1 = *reinterpret_cast<const f2u *>(A + (int64_t)b * lda + k0 + 2);
            const float dv[4] = {d.x, d.y, d.z, d.w}, xv[4] = {x0.x, x0.y, x1.x, x1.y};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[i][k] = fmaf(dv[i], xv[k], acc[i][k]);
        }
    } else {
#pragma unroll 4
        for (int b = wv; b < a.batch; b += kWWaves) {
            float dv[4], xv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dv[i] = i0 + i < N ? D[(int64_t)b * ldd + i0 + i] : 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[k] = k0 + k < K ? A[(int64_t)b * lda + k0 + k] : 1.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[i][k] = fmaf(dv[i], xv[k], acc[i][k]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) sred[wv][lane / 8 * 4 + i][lane % 8 * 4 + k] = acc[i][k];
    __syncthreads();
    const int ti = tid / kWT, tk = tid % kWT;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kWWaves; ++w) s += sred[w][ti][tk];
    const int i = it * kWT + ti, k = kt * kWT + tk;
    if (i < N && k < K) gw[(int64_t)i * K + k] = s;
    if (i < N && k == K) gb[i] = s;
}

// Adam with bias correction factors c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ __launch_bounds__(kThreads) void adam_kernel(int64_t count, float *__restrict__ p,
                                                        const float *__restrict__ g, float *__restrict__ m,
                                                        float *__restrict__ v, float lr, float b1, float b2,
                                                        float c1, float c2, float eps) {
    for (int64_t e = blockIdx.x * (int64_t)kThreads + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * kThreads) {
        const float ge = g[e];
        const float me = fmaf(b1, m[e], (1.0f - b1) * ge);
        const float ve = fmaf(b2, v[e], (1.0f - b2) * ge * ge);
        m[e] = me;
        v[e] = ve;
        p[e] -= lr * (me * c1) / (sqrtf(ve * c2) + eps);
    }
}

int gemm(int M, int N, int K, const float *A, int lda, const float *B, int ldb, float *C, int ldc,
         const float *bias, bool relu, hipStream_t s) {
    const dim3 grid((N + kTile - 1) / kTile, (M + kTile - 1) / kTile);
    hipLaunchKernelGGL(gemm_kernel, grid, dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc, bias, relu ? 1 : 0);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

// Workspace of a batch: H1, H2 (batch x 128), Y, dY (batch x 2), dZ2, dZ1 (batch x 128).
struct MlpWork {
    float *h1, *h2, *y, *dy, *dz2, *dz1;
};

size_t mlp_work_layout(int batch, char *base, MlpWork *w) {
    size_t at = 0;
    auto take = [&](size_t floats) {
        char *p = base ? base + at : nullptr;
        at = round_up(at + floats * sizeof(float), 256);
        return reinterpret_cast<float *>(p);
    };
    MlpWork t;
    t.h1 = take((size_t)batch * kHid);
    t.h2 = take((size_t)batch * kHid);
    t.y = take((size_t)batch * kOut);
    t.dy = take((size_t)batch * kOut);
    t.dz2 = take((size_t)batch * kHid);
    t.dz1 = take((size_t)batch * kHid);
    if (w) *w = t;
    return at;
}

// The forward pass takes the rows kernel up to this batch and layer-wise GEMMs past it
// (16000 rows: 79 and 102 us; 32000: 154 and 122).  Outputs that lie inside the features
// or the parameters take the GEMMs too: their first launches have read these before the
// last one writes, while in the rows kernel other workgroups still read them.
constexpr int kRowsMax = 16384;

int check_batch(int batch, const void *d_work, size_t work_bytes, size_t *need) {
    CHEBFD_REQUIRE(batch >= 1 && batch <= (1 << 20), "batch = %d out of range [1, 2^20]", batch);
    *need = mlp_work_layout(batch, nullptr, nullptr);
    CHEBFD_REQUIRE(d_work && aligned(d_work, 256), "d_work must be non-NULL and 256-byte aligned");
    if (work_bytes < *need) CHEBFD_FAIL(CHEBFD_EWORKSPACE, "MLP workspace %zu < %zu", work_bytes, *need);
    return CHEBFD_OK;
}

// Rows kernel launch: one row at a time while every row has a CU of its own, else
// four (the weights stay in registers, the barriers are shared)
template <bool GRAD>
int launch_rows(const MlpRows &a, hipStream_t s) {
    DeviceProps d;
    const int rc = device_props(&d);
    if (rc) return rc;
    if (a.batch <= d.num_cus)
        hipLaunchKernelGGL((mlp_rows_kernel<1, GRAD>), dim3(a.batch), dim3(kRowT), 0, s, a);
    else
        hipLaunchKernelGGL((mlp_rows_kernel<4, GRAD>), dim3(std::min(d.num_cus, (a.batch + 3) / 4)), dim3(kRowT), 0, s,
                           a);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int forward(const float *P, int batch, const float *X, float *Y, const MlpWork &w, hipStream_t s) {
    int rc;
    const size_t ybytes = sizeof(float) * kOut * (size_t)batch;
    const bool apart = !overlap(Y, ybytes, X, sizeof(float) * kIn * (size_t)batch) &&
                       !overlap(Y, ybytes, P, sizeof(float) * kParams);
    if (batch <= kRowsMax && apart) {
        MlpRows a{};
        a.P = P;
        a.X = X;
        a.Y = Y;
        a.batch = batch;
        return launch_rows<false>(a, s);
    }
    if ((rc = gemm(batch, kHid, kIn, X, kIn, P + kOffW1, kIn, w.h1, kHid, P + kOffB1, true, s))) return rc;
    if ((rc = gemm(batch, kHid, kHid, w.h1, kHid, P + kOffW2, kHid, w.h2, kHid, P + kOffB2, true, s))) return rc;
    return gemm(batch, kOut, kHid, w.h2, kHid, P + kOffW3, kHid, Y, kOut, P + kOffB3, false, s);
}

}  // namespace
}  // namespace chebfd

using namespace chebfd;

extern "C" {

int chebfd_mlp_query(int32_t batch, int32_t *n_params, size_t *work_bytes) {
    clear_error();
    CHEBFD_REQUIRE(batch >= 1 && batch <= (1 << 20), "batch = %d out of range [1, 2^20]", batch);
    if (n_params) *n_params = (int32_t)kParams;
    if (work_bytes) *work_bytes = mlp_work_layout(batch, nullptr, nullptr);
    return CHEBFD_OK;
}

int chebfd_mlp_forward(const float *d_params, int32_t batch, const float *d_x, float *d_y, void *d_work,
                       size_t work_bytes, void *stream) {
    clear_error();
    size_t need;
    int rc;
    if ((rc = check_batch(batch, d_work, work_bytes, &need))) return rc;
    CHEBFD_REQUIRE(d_params && d_x && d_y, "NULL device buffer");
    CHEBFD_REQUIRE(!overlap(d_y, sizeof(float) * kOut * (size_t)batch, d_work, need), "d_y overlaps d_work");
    MlpWork w;
    mlp_work_layout(batch, static_cast<char *>(d_work), &w);
    return forward(d_params, batch, d_x, d_y, w, static_cast<hipStream_t>(stream));
}

int chebfd_mlp_grad(const float *d_params, int32_t batch, const float *d_x, const float *d_t, float *d_loss,
                    float *d_grad, void *d_work, size_t work_bytes, void *stream) {
    clear_error();
    size_t need;
    int rc;
    if ((rc = check_batch(batch, d_work, work_bytes, &need))) return rc;
    CHEBFD_REQUIRE(d_params && d_x && d_t && d_loss && d_grad, "NULL device buffer");
    CHEBFD_REQUIRE(!overlap(d_grad, sizeof(float) * kParams, d_params, sizeof(float) * kParams) &&
                       !overlap(d_grad, sizeof(float) * kParams, d_work, need),
                   "d_grad overlaps d_params or d_work");
    hipStream_t s = static_cast<hipStream_t>(stream);
    MlpWork w;
    mlp_work_layout(batch, static_cast<char *>(d_work), &w);
    MlpRows a{};
    a.P = d_params;
    a.X = d_x;
    a.T = d_t;
    a.h1 = w.h1;
    a.h2 = w.h2;
    a.dz2 = w.dz2;
    a.dz1 = w.dz1;
    a.dy = w.dy;
    a.lossrow = w.y;
    a.inv_b = 1.0f / (float)batch;
    a.batch = batch;
    if ((rc = launch_rows<true>(a, s))) return rc;
    // a loss that lies inside the gradient is written first, so that the gradient is whole
    const bool apart = !overlap(d_loss, sizeof(float), d_grad, sizeof(float) * kParams);
    if (!apart) {
        hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(1), dim3(kRowT), 0, s, a, d_grad, d_loss, kWTiles);
        CHEBFD_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(apart ? kWTiles + 1 : kWTiles), dim3(kRowT), 0, s, a, d_grad, d_loss, 0);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

int chebfd_mlp_adam(float *d_params, const float *d_grad, float *d_m, float *d_v, int32_t step, float lr,
                    float beta1, float beta2, float eps, void *stream) {
    clear_error();
    CHEBFD_REQUIRE(d_params && d_grad && d_m && d_v, "NULL device buffer");
    CHEBFD_REQUIRE(step >= 1, "step = %d must count from 1", step);
    CHEBFD_REQUIRE(lr > 0.0f && beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps > 0.0f,
                   "Adam hyper-parameters out of range");
    const double c1 = 1.0 / (1.0 - std::pow((double)beta1, step));
    const double c2 = 1.0 / (1.0 - std::pow((double)beta2, step));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((kParams + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       static_cast<hipStream_t>(stream), kParams, d_params, d_grad, d_m, d_v, lr, beta1, beta2,
                       (float)c1, (float)c2, eps);
    CHEBFD_HIP(hipGetLastError());
    return CHEBFD_OK;
}

}  // extern "C"
