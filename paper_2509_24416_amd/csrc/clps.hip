// Single-layer CLPS clip search on the GPU (CLQ, arXiv 2509.24416, Sec. 3.4:
// a grid search of the quantizer bounds between quantiles of the layer's
// weights that minimises the squared Frobenius norm of the output error,
// Eq. (3); Sec. 4.1: beta = 0, gamma = 0.01, one percentile for every
// channel of a matrix).  The target is the layer's own unquantised output;
// the searched quantity is the weight clip ratio alpha of the hot path
// (row bound alpha * max|w~_row|).
//
// Steps, all on the caller's stream with no host synchronisation:
//   clps_row_ratio_kernel  per weight row: gather, block FWHT (the quantizer's
//                          fp32 butterflies), then the order statistic of |.|
//                          with floor(gamma (K-1)) values above it over the
//                          max.
//   clps_grid_kernel       alpha_lo = min of the row ratios; the G candidates
//                          alpha_i = 1 - ((1 - alpha_lo)(G-1-i)) / (G-1).
//   per batch of up to     the hot path's weight quantizer, which rotates a row
//   kQuantBatch candidates once and quantizes it with every candidate's alpha_i
//                          (read from device memory), then the W4A4 GEMM in
//                          its squared-error mode over all of the batch's
//                          tiles: the epilogue forms (Y0 - sum * x_scale *
//                          w_scale)^2 in fp64 from the exact integer sums and
//                          keeps one partial per wave of each output tile (no
//                          product is stored);
//   clps_sum_kernel        one workgroup per candidate adds that candidate's
//                          partials in index order, so results are
//                          deterministic; the last one to finish picks the
//                          smallest error, ties to the lower index.
// The activations are rotated and quantized once.
//
// The GEMMs bound the search.  One candidate of a 4096 x 3456 layer has 432
// tiles for the 512 workgroups the chip holds, so a launch per candidate is
// one badly filled round of latency-bound tiles; a batch of 7 has 3024.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clq_internal.h"
#include "radix_select.h"
#include "rq_device.h"

namespace clq {
namespace {

constexpr int kRatioThreads = 256;
constexpr int kMaxGrid = 256;   // candidates per search (checked by the caller)
constexpr int kQuantBatch = 8;  // candidates whose weights exist at a time

// Rows of up to 4096 columns: one wave per row, NV 8-column chunks per lane in
// registers (the split of rq_device.h), no LDS and no barrier.  The A-th
// largest magnitude by bisection on bit patterns (non-negative floats order as
// their bits): hi stays above it, at least A values stay at or above lo; a
// probe with exactly A values at or above it ends the search at their minimum.
// The probes start at half the maximum, so a row of continuous values takes
// about 7 counts (two instructions a value) where four 8-bit radix passes
// through LDS serialise on the few exponents in use: 3456 x 1152 33 -> 12 us.
template <int B, int NV>
__global__ void __launch_bounds__(kRatioThreads)
clps_row_ratio_wave_kernel(const uint16_t *__restrict__ W, const int32_t *__restrict__ perm, int64_t N, int K,
                           int order_idx, float *__restrict__ ratio)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (kRatioThreads / 64) + (threadIdx.x >> 6);
    if (row >= N) return;   // a whole wave
    const uint16_t *src = W + row * K;
    const int cpr = K >> 3, lc = logical_lane(lane);
    const CrossSigns cs = cross_signs<B>(lc);
    float x[NV][8];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int chunk = lc + 64 * i, cc = min(chunk, cpr - 1);
        if (perm == nullptr) {
            uint4 v = *reinterpret_cast<const uint4 *>(src + cc * 8);
            if (chunk >= cpr) v = make_uint4(0u, 0u, 0u, 0u);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) stage1_packed(w[e], x[i][2 * e], x[i][2 * e + 1]);
        } else {
            uint32_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = src[perm[cc * 8 + e]];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = chunk < cpr ? h[e] : 0u;
#pragma unroll
            for (int e = 0; e < 8; e += 2) stage1_pair(h[e], h[e + 1], x[i][e], x[i][e + 1]);
        }
        fwht8_rest(x[i]);
    }
    cross_stages<B, NV>(x, cs);
    // magnitudes (signs do not matter; columns past the row's end are zeros,
    // which never displace one of the K values from the top K)
    uint32_t key[NV][8], kmax = 0u;
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = fabsf(x[i][e]);
            key[i][e] = __float_as_uint(v);
            kmax = max(kmax, key[i][e]);
            mx = fmaxf(mx, v);
        }
    for (int off = 32; off > 0; off >>= 1) {
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
        mx = fmaxf(mx, __shfl_xor(mx, off));
    }
    const int A = K - order_idx;
    uint32_t lo = 0u, hi = __builtin_amdgcn_readfirstlane(kmax) + 1u;
    uint32_t mid = __builtin_amdgcn_readfirstlane(__float_as_uint(0.5f * mx));
    bool exact = false;
    if (mid >= hi) mid = hi >> 1;
    while (hi - lo > 1u) {
        if (mid <= lo) mid = lo + ((hi - lo) >> 1);
        int c = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i][e] >= mid));
        if (c >= A) lo = mid;
        else hi = mid;
        if (c == A) {
            exact = true;
            break;
        }
        mid = lo + ((hi - lo) >> 1);
    }
    uint32_t q = lo;
    if (exact) {   // the smallest of the A values at or above lo
        q = ~0u;
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (key[i][e] >= lo) q = min(q, key[i][e]);
        for (int off = 32; off > 0; off >>= 1) q = min(q, (uint32_t)__shfl_xor((int)q, off));
    }
    if (lane == 0) ratio[row] = mx == 0.0f ? 1.0f : __uint_as_float(q) / mx;
}

// wider rows: one workgroup per row; LDS holds the row
__global__ void __launch_bounds__(kRatioThreads)
clps_row_ratio_kernel(const uint16_t *__restrict__ W, const int32_t *__restrict__ perm, int K, int block,
                      int order_idx, float *__restrict__ ratio)
{
    extern __shared__ float w[];   // [K]
    const int row = blockIdx.x, t = threadIdx.x;
    const uint16_t *src = W + (int64_t)row * K;
    for (int i = t; i < K; i += kRatioThreads)
        w[i] = __half2float(__ushort_as_half(src[perm ? perm[i] : i]));
    __syncthreads();
    // block FWHT: stage h pairs (i, i + h) with (i mod 2h) < h, ascending h
    for (int h = 1; h < block; h <<= 1) {
        for (int p = t; p < K / 2; p += kRatioThreads) {
            const int i = (p / h) * 2 * h + (p % h);
            const float u = w[i], v = w[i + h];
            w[i] = u + v;
            w[i + h] = u - v;
        }
        __syncthreads();
    }
    // |w~| as integer keys (non-negative floats order as their bit patterns)
    // and its maximum; then the order statistic by radix selection (exact
    // with repeated values)
    __shared__ float redf[kRatioThreads / 64];
    __shared__ uint32_t hist[256], wsum[4], pick[2];
    uint32_t *keys = reinterpret_cast<uint32_t *>(w);
    const int lane = t & 63, wv = t >> 6;
    float m = 0.0f;
    for (int i = t; i < K; i += kRatioThreads) {
        const float v = fabsf(w[i]);
        keys[i] = __float_as_uint(v);
        m = fmaxf(m, v);
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if (lane == 0) redf[wv] = m;
    __syncthreads();
    float mx = redf[0];
    for (int k = 1; k < kRatioThreads / 64; ++k) mx = fmaxf(mx, redf[k]);
    const float q = __uint_as_float(radix_select<kRatioThreads>(keys, K, order_idx, hist, wsum, pick));
    if (t == 0) ratio[row] = mx == 0.0f ? 1.0f : q / mx;
}

__global__ void __launch_bounds__(256)
clps_grid_kernel(const float *__restrict__ ratio, int64_t N, int G, float *__restrict__ alphas,
                 unsigned *__restrict__ finished)
{
    __shared__ float red[256];
    if (threadIdx.x == 0) *finished = 0u;   // the sum kernel's count of finished workgroups
    float m = 1.0f;
    for (int64_t i = threadIdx.x; i < N; i += 256) m = fminf(m, ratio[i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fminf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    const float lo = red[0];
    for (int i = threadIdx.x; i < G; i += 256) {
        if (G == 1) {
            alphas[i] = 1.0f;
        } else {
            const float tt = 1.0f - lo;
            const float u = tt * (float)(G - 1 - i);
            const float v = u / (float)(G - 1);
            alphas[i] = 1.0f - v;
        }
    }
}

// workgroup g: errors[g] = the sum of partial[g * n .. g * n + n) (thread t
// takes t, t + 256, ... in order, then a fixed tree); the last workgroup to
// finish then picks the smallest error
__global__ void __launch_bounds__(256)
clps_sum_kernel(const double *__restrict__ partial, int n, double *__restrict__ errors,
                unsigned *__restrict__ finished, int32_t *__restrict__ best)
{
    __shared__ double red[256];
    const int G = (int)gridDim.x;
    partial += (int64_t)blockIdx.x * n;
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    __shared__ int last;
    const int t = threadIdx.x;
    if (t == 0) {
        __hip_atomic_store(errors + blockIdx.x, red[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        last = __hip_atomic_fetch_add(finished, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)G - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (t < G) red[t] = __hip_atomic_load(errors + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (t == 0) {
        int b = 0;
        for (int i = 1; i < G; ++i)
            if (red[i] < red[b]) b = i;
        *best = b;
    }
}

struct ClpsLayout {
    size_t ratio, finished, xq, xs, wq, ws, partial, total;
    size_t wq_stride, ws_stride;   // between the quantized weights of a batch's candidates
};

constexpr int kWaveRatioCols = 4096;

template <int B>
void launch_ratio_wave(const uint16_t *W, const int32_t *perm, int64_t N, int K, int order_idx, float *ratio,
                       hipStream_t stream) {
    const dim3 grid((unsigned)((N + 3) / 4)), block(kRatioThreads);
    const int nv = (K + 511) / 512;
#define CLQ_RATIO(NV) hipLaunchKernelGGL((clps_row_ratio_wave_kernel<B, NV>), grid, block, 0, stream, W, perm, N, K, order_idx, ratio)
    if (nv <= 1) CLQ_RATIO(1);
    else if (nv == 2) CLQ_RATIO(2);
    else if (nv == 3) CLQ_RATIO(3);
    else if (nv == 4) CLQ_RATIO(4);
    else if (nv <= 6) CLQ_RATIO(6);
    else CLQ_RATIO(8);
#undef CLQ_RATIO
}

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

ClpsLayout clps_layout(int64_t M, int64_t N, int64_t K) {
    ClpsLayout l{};
    size_t off = 0;
    l.ratio = off;   off += align256((size_t)N * 4);
    l.finished = off; off += 256;
    l.xq = off;      off += align256((size_t)padded_act_rows(M) * (size_t)(K / 2));
    l.xs = off;      off += align256((size_t)M * 4);
    l.wq_stride = align256((size_t)padded_rows(N) * (size_t)(K / 2));
    l.ws_stride = align256((size_t)N * 4);
    l.wq = off;      off += kQuantBatch * l.wq_stride;
    l.ws = off;      off += kQuantBatch * l.ws_stride;
    // room for every candidate's partials (the grid is at most kMaxGrid)
    l.partial = off; off += align256((size_t)kMaxGrid * (size_t)gemm_err_partials(M, N) * 8);
    l.total = off;
    return l;
}

}  // namespace

size_t clps_workspace_bytes(int64_t M, int64_t N, int64_t K) { return clps_layout(M, N, K).total; }

hipError_t launch_clps(const uint16_t *X, int64_t ldx, const uint16_t *W, const float *Y0, int64_t ldy0,
                       const int32_t *perm, int64_t M, int64_t N, int K, int block, int order_idx,
                       int grid, void *workspace, float *alphas, double *errors, int32_t *best,
                       hipStream_t stream) {
    const ClpsLayout l = clps_layout(M, N, K);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    float *ratio = reinterpret_cast<float *>(base + l.ratio);
    uint8_t *xq = base + l.xq;
    float *xs = reinterpret_cast<float *>(base + l.xs);
    uint8_t *wq = base + l.wq;
    float *wsc = reinterpret_cast<float *>(base + l.ws);
    double *partial = reinterpret_cast<double *>(base + l.partial);
    const int64_t P = gemm_err_partials(M, N);
    if (grid < 1 || grid > kMaxGrid || P > INT32_MAX) return hipErrorInvalidValue;

    unsigned *finished = reinterpret_cast<unsigned *>(base + l.finished);
    hipError_t e = hipSuccess;
    if (K <= kWaveRatioCols) {
        switch (block) {
            case 32: launch_ratio_wave<32>(W, perm, N, K, order_idx, ratio, stream); break;
            case 64: launch_ratio_wave<64>(W, perm, N, K, order_idx, ratio, stream); break;
            case 128: launch_ratio_wave<128>(W, perm, N, K, order_idx, ratio, stream); break;
            default: return hipErrorInvalidValue;
        }
    } else {
        e = hipFuncSetAttribute((const void *)clps_row_ratio_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                16384 * 4);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(clps_row_ratio_kernel, dim3((unsigned)N), dim3(kRatioThreads), (size_t)K * 4, stream, W,
                           perm, K, block, order_idx, ratio);
    }
    hipLaunchKernelGGL(clps_grid_kernel, dim3(1), dim3(256), 0, stream, ratio, N, grid, alphas, finished);
    e = launch_rotate_quant(X, ldx, perm, M, padded_act_rows(M), K, block, 1.0f, false, 1.0f, xq, xs, stream);
    if (e != hipSuccess) return e;
    const int64_t wqs = (int64_t)l.wq_stride, wss = (int64_t)(l.ws_stride / 4);
    // batches of nearly equal size, at most kQuantBatch candidates (and under
    // 2^32 lanes of the error GEMM, 64 for each partial)
    const int most = (int)std::max<int64_t>(1, std::min<int64_t>(kQuantBatch, UINT32_MAX / (64 * P)));
    const int batches = (grid + most - 1) / most;
    for (int i = 0, i0 = 0; i < batches; ++i) {
        const int nc = (grid - i0 + (batches - i) - 1) / (batches - i);
        e = launch_rotate_quant(W, K, perm, N, padded_rows(N), K, block, 1.0f, true, 1.0f / (float)block, wq, wsc,
                                stream, 4, alphas + i0, nc, wqs, wss);
        if (e != hipSuccess) return e;
        e = launch_gemm_err(xq, xs, wq, wsc, nc, wqs, wss, M, N, K, Y0, ldy0, partial + (int64_t)i0 * P, stream);
        if (e != hipSuccess) return e;
        i0 += nc;
    }
    hipLaunchKernelGGL(clps_sum_kernel, dim3((unsigned)grid), dim3(256), 0, stream, partial, (int)P, errors, finished,
                       best);
    return hipGetLastError();
}

}  // namespace clq
