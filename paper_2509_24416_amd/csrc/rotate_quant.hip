// Fused online rotation + per-row quantization (gfx950).
//
// Paper (CLQ, arXiv 2509.24416): Sec. 3.3 applies G = S.H to the activations
// at inference time with a fast Hadamard transform (S a column swap given as a
// gather vector, H block-diagonal with +-1 entries) and absorbs the same G
// into the weights offline; Sec. 3.1 Eq. (1) quantizes with Round(Clip(.)),
// n = 4, dynamically per token for activations and once per output channel
// for weights.
//
// One kernel serves activations and weights in every code storage.  What
// bounds it is memory (2 bytes in, 0.5 to 1 byte out per element), so the
// split is chosen for the accesses: a lane owns one 16-byte chunk (8 columns)
// of four rows.  A wave's loads are then whole contiguous kilobytes with four
// in flight per lane, and no row passes through LDS.
//
//   rotation   stages h = 1, 2, 4 inside the lane (h = 1 fused with the fp16
//              -> fp32 widening), h = 8, 16, 32, 64 across lanes, one fp32
//              operation per element and stage (rq_device.h: the stage order
//              and the roundings are those of the plain butterflies);
//   row max    per lane, then over 8 lanes by lane permutes, then one LDS max
//              per 8 lanes and row, between two barriers (the clear of the
//              maxima, with gathered inputs their staging, and the maxima);
//   codes      each lane of a quad divides once (correctly rounded) for one
//              of the four rows and the quad shares the reciprocals; one fma
//              per element:
//                  fma(x, r, 1.5 * 2^23 + 8)
//              rounds the exact product x * r to the nearest integer, ties to
//              even (the sum lands in the binade where the float spacing is
//              1), and leaves q + 8 in the low nibble of the result's bit
//              pattern with bits 4..21 clear, which makes packing a few
//              shifts and one byte permute;
//   stores     the quad transposes 4 rows x 4 chunks, so that each lane holds
//              the 32 codes of one row and the quad writes four rows' 16-byte
//              pieces (64 contiguous bytes of every code layout).
//
// The row groups of a 32-row unit go to workgroups of one XCD, next to each
// other in its dispatch order: the 128-byte lines of the code layouts hold
// the pieces of 8 rows, and their halves meet in that XCD's L2.
//
// Measured inside the block workloads (us; before: rows staged through LDS,
// one Hadamard block per lane, pipelined batches): activations 4608 x 12288,
// b = 128: 66.9 -> 38.1; 4608 x 3072: 17.5 -> 11.9; 43200 x 1152, b = 64: 33.5 ->
// 29.3 to 32.2; 43200 x 4608: 132.9 -> 119.0 (4.2 TB/s while the previous
// product's output drains); weights 12288 x 3072, b = 128: 42.7 -> 18.9 for the
// whole call (5.0 TB/s), whose 8-byte pieces used to go out one by one.  Timed
// alone, cached: 8192 x 1152 9.8 -> 8.2, 1024 x 1152 (all launch and latency)
// 5.1 -> 3.8, gathered 7.1 -> 4.0.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clq_internal.h"
#include "rq_device.h"
#include "f6_codes.h"

namespace clq {
namespace {

constexpr int kMaxGroups = 8;    // four-row groups per workgroup
constexpr int kMaxLanes = 1024;

struct RqArgs {
    const uint16_t *X;
    int64_t ldx;
    const int32_t *perm;
    int64_t rows_valid, rows_alloc;
    int64_t unit0;          // first 32-row unit of this launch
    int units;              // units of this launch
    int K;
    int groups;             // four-row groups per workgroup (a power of two, at most 8)
    int stride;             // lanes per group (NCH == 1: the row's chunks)
    float alpha;            // weights: the clip ratio,
    const float *alpha_dev; //   or its address (then alpha is unused)
    float post_scale;
    uint8_t *out;
    float *scale;
    int batch;              // quantizations of the same rows, quantization y with
    int64_t out_stride, scale_stride;   // alpha_dev[y], at y * stride
};

// Exchange between the two lanes of a pair (CTRL: xor 1 or 2; b: the lane's
// side): lo becomes side 0's own lo or side 1's view of the partner's hi, hi
// side 1's own hi or side 0's view of the partner's lo.  The permutes run on
// every lane before the selects.
template <int CTRL>
__device__ __forceinline__ void pair_exchange(uint32_t &lo, uint32_t &hi, bool b) {
    const uint32_t plo = lane_xchg<CTRL>(lo), phi = lane_xchg<CTRL>(hi);
    lo = b ? phi : lo;
    hi = b ? hi : plo;
}

// Transposes a quad's 4 x 4 dwords: lane k of the quad (b0, b1: the bits of
// its logical index k) ends with d[j] = lane j's d[k].
__device__ __forceinline__ void quad_transpose(uint32_t (&d)[4], bool b0, bool b1) {
    pair_exchange<kLaneXor1>(d[0], d[1], b0);
    pair_exchange<kLaneXor1>(d[2], d[3], b0);
    pair_exchange<kLaneXor2>(d[0], d[2], b1);
    pair_exchange<kLaneXor2>(d[1], d[3], b1);
}

// The codes of one chunk column of a quad's four rows, from the rotated
// values x[row][8] and their signed reciprocals rs[row].  u, rho0: the rows'
// unit and first fragment row (rho0 % 4 == 0, rows rho0 .. rho0 + 3); chunk:
// this lane's chunk.
template <int QB, bool WEIGHT>
__device__ __forceinline__ void store_codes(const float (&x)[4][8], const float (&rs)[4], int64_t u, int rho0,
                                            int chunk, int K, uint8_t *__restrict__ out, bool active) {
    constexpr float M = Grid<QB>::magic, Q = Grid<QB>::qmax;
    const int lam = chunk & 3;
    const bool b0 = lam & 1, b1 = lam & 2;
    const int64_t c32 = chunk >> 2;
    auto code = [&](int r, int e) -> float {
        float v = __builtin_fmaf(x[r][e], rs[r], M);
        if constexpr (WEIGHT) v = __builtin_amdgcn_fmed3f(v, M - Q, M + Q);
        return v;
    };
    if constexpr (QB == 4) {
        uint32_t d[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            uint32_t w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __float_as_uint(code(r, e));
            d[r] = pack8(w);
        }
        quad_transpose(d, b0, b1);
        if (active)
            *reinterpret_cast<uint4 *>(out + ((u * (K >> 6) + (c32 >> 1)) * 64 + (c32 & 1) * 32 + rho0 + lam) * 16) =
                make_uint4(d[0], d[1], d[2], d[3]);
    } else if constexpr (QB == 8) {
        // a 16-byte operand piece is the even codes of 16, then the odd: a
        // lane pair's.  Lane b0 of the pair takes rows b0 and 2 + b0.
        uint32_t ev[4], od[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            uint32_t w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __float_as_uint(code(r, e));
            ev[r] = low_bytes4(w[0], w[2], w[4], w[6]) ^ 0x80808080u;
            od[r] = low_bytes4(w[1], w[3], w[5], w[7]) ^ 0x80808080u;
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            pair_exchange<kLaneXor1>(ev[2 * s], ev[2 * s + 1], b0);
            pair_exchange<kLaneXor1>(od[2 * s], od[2 * s + 1], b0);
            if (active)
                *reinterpret_cast<uint4 *>(out + q8_piece_offset(u, rho0 + 2 * s + (lam & 1), c32, lam >> 1, K)) =
                    make_uint4(ev[2 * s], ev[2 * s + 1], od[2 * s], od[2 * s + 1]);
        }
    } else {
        // fp6: the codes as exact fp16 pairs, transposed, then the
        // matrix-operand conversion of a row's 32
        uint32_t h[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) h[j][r] = f6_half_pair(code(r, 2 * j) - M, code(r, 2 * j + 1) - M);
            quad_transpose(h[j], b0, b1);
        }
        uint32_t p[16], w6[6];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) p[4 * k + j] = h[j][k];
        f6_from_half_codes(p, w6);
        if (active) f6_store(out + f6_unit_offset(u, c32, K), f6_lane(c32, rho0 + lam), w6);
    }
}

// NCH: chunks per lane, held in registers from the rotation to the codes (1:
// rows of up to 8192 columns, 2: up to 16384).  With one chunk the registers
// are held to 72, for 28 waves a compute unit.
template <int B, int QB, bool WEIGHT, int NCH>
__global__ void __launch_bounds__(kMaxLanes) __attribute__((amdgpu_waves_per_eu(NCH == 1 ? 7 : 4)))
rotate_quant_kernel(RqArgs a)
{
    extern __shared__ __align__(16) uint2 gat[];   // gathered inputs: [group][K] columns of four rows
    __shared__ uint32_t rowmax[kMaxGroups * 4];
    const int t = threadIdx.x;
    const int wpu = 8 / a.groups;                   // workgroups per unit
    const int idx = blockIdx.x >> 3;
    const int64_t ul = (int64_t)(blockIdx.x & 7) + 8 * (int64_t)(idx / wpu);
    if (ul >= a.units) return;
    const int64_t u = a.unit0 + ul;
    const int cpr = a.K >> 3;
    const int gl = t / a.stride, t0 = t - gl * a.stride;
    const bool glive = gl < a.groups;
    // fragment-row order: group s of a unit holds fragment rows 4s .. 4s + 3,
    // the consecutive rows 4s (activations) or 16 (s & 1) + 4 (s >> 1)
    // (weights) onwards
    const int s = (idx % wpu) * a.groups + (glive ? gl : 0);
    const int64_t row0 = u * 32 + (WEIGHT ? 16 * (s & 1) + 4 * (s >> 1) : 4 * s);

    // the logical chunk of a lane among the eight of its octet (rq_device.h)
    const int lane_c = logical_lane(t0);
    const CrossSigns cs = cross_signs<B>(lane_c);

    if (t < kMaxGroups * 4) rowmax[t] = 0u;
    const uint16_t *xr[4];
    bool rv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        rv[r] = glive && row0 + r < a.rows_valid;
        xr[r] = a.X + (rv[r] ? row0 + r : 0) * a.ldx;
    }
    const bool gather = a.perm != nullptr;

    auto load = [&](int chunk, uint4 (&v)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)   // (unconditional, so that all four are in flight)
            v[r] = *reinterpret_cast<const uint4 *>(xr[r] + min(chunk, cpr - 1) * 8);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (!rv[r] || chunk >= cpr) v[r] = make_uint4(0u, 0u, 0u, 0u);
    };
    // rotated values of one chunk of the four rows (a lane past the row's end
    // works on zeros: every lane takes part in the exchanges)
    auto rotate = [&](const uint4 (&v)[4], float (&x)[4][8]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t w[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) stage1_packed(w[e], x[r][2 * e], x[r][2 * e + 1]);
            fwht8_rest(x[r]);
        }
        cross_stages<B, 4>(x, cs);
    };
    auto rotate_gathered = [&](int chunk, float (&x)[4][8]) {
        const int32_t *p = a.perm + (int64_t)min(chunk, cpr - 1) * 8;
        const uint2 *grow = gat + (glive ? gl : 0) * a.K;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const int k0 = p[e], k1 = p[e + 1];
            const uint2 q0 = grow[k0], q1 = grow[k1];
            stage1_pair(q0.x, q1.x, x[0][e], x[0][e + 1]);
            stage1_pair_hi(q0.x, q1.x, x[1][e], x[1][e + 1]);
            stage1_pair(q0.y, q1.y, x[2][e], x[2][e + 1]);
            stage1_pair_hi(q0.y, q1.y, x[3][e], x[3][e + 1]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) fwht8_rest(x[r]);
        cross_stages<B, 4>(x, cs);
    };

    constexpr int NX = NCH;
    float x[NX][4][8];
    float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto take_max = [&](const float (&y)[4][8]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < 8; e += 2) m[r] = fmaxf(fmaxf(m[r], fabsf(y[r][e])), fabsf(y[r][e + 1]));
    };
    uint4 v[NX][4];
#pragma unroll
    for (int i = 0; i < NX; ++i) load(lane_c + i * a.stride, v[i]);
    if (gather) {
        // columns k of the group's four rows side by side: one 8-byte read
        // per gathered column serves all four
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int chunk = lane_c + i * a.stride;
            uint32_t q[16];
            interleave_rows(v[i], q);
            if (glive && chunk < cpr) {
                uint4 *dst = reinterpret_cast<uint4 *>(gat + gl * a.K + chunk * 8);
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[j] = make_uint4(q[4 * j], q[4 * j + 1], q[4 * j + 2], q[4 * j + 3]);
            }
        }
        __syncthreads();   // also orders the clear of rowmax
        // (an octet past the row's end works on other columns, and is
        // left out of the maximum and the codes)
#pragma unroll
        for (int i = 0; i < NX; ++i) rotate_gathered(lane_c + i * a.stride, x[i]);
    } else {
#pragma unroll
        for (int i = 0; i < NX; ++i) rotate(v[i], x[i]);
        __syncthreads();   // rowmax cleared
    }
#pragma unroll
    for (int i = 0; i < NX; ++i)
        if (lane_c + i * a.stride < cpr) take_max(x[i]);

    // row maxima: over the octet, then lane k < 4 of it reports row k
    octet_max(m);
    const int k8 = t & 7;
    const float mk = k8 == 0 ? m[0] : k8 == 1 ? m[1] : k8 == 2 ? m[2] : m[3];
    if (k8 < 4 && glive) atomicMax(&rowmax[gl * 4 + k8], __float_as_uint(mk));
    __syncthreads();

    const int prow = t & 3;   // the row this lane divides for
    const float am = glive ? __uint_as_float(rowmax[gl * 4 + prow]) : 0.0f;
    // (several quantizations of the same rows: 4-bit weights only, so that the
    // others need not keep the rotated values past their codes)
    const int batch = WEIGHT && QB == 4 ? a.batch : 1;
    for (int y = 0; y < batch; ++y) {
        const float al = a.alpha_dev != nullptr ? a.alpha_dev[y] : a.alpha;
        const float ac = WEIGHT ? al * am : am;
        const float rc = (ac == 0.0f) ? 0.0f : Grid<QB>::qmax / ac;
        if (t0 < 4 && glive && row0 + prow < a.rows_valid)
            a.scale[y * a.scale_stride + row0 + prow] = (ac / Grid<QB>::qmax) * a.post_scale;
        float rs[4];
        rs[0] = lane_xchg<kQuadLane0>(rc) * cs.sign;
        rs[1] = lane_xchg<kQuadLane1>(rc) * cs.sign;
        rs[2] = lane_xchg<kQuadLane2>(rc) * cs.sign;
        rs[3] = lane_xchg<kQuadLane3>(rc) * cs.sign;
        uint8_t *out = a.out + y * a.out_stride;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int chunk = lane_c + i * a.stride;
            store_codes<QB, WEIGHT>(x[i], rs, u, 4 * s, chunk, a.K, out, glive && chunk < cpr);
        }
    }
}

// ---- rows of more than 16384 columns, and few long rows ----------------------------
// Four rows past 16384 columns do not fit a workgroup's registers.  One workgroup per row: the
// row staged in LDS with coalesced 16-byte loads (each chunk of a Hadamard
// block in an XOR-swizzled slot, so that the block reads hit distinct banks),
// then one block per lane in registers.  Rotating twice with the kernel above
// instead took 17 us for 64 x 32768 against 7, and gathering its inputs from
// memory 115 against 10.
// (Lanes per workgroup never exceed 512 for b >= 64, which lets the compiler
// keep a 128-element block in registers.  R is 1 and the batch one quantization at
// every call; with the two arguments taken out the compiler keeps more registers,
// and 700 x 32768 took 25.1 us instead of 22.4.)
// Sixteen quantized words (code + 128 in bits 0..7, bits 8..21 clear) into
// one 16-byte int8 operand piece: codes 0, 2, ..., 14 in bytes 0..7, codes 1,
// 3, ..., 15 in bytes 8..15 (the order of the widened 4-bit operands), two's
// complement.
__device__ __forceinline__ uint4 pack16_q8(const uint32_t *w) {
    auto four = [](uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
        const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
        const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
        return __builtin_amdgcn_perm(cd, ab, 0x05040100u) ^ 0x80808080u;
    };
    return make_uint4(four(w[0], w[2], w[4], w[6]), four(w[8], w[10], w[12], w[14]),
                      four(w[1], w[3], w[5], w[7]), four(w[9], w[11], w[13], w[15]));
}

// The int8 codes of one lane's b-element block (codes 32c .. of the row's
// 32-code chunks j * b/32 + c): two 16-byte operand pieces per chunk.
template <int B, bool WEIGHT>
__device__ __forceinline__ void store_q8(const float *x, float rc, int64_t grow, int j, int K,
                                         uint8_t *__restrict__ out) {
    constexpr float M = Grid<8>::magic, Q = Grid<8>::qmax;
    const int64_t u = grow >> 5;
    const int rho = WEIGHT ? wq_rho((int)(grow & 31)) : (int)(grow & 31);
#pragma unroll
    for (int c = 0; c < B / 32; ++c) {
        const int64_t c32 = (int64_t)j * (B / 32) + c;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint32_t w[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                float v = __builtin_fmaf(x[32 * c + 16 * q + t], rc, M);
                if constexpr (WEIGHT) v = __builtin_amdgcn_fmed3f(v, M - Q, M + Q);
                w[t] = __float_as_uint(v);
            }
            *reinterpret_cast<uint4 *>(out + q8_piece_offset(u, rho, c32, q, K)) = pack16_q8(w);
        }
    }
}

template <int B>
constexpr int wide_max_threads() { return B == 32 ? 1024 : 512; }

template <int B, bool WEIGHT, int QB>
__global__ void __launch_bounds__(wide_max_threads<B>())
rotate_quant_wide_kernel(const uint16_t *__restrict__ X, int64_t ldx,
                    const int32_t *__restrict__ perm, int64_t rows_valid,
                    int64_t rows_alloc, int K, int R, float alpha, const float *__restrict__ alpha_dev,
                    float post_scale, uint8_t *__restrict__ out, float *__restrict__ scale_out,
                    int64_t out_stride, int64_t scale_stride)
{
    extern __shared__ __align__(16) unsigned char smem[];
    // blockIdx.y selects one of several quantizations of the same rows
    // (clip ratio alpha_dev[y], outputs at y * stride)
    out += (int64_t)blockIdx.y * out_stride;
    scale_out += (int64_t)blockIdx.y * scale_stride;
    if (alpha_dev != nullptr) alpha_dev += blockIdx.y;
    constexpr int CPB = B / 8;            // 16-byte chunks per block
    const int cpr = K >> 3;               // chunks per row
    const int nb = K / B;                 // blocks per row
    uint4 *tile = reinterpret_cast<uint4 *>(smem);
    unsigned *rowmax = reinterpret_cast<unsigned *>(smem + (size_t)R * K * 2);

    const int t = threadIdx.x;
    const int T = blockDim.x;
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int rows = (int)min((int64_t)R, rows_alloc - row0);

    if (t < R) rowmax[t] = 0u;

    // 1. coalesced copy of the rows into LDS (rows past rows_valid are zeros)
    {
        int r = t / cpr, cc = t - r * cpr;
        const int dr = T / cpr, dc = T - dr * cpr;
        while (r < rows) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            const int64_t grow = row0 + r;
            if (grow < rows_valid)
                v = *reinterpret_cast<const uint4 *>(X + grow * ldx + (int64_t)cc * 8);
            const int j = cc / CPB, i = cc % CPB;
            tile[r * cpr + j * CPB + chunk_slot<B>(i, j)] = v;
            cc += dc;
            r += dr;
            if (cc >= cpr) { cc -= cpr; ++r; }
        }
    }
    __syncthreads();

    // 2. one Hadamard block per lane
    const int r = t / nb, j = t - r * nb;
    const bool active = r < rows;
    float x[B];
    float bmax = 0.0f;
    if (active) {
        if (perm == nullptr) {
            const uint4 *src = tile + r * cpr + j * CPB;
#pragma unroll
            for (int i = 0; i < CPB; ++i) {
                const uint4 v = src[chunk_slot<B>(i, j)];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    stage1_packed(w[e], x[8 * i + 2 * e], x[8 * i + 2 * e + 1]);   // stage h = 1
                }
            }
        } else {
            const uint16_t *rowh = reinterpret_cast<const uint16_t *>(tile + r * cpr);
            const int32_t *p = perm + j * B;
#pragma unroll
            for (int e = 0; e < B; e += 2) {
                const int k0 = p[e], k1 = p[e + 1];
                const int c0 = k0 >> 3, c1 = k1 >> 3;
                const int s0 = (c0 / CPB) * CPB + chunk_slot<B>(c0 % CPB, c0 / CPB);
                const int s1 = (c1 / CPB) * CPB + chunk_slot<B>(c1 % CPB, c1 / CPB);
                stage1_pair(rowh[s0 * 8 + (k0 & 7)], rowh[s1 * 8 + (k1 & 7)], x[e], x[e + 1]);
            }
        }
#pragma unroll
        for (int h = 2; h < B; h <<= 1) {
#pragma unroll
            for (int i = 0; i < B; ++i) {
                if ((i & h) == 0) {
                    const float u = x[i], v = x[i + h];
                    x[i] = u + v;
                    x[i + h] = u - v;
                }
            }
        }
        bmax = block_absmax<B>(x);
        atomicMax(&rowmax[r], __float_as_uint(bmax));
    }
    __syncthreads();
    if (!active) return;

    // 3. per-row scale and codes
    const float a = __uint_as_float(rowmax[r]);
    // the clip ratio: a launch argument, or read from device memory (a
    // search that picks it on the GPU)
    const float al = alpha_dev != nullptr ? *alpha_dev : alpha;
    const float ac = WEIGHT ? al * a : a;
    const float rc = (ac == 0.0f) ? 0.0f : Grid<QB>::qmax / ac;
    const int64_t grow = row0 + r;
    if (j == 0 && grow < rows_valid) scale_out[grow] = (ac / Grid<QB>::qmax) * post_scale;
    if constexpr (QB == 8) {
        store_q8<B, WEIGHT>(x, rc, grow, j, K, out);
        return;
    }

    if constexpr (QB == 6) {
        // fp6 layout: the codes as exact floats, six dwords per 32 codes
        const int rho = WEIGHT ? wq_rho((int)(grow & 31)) : (int)(grow & 31);
#pragma unroll
        for (int i = 0; i < B; ++i) {
            float v = __builtin_fmaf(x[i], rc, kMagic);
            if constexpr (WEIGHT) v = __builtin_amdgcn_fmed3f(v, kMagic - 7.0f, kMagic + 7.0f);
            x[i] = v - kMagic;
        }
#pragma unroll
        for (int c = 0; c < B / 32; ++c) {
            const int64_t c32 = (int64_t)j * (B / 32) + c;
            uint32_t w6[6];
            f6_from_codes(&x[32 * c], w6);
            f6_store(out + f6_unit_offset(grow >> 5, c32, K), f6_lane(c32, rho), w6);
        }
        return;
    }
    uint32_t words[B / 8];
#pragma unroll
    for (int g = 0; g < B / 8; ++g) {
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = __builtin_fmaf(x[8 * g + e], rc, kMagic);
            if constexpr (WEIGHT) v = __builtin_amdgcn_fmed3f(v, kMagic - 7.0f, kMagic + 7.0f);
            w[e] = __float_as_uint(v);
        }
        words[g] = pack8(w);
    }

    if constexpr (!WEIGHT) {
        // packed activation layout: one 16-byte chunk per 32 codes
#pragma unroll
        for (int c = 0; c < B / 32; ++c) {
            const int64_t c32 = (int64_t)j * (B / 32) + c;
            *reinterpret_cast<uint4 *>(out + xq_chunk_offset(grow, c32, K)) =
                make_uint4(words[4 * c], words[4 * c + 1], words[4 * c + 2], words[4 * c + 3]);
        }
    } else {
        // packed weight layout: one 8-byte piece per k-group of 16 codes
#pragma unroll
        for (int g = 0; g < B / 16; ++g) {
            const int64_t kg = (int64_t)j * (B / 16) + g;
            uint2 *dst = reinterpret_cast<uint2 *>(out + wq_piece_offset(grow, kg, K));
            *dst = make_uint2(words[2 * g], words[2 * g + 1]);
        }
    }
}

// ---- fp6 codes of rows of 4160 to 5120 columns, b = 64 ------------------------------
// Such a row's chunks are 9 waves, the last of them partly empty, or 10, of which a
// compute unit holds 20 of its 28, and in fp6 codes every store of four rows is a
// 64-byte piece and a 32-byte tail.  Here a workgroup takes batches of 8 rows,
// whose pieces are whole 128-byte lines: staged in LDS, one Hadamard block a lane
// with the rows fastest, the next batch's loads in registers under this one's
// work, one workgroup per compute unit.  Two barriers per batch: after the block
// reads (the buffer may be refilled, and the previous maxima have been read) and
// after the block maxima (codes may be formed).  Codes of a batch are formed at
// the top of the next iteration, from the registers that still hold its rotated
// blocks.  16384 rows, us, four rows a lane / here, inputs from memory: 4160 columns
// 43.7 / 39.9, 4352 44.4 / 41.0, 4864 48.5 / 45.9 (4.8 TB/s), 5120 49.2 / 47.4; the 9
// full waves of 4608 columns, 27 of them resident, gain 3% by themselves (44.6 / 43.3)
// and nothing behind a GEMM (a block 341.0 / 343.3), and nibble codes lose (12000 x
// 4608: 27.7 / 29.6).
constexpr int kRows8 = 8, kRows8Lanes = kRows8 * 80;

__global__ void __launch_bounds__(kRows8Lanes)
rotate_quant_rows8_f6_kernel(const uint16_t *__restrict__ X, int64_t ldx, int64_t rows_valid, int64_t rows_alloc,
                             int64_t nbatch, int K, uint8_t *__restrict__ out, float *__restrict__ scale_out)
{
    constexpr int R = kRows8, B = 64, CPB = B / 8;
    extern __shared__ __align__(16) unsigned char smem[];
    const int cpr = K >> 3, nb = K / B, chunks = R * cpr;
    uint4 *tile = reinterpret_cast<uint4 *>(smem);
    unsigned *rowmax = reinterpret_cast<unsigned *>(tile + chunks);   // [2][R]
    const int t = threadIdx.x, T = blockDim.x;
    const int64_t G = gridDim.x;

    // this lane's chunks: source offset, and LDS slot | row << 16 | valid << 19
    // (slots < 8 * 640)
    int lsrc[CPB], lmeta[CPB];
#pragma unroll
    for (int k = 0; k < CPB; ++k) {
        const int c = t + k * T;
        const int r = c / cpr, cc = c - r * cpr;
        lsrc[k] = r * (int)ldx + cc * 8;
        const int jj = cc / CPB, ii = cc - jj * CPB;
        lmeta[k] = c < chunks ? (r * cpr + jj * CPB + (ii ^ r)) | (r << 16) | (1 << 19) : 0;
    }
    uint4 ld[CPB];
    auto load = [&](int64_t batch) {
        const int64_t row0 = batch * R;
        const uint16_t *base = X + row0 * ldx;
#pragma unroll
        for (int k = 0; k < CPB; ++k) {
            ld[k] = make_uint4(0u, 0u, 0u, 0u);
            if ((lmeta[k] >> 19) && row0 + ((lmeta[k] >> 16) & 7) < rows_valid)
                ld[k] = *reinterpret_cast<const uint4 *>(base + lsrc[k]);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < CPB; ++k)
            if (lmeta[k] >> 19) tile[lmeta[k] & 0xFFFF] = ld[k];
    };

    const int j = t >> 3, r = t & 7;   // rows fastest
    const bool active = j < nb;
    int64_t b = blockIdx.x;
    if (b >= nbatch) return;
    if (t < 2 * R) rowmax[t] = 0u;
    load(b);
    stash();
    if (b + G < nbatch) load(b + G);
    __syncthreads();

    float x[B];
#pragma unroll
    for (int e = 0; e < B; ++e) x[e] = 0.0f;
    int64_t prev = -1;   // batch whose rotated blocks x holds, codes pending
    int i = 0;
    auto codes = [&](int64_t pb, int pi) {
        const float a = __uint_as_float(rowmax[(pi & 1) * R + r]);
        const float rc = (a == 0.0f) ? 0.0f : Grid<6>::qmax / a;
        const int64_t grow = pb * R + r;
        if (!active || grow >= rows_alloc) return;
        if (j == 0 && grow < rows_valid) scale_out[grow] = a / Grid<6>::qmax;
#pragma unroll
        for (int e = 0; e < B; ++e) x[e] = __builtin_fmaf(x[e], rc, kMagic) - kMagic;
#pragma unroll
        for (int c = 0; c < B / 32; ++c) {
            const int64_t c32 = (int64_t)j * (B / 32) + c;
            uint32_t w6[6];
            f6_from_codes(&x[32 * c], w6);
            f6_store(out + f6_unit_offset(grow >> 5, c32, K), f6_lane(c32, (int)(grow & 31)), w6);
        }
    };

    for (; b < nbatch; ++i, b += G) {
        if (prev >= 0) codes(prev, i - 1);
        if (active) {
            const uint4 *src = tile + r * cpr + j * CPB;
#pragma unroll
            for (int ii = 0; ii < CPB; ++ii) {
                const uint4 v = src[ii ^ r];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) stage1_packed(w[e], x[8 * ii + 2 * e], x[8 * ii + 2 * e + 1]);
            }
        }
        __syncthreads();   // every block read and every read of the previous maxima done
        if (t < R) rowmax[((i + 1) & 1) * R + t] = 0u;   // the next batch's, read last by the codes above
        if (active) {
#pragma unroll
            for (int h = 2; h < B; h <<= 1)
#pragma unroll
                for (int ii = 0; ii < B; ++ii)
                    if ((ii & h) == 0) {
                        const float u = x[ii], v = x[ii + h];
                        x[ii] = u + v;
                        x[ii + h] = u - v;
                    }
            atomicMax(&rowmax[(i & 1) * R + r], __float_as_uint(block_absmax<B>(x)));
        }
        if (b + G < nbatch) stash();
        if (b + 2 * G < nbatch) load(b + 2 * G);
        __syncthreads();   // maxima complete, next batch staged
        prev = b;
    }
    if (prev >= 0) codes(prev, i - 1);
}

constexpr int kLdsLimit = 160 * 1024 - 1024;   // gathered rows of a workgroup (dynamic LDS)

// Four-row groups per workgroup for rows of up to 8192 columns: the most live
// lanes on a compute unit, that is the lane utilisation of whole waves times
// the share of the 28 waves a unit holds that whole workgroups of this size
// fill: at 2048 columns 16-wave workgroups left 12 of them empty (20000 rows in
// fp6 codes 30.7 us with them, 23.3 with 4-wave ones and the registers within
// 28 waves).  More groups on a tie, up to 8 and 1024 lanes, but no more than
// leaves two workgroups per compute unit to the launch, nor than 12 waves: of
// 13 or 14, four on a SIMD, the unit's 7 a SIMD hold one workgroup and not two
// (12000 rows of 3584 columns, b = 64: 25.2 us with 14 waves, 19.1 with 7).
int pick_groups(int stride, int64_t total_groups, int cus) {
    int best = 1;
    double best_u = 0.0;
    for (int g = 1; g <= kMaxGroups && g * stride <= kMaxLanes; g <<= 1) {
        if (g > 1 && g * stride > 64 && total_groups / g < 2 * cus) break;
        const int waves = (g * stride + 63) / 64;
        if (g > 1 && waves > 12) break;
        const double u = (double)(g * stride) * (28 / waves);
        if (u >= best_u) {
            best_u = u;
            best = g;
        }
    }
    return best;
}

template <int B, int QB, bool WEIGHT, int NCH>
hipError_t launch_rq(RqArgs a, hipStream_t stream) {
    const int cpr = a.K >> 3;
    const int64_t units = a.rows_alloc / 32;
    int T;
    if constexpr (NCH == 1) {
        a.stride = cpr;
        a.groups = pick_groups(cpr, units * 8, compute_units());
        while (a.perm != nullptr && a.groups > 1 && (size_t)a.groups * a.K * 8 > kLdsLimit) a.groups >>= 1;
        T = (a.groups * cpr + 63) / 64 * 64;
    } else {
        a.groups = 1;
        a.stride = ((cpr + 1) / 2 + 63) / 64 * 64;
        T = a.stride;
    }
    const size_t lds = a.perm != nullptr ? (size_t)a.groups * a.K * 8 : 0;
    if (T > kMaxLanes || lds > kLdsLimit) return hipErrorInvalidConfiguration;
    if (lds > 65536 - 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)rotate_quant_kernel<B, QB, WEIGHT, NCH>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
        if (e != hipSuccess) return e;
    }
    // launches of at most 2^31 lanes
    const int64_t per_unit = (int64_t)(8 / a.groups) * T;
    const int64_t most = std::max<int64_t>(8, (((int64_t)1 << 31) / per_unit) / 8 * 8);
    for (a.unit0 = 0; a.unit0 < units; a.unit0 += most) {
        a.units = (int)std::min<int64_t>(most, units - a.unit0);
        const int64_t grid = ((int64_t)a.units + 7) / 8 * 8 * (8 / a.groups);
        hipLaunchKernelGGL((rotate_quant_kernel<B, QB, WEIGHT, NCH>), dim3((unsigned)grid), dim3(T), lds, stream, a);
    }
    return hipGetLastError();
}

template <int B, int QB, bool WEIGHT>
hipError_t launch_rq_wide(const RqArgs &a, hipStream_t stream) {
    const int T = (a.K / B + 63) / 64 * 64;
    const size_t lds = (size_t)a.K * 2 + 4;
    if (T > wide_max_threads<B>() || lds > 65536 + 4096) return hipErrorInvalidConfiguration;
    hipError_t e = hipFuncSetAttribute((const void *)rotate_quant_wide_kernel<B, WEIGHT, QB>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 65536 + 4096);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rotate_quant_wide_kernel<B, WEIGHT, QB>), dim3((unsigned)a.rows_alloc, (unsigned)a.batch),
                       dim3(T), lds, stream, a.X, a.ldx, a.perm, a.rows_valid, a.rows_alloc, a.K, 1, a.alpha,
                       a.alpha_dev, a.post_scale, a.out, a.scale, a.out_stride, a.scale_stride);
    return hipGetLastError();
}

// Few long rows: up to this many take one workgroup each as well.  A lane of the
// kernel above works through 32 or 64 values of four rows, whose latency is all
// there is to a launch that leaves compute units idle; one Hadamard block a lane
// is shorter while every row has a compute unit of its own, the more so the
// smaller the block and the dearer the codes.  Measured on either side (us, one
// workgroup a row / four rows): 64 x 16384, b = 32: 4.6 / 6.2, fp6 codes 4.9 / 7.4;
// 256 rows 6.0 / 6.3, fp6 6.3 / 6.9, int8 7.5 / 6.4; 64 x 9216, b = 64: 4.6 / 5.5,
// 384 rows 6.7 / 5.8; 64 x 9216, b = 128: 6.2 / 5.9; 64 x 4608, b = 32: 3.5 / 3.7, 384
// rows 4.4 / 3.9, gathered 1.03 times the four rows' time, at 8192 columns 0.88.
template <int B, int QB>
int few_rows(int K, bool gather) {
    if (K > 8 * kMaxLanes) {   // two chunks a lane
        if (B == 128) return QB == 6 && !gather && K > 12288 ? 64 : 0;
        if (B == 64) return (QB == 8 ? 128 : 192) - 64 * gather;
        return QB == 8 ? 128 : QB == 4 && gather ? 192 : 256;
    }
    if (B != 32 || K <= (gather && QB != 6 ? 6144 : 4096)) return 0;
    return QB == 8 || gather ? 128 : 192;
}

// Two or more rounds of a batch per compute unit, five sixths full (4864 columns,
// cached, four rows a lane / batches: 2560 rows, 1.25 rounds, 10.1 / 11.2; 3700, 1.8,
// 15.4 / 13.1; 5000, 2.4, 17.6 / 17.7; 6000, 2.9, 21.0 / 18.6).
bool rows8_fills(int64_t batches, int64_t cus) {
    const int64_t rounds = (batches + cus - 1) / cus;
    return rounds >= 2 && 6 * batches >= 5 * rounds * cus;
}

hipError_t launch_rq_rows8_f6(const RqArgs &a, hipStream_t stream) {
    const int T = (kRows8 * (a.K / 64) + 63) / 64 * 64;
    const size_t lds = (size_t)kRows8 * a.K * 2 + 2 * kRows8 * 4;
    if (T > kRows8Lanes || lds > kLdsLimit) return hipErrorInvalidConfiguration;
    hipError_t e = hipFuncSetAttribute((const void *)rotate_quant_rows8_f6_kernel,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
    if (e != hipSuccess) return e;
    const int64_t nbatch = (a.rows_alloc + kRows8 - 1) / kRows8;
    hipLaunchKernelGGL(rotate_quant_rows8_f6_kernel, dim3((unsigned)std::min<int64_t>(nbatch, compute_units())), dim3(T), lds,
                       stream, a.X, a.ldx, a.rows_valid, a.rows_alloc, nbatch, a.K, a.out, a.scale);
    return hipGetLastError();
}

template <int B, int QB, bool WEIGHT>
hipError_t launch_rq_width(const RqArgs &a, hipStream_t stream) {
    // (32-bit offsets within a batch)
    if constexpr (B == 64 && QB == 6 && !WEIGHT)
        if (a.perm == nullptr && a.K > 4096 && a.K <= 64 * (kRows8Lanes / kRows8) && a.K != 8 * 9 * 64 &&
            kRows8 * a.ldx <= INT32_MAX && rows8_fills(a.rows_alloc / kRows8, compute_units()))
            return launch_rq_rows8_f6(a, stream);
    if (a.batch == 1 && a.rows_alloc <= few_rows<B, QB>(a.K, a.perm != nullptr))
        return launch_rq_wide<B, QB, WEIGHT>(a, stream);
    if (a.K <= 8 * kMaxLanes) return launch_rq<B, QB, WEIGHT, 1>(a, stream);
    if (a.K <= 16 * kMaxLanes) return launch_rq<B, QB, WEIGHT, 2>(a, stream);
    return launch_rq_wide<B, QB, WEIGHT>(a, stream);
}

template <int B>
hipError_t launch_rq_block(const RqArgs &a, int bits, bool weight, hipStream_t stream) {
    switch (bits) {
        case 4: return weight ? launch_rq_width<B, 4, true>(a, stream) : launch_rq_width<B, 4, false>(a, stream);
        case 6: return weight ? launch_rq_width<B, 6, true>(a, stream) : launch_rq_width<B, 6, false>(a, stream);
        case 8: return weight ? launch_rq_width<B, 8, true>(a, stream) : launch_rq_width<B, 8, false>(a, stream);
    }
    return hipErrorInvalidValue;
}

__global__ void unswizzle_kernel(const uint8_t *__restrict__ Wq, int64_t N, int K,
                                 uint8_t *__restrict__ out) {
    const int64_t kgs = K / 16;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * kgs) return;
    const int64_t n = idx / kgs, kg = idx - n * kgs;
    const uint2 v = *reinterpret_cast<const uint2 *>(Wq + wq_piece_offset(n, kg, K));
    *reinterpret_cast<uint2 *>(out + n * (K / 2) + kg * 8) = v;
}

__global__ void unswizzle_act_kernel(const uint8_t *__restrict__ Xq, int64_t M, int K,
                                     uint8_t *__restrict__ out) {
    const int64_t cpr = K / 32;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= M * cpr) return;
    const int64_t r = idx / cpr, c = idx - r * cpr;
    const uint4 v = *reinterpret_cast<const uint4 *>(Xq + xq_chunk_offset(r, c, K));
    *reinterpret_cast<uint4 *>(out + r * (K / 2) + c * 16) = v;
}

// one 16-byte operand piece per thread, scattered back to canonical codes
__global__ void unswizzle8_kernel(const uint8_t *__restrict__ q8, int64_t rows, int K, bool weights,
                                  int8_t *__restrict__ out) {
    const int64_t cpr = K / 32;   // 32-code chunks per row
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * cpr * 2) return;
    const int q = (int)(idx & 1);
    const int64_t rc = idx >> 1, r = rc / cpr, c = rc - r * cpr;
    const int rho = weights ? wq_rho((int)(r & 31)) : (int)(r & 31);
    const uint4 v = *reinterpret_cast<const uint4 *>(q8 + q8_piece_offset(r >> 5, rho, c, q, K));
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    int8_t *dst = out + r * K + c * 32 + q * 16;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int byte = (t & 1) * 8 + (t >> 1);
        dst[t] = (int8_t)(w[byte >> 2] >> (8 * (byte & 3)));
    }
}

}  // namespace

hipError_t launch_unswizzle8(const uint8_t *q8, int64_t rows, int K, bool weights, int8_t *out,
                             hipStream_t stream) {
    const int64_t total = rows * (K / 32) * 2;
    hipLaunchKernelGGL(unswizzle8_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       q8, rows, K, weights, out);
    return hipGetLastError();
}

hipError_t launch_rotate_quant(const uint16_t *X, int64_t ldx, const int32_t *perm,
                               int64_t rows, int64_t rows_alloc, int K, int block,
                               float alpha, bool weight_mode, float post_scale,
                               uint8_t *out, float *scale, hipStream_t stream, int bits,
                               const float *alpha_dev, int batch, int64_t out_stride, int64_t scale_stride) {
    if (batch > 1 && (!weight_mode || alpha_dev == nullptr || bits != 4)) return hipErrorInvalidValue;
    RqArgs a{};
    a.X = X;
    a.ldx = ldx;
    a.perm = perm;
    a.rows_valid = rows;
    a.rows_alloc = rows_alloc;
    a.K = K;
    a.alpha = alpha;
    a.alpha_dev = alpha_dev;
    a.post_scale = post_scale;
    a.out = out;
    a.scale = scale;
    a.batch = batch;
    a.out_stride = out_stride;
    a.scale_stride = scale_stride;
    switch (block) {
        case 32: return launch_rq_block<32>(a, bits, weight_mode, stream);
        case 64: return launch_rq_block<64>(a, bits, weight_mode, stream);
        case 128: return launch_rq_block<128>(a, bits, weight_mode, stream);
    }
    return hipErrorInvalidValue;
}

namespace {

// canonical packed int4 codes [rows][K/2] of an fp6 operand (weights: the
// fragment-row order undone): one thread per 32-code chunk
__global__ void unswizzle_f6_kernel(const uint8_t *__restrict__ q6, int64_t rows, int K, bool weights,
                                    uint8_t *__restrict__ out) {
    const int64_t cpr = K / 32;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * cpr) return;
    const int64_t r = idx / cpr, c32 = idx - r * cpr;
    const int rho = weights ? wq_rho((int)(r & 31)) : (int)(r & 31);
    const uint8_t *unit = q6 + f6_unit_offset(r >> 5, c32, K);
    const int l = f6_lane(c32, rho);
    const uint4 a = *reinterpret_cast<const uint4 *>(unit + l * 16);
    const uint2 b = *reinterpret_cast<const uint2 *>(unit + f6_tail_offset(l));
    const uint32_t w[6] = {a.x, a.y, a.z, a.w, b.x, b.y};
    uint32_t d[4];
    nibbles_from_f6(w, d);
    *reinterpret_cast<uint4 *>(out + r * (K / 2) + c32 * 16) = make_uint4(d[0], d[1], d[2], d[3]);
}

}  // namespace

hipError_t launch_unswizzle_f6(const uint8_t *q6, int64_t rows, int K, bool weights, uint8_t *out,
                               hipStream_t stream) {
    const int64_t total = rows * (K / 32);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(unswizzle_f6_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, q6, rows, K,
                       weights, out);
    return hipGetLastError();
}

hipError_t launch_unswizzle(const uint8_t *Wq, int64_t N, int K, uint8_t *out,
                            hipStream_t stream) {
    const int64_t total = N * (K / 16);
    const int64_t grid = (total + 255) / 256;
    hipLaunchKernelGGL(unswizzle_kernel, dim3((unsigned)grid), dim3(256), 0, stream, Wq, N, K, out);
    return hipGetLastError();
}

hipError_t launch_unswizzle_act(const uint8_t *Xq, int64_t M, int K, uint8_t *out,
                                hipStream_t stream) {
    const int64_t total = M * (K / 32);
    const int64_t grid = (total + 255) / 256;
    hipLaunchKernelGGL(unswizzle_act_kernel, dim3((unsigned)grid), dim3(256), 0, stream, Xq, M, K, out);
    return hipGetLastError();
}

}  // namespace clq
