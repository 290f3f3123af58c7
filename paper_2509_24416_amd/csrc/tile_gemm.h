// One-tile-per-workgroup GEMM shared by the code storages (CLQ, arXiv
// 2509.24416: the product of the quantized codes with the dequantising
// epilogue of Eq. (1) fused; Sec. 4.1's W4A4, W4A8 and W8A8 settings).
//
// A workgroup of WM waves computes 128 channels x 64 WM tokens, each wave 128
// channels x 64 tokens (4 x 2 fragments of 32 x 32, 128 accumulator
// registers).  A k-stage is 64 codes.  Operand units go global -> LDS
// (global_load_lds, no registers) through a ring of NS stages; each wave reads
// a stage's units back one stage ahead of its use, into the register set that
// the matrix instructions do not read, and 4-bit operands are widened fragment
// by fragment right before their matrix instructions, so that only one
// fragment of widened operands is live.
//
// What bounds it: the k loop's matrix instructions (16 per wave and stage of
// 32 cycles each on the int8 path) share their issue port with the loop's
// other vector instructions (72 for widening), so the loop has nothing else in
// it: ring slots are scalar offsets, there is no test but the loop's own, and
// transfers past the end repeat the last stage so that the wait counts stay
// constant.  Two workgroups share a compute unit, so that one's prologue and
// epilogue run under the other's k loop.
//
// Ring protocol: iteration s waits until stage s + 1 has landed (transfers
// complete in issue order: at most the NS - 2 later stages' may be
// outstanding) and until its own LDS reads of stage s are in, then the
// workgroup barrier: every wave holds stage s in registers, so its slot is
// refilled with stage s + NS, and stage s + 1 is read.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "clq_internal.h"
#include "f6_codes.h"

#ifndef CLQ_LDS
#define CLQ_LDS __attribute__((address_space(3)))
#endif

namespace clq {
namespace {
namespace tg {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
template <int Q> using IC = std::integral_constant<int, Q>;

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(IC<I>{});
        static_for<I + 1, N>(f);
    }
}
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return (uint32_t)reinterpret_cast<size_t>((CLQ_LDS const void *)p);
}
// (plain functions: the builtin's operands must not depend on a template
// parameter in the host compilation pass)
__device__ __forceinline__ void dma16(const uint8_t *src, uint32_t dst) {
    __builtin_amdgcn_global_load_lds(src, (CLQ_LDS void *)(size_t)dst, 16, 0, 0);
}
// LDS reads are asm: the compiler would otherwise wait for every transfer in
// flight before them.  Their wait names the destination registers.
template <int OFF>
__device__ __forceinline__ v4u read16(uint32_t addr) {
    v4u v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ v2u read8(uint32_t addr) {
    v2u v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
// 16 int4 codes (two dwords) -> 16 int8 holding 16 q: even codes, then odd
__device__ __forceinline__ v4i widen16(uint32_t d0, uint32_t d1) {
    return v4i{(int)((d0 << 4) & 0xF0F0F0F0u), (int)((d1 << 4) & 0xF0F0F0F0u),
               (int)(d0 & 0xF0F0F0F0u), (int)(d1 & 0xF0F0F0F0u)};
}
// two fp16 outputs fma(p, w, b), each rounded once (the same instruction in
// every GEMM of the library, so that all schedules give the same bits)
__device__ __forceinline__ uint32_t fma_mix2f(float p0, float w0, float b0, float p1, float w1, float b1) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, %6"
        : "=&v"(r)
        : "v"(p0), "v"(w0), "v"(b0), "v"(p1), "v"(w1), "v"(b1));
    return r;
}

// the same with the biases as a packed fp16 pair (low half: first output)
__device__ __forceinline__ uint32_t fma_mix2(float p0, float w0, float p1, float w1, uint32_t b) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[0,0,1]\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, %3 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
        : "=&v"(r)
        : "v"(p0), "v"(w0), "v"(b), "v"(p1), "v"(w1));
    return r;
}

// Code storages: bytes of a 32 x 64 unit, and the factor by which the
// accumulator exceeds the sum of code products (a power of two).
enum class Fmt { W4A4, F6, W4A8, W8A8 };
template <Fmt F> struct FmtInfo;
template <> struct FmtInfo<Fmt::W4A4> { static constexpr int WU = 1024, XU = 1024, LOG = 8; };
template <> struct FmtInfo<Fmt::F6> { static constexpr int WU = kF6Unit, XU = kF6Unit, LOG = 0; };
template <> struct FmtInfo<Fmt::W4A8> { static constexpr int WU = 1024, XU = 2048, LOG = 4; };
template <> struct FmtInfo<Fmt::W8A8> { static constexpr int WU = 2048, XU = 2048, LOG = 0; };

template <Fmt F, int WM_, int NS_>
struct Cfg {
    static constexpr Fmt fmt = F;
    static constexpr int WM = WM_, NS = NS_, FN = 4, FM = 2;
    static constexpr int NT = WM * 64, BN = 128, BM = WM * 64;
    static constexpr int WU = FmtInfo<F>::WU, XU = FmtInfo<F>::XU;
    static constexpr int W_UNITS = BN / 32, X_UNITS = BM / 32;
    static constexpr int W_BYTES = W_UNITS * WU, STAGE = W_BYTES + X_UNITS * XU;
    // transfers of 1 KB (fp6: a 1 KB and a 512-byte one per unit)
    static constexpr int PIECES = F == Fmt::F6 ? 2 * (W_UNITS + X_UNITS) : STAGE / 1024;
    static constexpr int PPW = PIECES / WM;
    static_assert(PIECES % WM == 0, "transfers split evenly over waves");
    static constexpr int EPN = 2 * BN + BM;   // epilogue operands (floats)
    static constexpr int POOL = NS * STAGE;
};

struct Args {
    const uint8_t *Xq;
    const float *xs;
    const uint8_t *Wq;
    const float *ws;
    const uint16_t *bias;
    void *Y;
    int64_t ldy;
    int M, N, K, tiles_m, tiles_n;
    int group_m;   // token panels per tile group
    // squared-error mode: fp32 target [M][ldy0]; nc candidate weights (codes
    // and scales at strides wq_stride bytes, ws_stride floats); one fp64 partial
    // per wave of every tile, candidate c's at errp + c * p_stride
    const float *y0;
    int64_t ldy0;
    double *errp;
    int nc;
    int64_t wq_stride, ws_stride, p_stride;
};

// a stage's operands of one wave: 4 channel units, 2 token units.  read: from
// the units' LDS addresses (wa, xa: of lane 0's bytes); wait<VM>: at most VM
// transfers outstanding and the reads in, then the workgroup barrier; load:
// straight from memory, stage k of the units at ws and xs.
#define CLQ_STAGE_WAIT "s_waitcnt vmcnt(%c[vm]) lgkmcnt(0)\n\ts_barrier"
template <Fmt F> struct Operands;
template <> struct Operands<Fmt::W4A4> {
    v4u w[4], x[2];
    __device__ __forceinline__ void read(uint32_t wa, uint32_t xa, int lane) {
        const uint32_t wl = wa + lane * 16, xl = xa + lane * 16;
        static_for<0, 4>([&](auto f) { w[f] = read16<decltype(f)::value * 1024>(wl); });
        static_for<0, 2>([&](auto f) { x[f] = read16<decltype(f)::value * 1024>(xl); });
    }
    __device__ __forceinline__ void load(const uint8_t *const (&ws)[4], const uint8_t *const (&xs)[2], int k, int lane) {
        const uint32_t off = (uint32_t)(k * 1024 + lane * 16);
#pragma unroll
        for (int f = 0; f < 4; ++f) w[f] = *reinterpret_cast<const v4u *>(ws[f] + off);
#pragma unroll
        for (int f = 0; f < 2; ++f) x[f] = *reinterpret_cast<const v4u *>(xs[f] + off);
    }
    template <int VM>
    __device__ __forceinline__ void wait() {
        asm volatile(CLQ_STAGE_WAIT
                     : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(x[0]), "+v"(x[1])
                     : [vm] "n"(VM)
                     : "memory");
    }
};
template <> struct Operands<Fmt::F6> {
    v4u w[4], x[2];
    v2u wt[4], xt[2];
    __device__ __forceinline__ void read(uint32_t wa, uint32_t xa, int lane) {
        const uint32_t wl = wa + lane * 16, xl = xa + lane * 16, to = f6_tail_offset(lane);
        const uint32_t wtl = wa + to, xtl = xa + to;
        static_for<0, 4>([&](auto f) {
            w[f] = read16<decltype(f)::value * kF6Unit>(wl);
            wt[f] = read8<decltype(f)::value * kF6Unit>(wtl);
        });
        static_for<0, 2>([&](auto f) {
            x[f] = read16<decltype(f)::value * kF6Unit>(xl);
            xt[f] = read8<decltype(f)::value * kF6Unit>(xtl);
        });
    }
    __device__ __forceinline__ void load(const uint8_t *const (&ws)[4], const uint8_t *const (&xs)[2], int k, int lane) {
        const uint32_t off = (uint32_t)(k * kF6Unit + lane * 16), to = (uint32_t)(k * kF6Unit + f6_tail_offset(lane));
        static_for<0, 4>([&](auto f) {
            w[f] = *reinterpret_cast<const v4u *>(ws[f] + off);
            wt[f] = *reinterpret_cast<const v2u *>(ws[f] + to);
        });
        static_for<0, 2>([&](auto f) {
            x[f] = *reinterpret_cast<const v4u *>(xs[f] + off);
            xt[f] = *reinterpret_cast<const v2u *>(xs[f] + to);
        });
    }
    template <int VM>
    __device__ __forceinline__ void wait() {
        asm volatile(CLQ_STAGE_WAIT
                     : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(x[0]), "+v"(x[1]), "+v"(wt[0]),
                       "+v"(wt[1]), "+v"(wt[2]), "+v"(wt[3]), "+v"(xt[0]), "+v"(xt[1])
                     : [vm] "n"(VM)
                     : "memory");
    }
};
template <> struct Operands<Fmt::W4A8> {
    v4u w[4], x[2][2];
    __device__ __forceinline__ void read(uint32_t wa, uint32_t xa, int lane) {
        const uint32_t wl = wa + lane * 16, xl = xa + lane * 16;
        static_for<0, 4>([&](auto f) { w[f] = read16<decltype(f)::value * 1024>(wl); });
        static_for<0, 4>([&](auto f) {
            x[decltype(f)::value >> 1][decltype(f)::value & 1] = read16<decltype(f)::value * 1024>(xl);
        });
    }
    __device__ __forceinline__ void load(const uint8_t *const (&ws)[4], const uint8_t *const (&xs)[2], int k, int lane) {
        const uint32_t off = (uint32_t)(k * 1024 + lane * 16), xoff = (uint32_t)(k * 2048 + lane * 16);
#pragma unroll
        for (int f = 0; f < 4; ++f) w[f] = *reinterpret_cast<const v4u *>(ws[f] + off);
#pragma unroll
        for (int f = 0; f < 4; ++f) x[f >> 1][f & 1] = *reinterpret_cast<const v4u *>(xs[f >> 1] + xoff + (f & 1) * 1024);
    }
    template <int VM>
    __device__ __forceinline__ void wait() {
        asm volatile(CLQ_STAGE_WAIT
                     : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[1][0]),
                       "+v"(x[1][1])
                     : [vm] "n"(VM)
                     : "memory");
    }
};
template <> struct Operands<Fmt::W8A8> {
    v4u w[4][2], x[2][2];
    __device__ __forceinline__ void read(uint32_t wa, uint32_t xa, int lane) {
        const uint32_t wl = wa + lane * 16, xl = xa + lane * 16;
        static_for<0, 8>([&](auto f) {
            w[decltype(f)::value >> 1][decltype(f)::value & 1] = read16<decltype(f)::value * 1024>(wl);
        });
        static_for<0, 4>([&](auto f) {
            x[decltype(f)::value >> 1][decltype(f)::value & 1] = read16<decltype(f)::value * 1024>(xl);
        });
    }
    __device__ __forceinline__ void load(const uint8_t *const (&ws)[4], const uint8_t *const (&xs)[2], int k, int lane) {
        const uint32_t off = (uint32_t)(k * 2048 + lane * 16);
#pragma unroll
        for (int f = 0; f < 8; ++f) w[f >> 1][f & 1] = *reinterpret_cast<const v4u *>(ws[f >> 1] + off + (f & 1) * 1024);
#pragma unroll
        for (int f = 0; f < 4; ++f) x[f >> 1][f & 1] = *reinterpret_cast<const v4u *>(xs[f >> 1] + off + (f & 1) * 1024);
    }
    template <int VM>
    __device__ __forceinline__ void wait() {
        asm volatile(CLQ_STAGE_WAIT
                     : "+v"(w[0][0]), "+v"(w[1][0]), "+v"(w[2][0]), "+v"(w[3][0]), "+v"(w[0][1]), "+v"(w[1][1]),
                       "+v"(w[2][1]), "+v"(w[3][1]), "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[1][0]), "+v"(x[1][1])
                     : [vm] "n"(VM)
                     : "memory");
    }
};
#undef CLQ_STAGE_WAIT

template <Fmt F> using Acc = std::conditional_t<F == Fmt::F6, v16f, v16i>;
// the matrix work of one stage on the int8 instruction: 4 x 2 fragments
template <Fmt F>
__device__ __forceinline__ void stage_mma(const Operands<F> &o, Acc<F> (&acc)[4][2]) {
    // two 32-code halves
    static_for<0, 2>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        v4i b[2];
#pragma unroll
        for (int fm = 0; fm < 2; ++fm) {
            if constexpr (F == Fmt::W4A4) b[fm] = widen16(o.x[fm][2 * h], o.x[fm][2 * h + 1]);
            else b[fm] = __builtin_bit_cast(v4i, o.x[fm][h]);
        }
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) {
            v4i w;
            if constexpr (F == Fmt::W8A8) w = __builtin_bit_cast(v4i, o.w[fn][h]);
            else w = widen16(o.w[fn][2 * h], o.w[fn][2 * h + 1]);
#pragma unroll
            for (int fm = 0; fm < 2; ++fm)
                acc[fn][fm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, b[fm], acc[fn][fm], 0, 0, 0);
        }
    });
}

// the same on the fp6 instruction, one per fragment and stage (format codes 2,
// 2: both operands e2m3, no block scales).  Written where it is used: behind a
// function's reference parameter the compiler keeps the operands in memory.
#define CLQ_STAGE_MMA_F6(o, acc)                                                                                     \
    v8i b6[2];                                                                                                       \
    _Pragma("unroll") for (int fm = 0; fm < 2; ++fm) b6[fm] =                                                        \
        v8i{(int)o.x[fm][0], (int)o.x[fm][1], (int)o.x[fm][2], (int)o.x[fm][3], (int)o.xt[fm][0], (int)o.xt[fm][1], 0, 0}; \
    _Pragma("unroll") for (int fn = 0; fn < 4; ++fn) {                                                               \
        const v8i w6 = v8i{(int)o.w[fn][0], (int)o.w[fn][1], (int)o.w[fn][2], (int)o.w[fn][3], (int)o.wt[fn][0],     \
                           (int)o.wt[fn][1], 0, 0};                                                                  \
        _Pragma("unroll") for (int fm = 0; fm < 2; ++fm)                                                             \
            acc[fn][fm] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w6, b6[fm], acc[fn][fm], 2, 2, 0, 0, 0, 0); \
    }

// the epilogue of one 32 x 32 fragment: the lane's 16 channels n0 .. n0 + 15 of
// token m.  ep: channel scales, biases (floats), token scales of the tile; c0,
// r0: the channel and token inside the tile.
template <Fmt F, int BN, bool I32OUT, bool RAGGED, bool BIAS>
__device__ __forceinline__ void store_fragment(const Args &a, const Acc<F> &x, const float *ep, int c0, int r0, int n0,
                                               int m) {
    constexpr int LOG = FmtInfo<F>::LOG;
    if (m >= a.M || n0 >= a.N) return;
    if constexpr (I32OUT) {
        int32_t s[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = (int)x[v] >> LOG;
        int32_t *dst = reinterpret_cast<int32_t *>(a.Y) + (int64_t)m * a.ldy + n0;
        if constexpr (!RAGGED) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                reinterpret_cast<v4i *>(dst)[q] = v4i{s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]};
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (n0 + v < a.N) dst[v] = s[v];
        }
    } else {
        const float xsc = ep[2 * BN + r0] * (1.0f / (float)(1 << LOG));
        uint32_t hv[8];
#pragma unroll
        for (int v = 0; v < 16; v += 2)
            hv[v / 2] = fma_mix2f((float)x[v] * xsc, ep[c0 + v], BIAS ? ep[BN + c0 + v] : 0.0f, (float)x[v + 1] * xsc,
                                  ep[c0 + v + 1], BIAS ? ep[BN + c0 + v + 1] : 0.0f);
        uint16_t *dst = reinterpret_cast<uint16_t *>(a.Y) + (int64_t)m * a.ldy + n0;
        if (!RAGGED || n0 <= a.N - 16) {
            reinterpret_cast<v4u *>(dst)[0] = v4u{hv[0], hv[1], hv[2], hv[3]};
            reinterpret_cast<v4u *>(dst)[1] = v4u{hv[4], hv[5], hv[6], hv[7]};
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (n0 + v < a.N) dst[v] = (uint16_t)(hv[v >> 1] >> (16 * (v & 1)));
        }
    }
}

// Tile number of this workgroup: workgroups are dealt to the 8 XCDs
// round-robin, and each XCD takes a contiguous run.
__device__ __forceinline__ int tile_of_block() {
    const int G = gridDim.x, x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int per = G >> 3, rem = G & 7;
    return x * per + min(x, rem) + j;
}
// Its place, in the grouped order (group_m token panels at a time) whose panels
// an XCD's L2 holds.
__device__ __forceinline__ void tile_coords(const Args &a, int L, int &tm, int &tn) {
    const int gsz = a.group_m * a.tiles_n;
    const int g = L / gsz, r = L - g * gsz;
    const int m0 = g * a.group_m;
    const int gm = min(a.tiles_m - m0, a.group_m);
    tn = r / gm;
    tm = m0 + (r - tn * gm);
}

// Epilogue operands of a tile (channel scales, biases, token scales), spread
// over the NT threads of the workgroup: loaded early at clamped indices,
// without branches or conversions that would wait for them, and written to LDS
// as floats after the k loop.
template <int BN, int BM, int NT, bool BIAS>
struct EpilogueOperands {
    static constexpr int EPN = 2 * BN + BM, EPR = (EPN + NT - 1) / NT;
    float v[EPR];
    _Float16 b[EPR];
    __device__ __forceinline__ void load(const Args &a, int tm, int tn, int tid) {
#pragma unroll
        for (int r = 0; r < EPR; ++r) {
            const int e = min(tid + r * NT, EPN - 1);
            const int ec = min(tn * BN + (e & (BN - 1)), a.N - 1), er = min(tm * BM + max(e - 2 * BN, 0), a.M - 1);
            const float *p = e < 2 * BN ? a.ws + ec : a.xs + er;
            v[r] = *p;
            if constexpr (BIAS) b[r] = reinterpret_cast<const _Float16 *>(a.bias)[ec];
        }
    }
    __device__ __forceinline__ void store(float *ep, int tid) const {
#pragma unroll
        for (int r = 0; r < EPR; ++r) {
            const int e = min(tid + r * NT, EPN - 1);
            float t = v[r];
            if constexpr (BIAS) t = e >= BN && e < 2 * BN ? (float)b[r] : t;
            ep[e] = t;
        }
    }
};

// ERR: nothing is stored; the epilogue sums (Y0 - sum * x_scale * w_scale)^2
// over the tile in fp64 (the integer sum exact) and keeps one partial per wave.
// A target tile's candidates are neighbours in the tile order, so that one
// XCD's L2 serves the target and the activation panel to all of them.
template <class C, bool I32OUT, bool RAGGED, bool BIAS, bool ERR = false>
__global__ void __launch_bounds__(C::NT, 2) tile_gemm_kernel(Args a)
{
    static_assert(!(I32OUT && BIAS), "no bias on the integer output");
    static_assert(!ERR || (!I32OUT && !BIAS), "the error mode has no output and no bias");
    constexpr Fmt F = C::fmt;
    constexpr int NS = C::NS;
    __shared__ __align__(16) uint8_t pool[C::POOL];
    __shared__ float ep[C::EPN];   // channel scales, biases (fp16 widened), token scales
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, N = a.N, nks = a.K >> 6;

    int tm, tn, cand = 0, tile = tile_of_block();
    if constexpr (ERR) {
        const int t = tile / a.nc;
        cand = tile - t * a.nc;
        tile = t;
        a.Wq += cand * a.wq_stride;
        a.ws += cand * a.ws_stride;
    }
    tile_coords(a, tile, tm, tn);
    const int wunits = (int)(padded_rows(N) >> 5), xunits = (int)(padded_act_rows(M) >> 5);

    // ---- producer: this wave's transfers of a stage ---------------------------
    const uint8_t *src[C::PPW];
    uint32_t dsto[C::PPW];
    constexpr bool kTwoSteps = C::WU != C::XU;   // bytes per stage differ between the operands
    bool wpiece[C::PPW];
    static_for<0, C::PPW>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (F == Fmt::F6) {
            // units first their 1 KB, then (i >= PPW / 2) their 512 bytes
            constexpr int half = C::PPW / 2;
            const int u = wave * half + i % half;
            const uint8_t *base = u < C::W_UNITS
                                      ? a.Wq + (int64_t)min(tn * C::W_UNITS + u, wunits - 1) * nks * C::WU
                                      : a.Xq + (int64_t)min(tm * C::X_UNITS + u - C::W_UNITS, xunits - 1) * nks * C::XU;
            src[i] = base + (i >= half ? 1024 : 0);
            dsto[i] = (uint32_t)(u * kF6Unit + (i >= half ? 1024 : 0));
            wpiece[i] = true;
        } else {
            const int p = wave * C::PPW + i;   // 1 KB pieces, channel units first
            wpiece[i] = p < C::W_BYTES / 1024;
            if (wpiece[i]) {
                constexpr int per = C::WU / 1024;
                src[i] = a.Wq + (int64_t)min(tn * C::W_UNITS + p / per, wunits - 1) * nks * C::WU + (p % per) * 1024;
            } else {
                constexpr int per = C::XU / 1024;
                const int px = p - C::W_BYTES / 1024;
                src[i] = a.Xq + (int64_t)min(tm * C::X_UNITS + px / per, xunits - 1) * nks * C::XU + (px % per) * 1024;
            }
            dsto[i] = (uint32_t)(p * 1024);
        }
    });
    const uint32_t pool0 = lds_addr(pool), l16 = (uint32_t)lane * 16;
    // stage k into the slot at byte offset `slot`
    auto produce = [&](uint32_t slot, int k) __attribute__((always_inline)) {
        const int kc = min(k, nks - 1);
        const uint32_t vw = l16 + (uint32_t)(kc * C::WU), vx = l16 + (uint32_t)(kc * C::XU);
        const uint32_t d0 = pool0 + slot;
        if constexpr (F == Fmt::F6) {
            static_for<0, C::PPW / 2>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const uint8_t *sp = src[i] + vw;
                dma16(sp, d0 + dsto[i]);
            });
            if (lane < 32)
                static_for<C::PPW / 2, C::PPW>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const uint8_t *sp = src[i] + vw;
                    dma16(sp, d0 + dsto[i]);
                });
        } else {
            static_for<0, C::PPW>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const uint8_t *sp = src[i] + (!kTwoSteps || wpiece[i] ? vw : vx);
                dma16(sp, d0 + dsto[i]);
            });
        }
    };

    // ---- epilogue operands: loaded ahead of the transfers, held in registers
    // through the k loop, written to LDS after it (an LDS store while transfers
    // into LDS are in flight would wait for all of them)
    EpilogueOperands<C::BN, C::BM, C::NT, BIAS> eo;
    if constexpr (!I32OUT) eo.load(a, tm, tn, tid);
    __builtin_amdgcn_sched_barrier(0);

    // ---- consumer ---------------------------------------------------------------
    Operands<F> op[2];
    const uint32_t xo = (uint32_t)(C::W_BYTES + wave * 2 * C::XU);
    auto read_stage = [&](uint32_t slot, auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        op[P].read(pool0 + slot, pool0 + slot + xo, lane);
    };
    Acc<F> acc[C::FN][C::FM];
    static_for<0, C::FN>([&](auto fn) {
        static_for<0, C::FM>([&](auto fm) { acc[decltype(fn)::value][decltype(fm)::value] = Acc<F>{}; });
    });
    auto mma = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        if constexpr (F == Fmt::F6) {
            CLQ_STAGE_MMA_F6(op[P], acc)
        } else {
            stage_mma<F>(op[P], acc);
        }
    };
    // prologue: stages 0 .. NS - 1 in flight, stage 0 landed and being read
    static_for<0, NS>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        produce(q * C::STAGE, q);
    });
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * C::PPW) : "memory");
    read_stage(0, IC<0>{});
    uint32_t cur = 0;   // slot of the current stage
    int k = 0;
    auto stage = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        op[P].template wait<(NS - 2) * C::PPW>();
        const uint32_t nxt = cur == (uint32_t)((NS - 1) * C::STAGE) ? 0u : cur + C::STAGE;
        read_stage(nxt, IC<1 - P>{});
        produce(cur, k + NS);
        mma(pc);
        cur = nxt;
        ++k;
    };
    for (int pairs = nks >> 1; pairs > 0; --pairs) {
        stage(IC<0>{});
        stage(IC<1>{});
    }
    if (nks & 1) stage(IC<0>{});
    // drain: the last transfers, and the last read, whose data is not used: both
    // register sets are named here, so that none of their registers can serve
    // another value while that read is still in flight
    op[0].template wait<0>();
    op[1].template wait<0>();
    if constexpr (!I32OUT) {
        eo.store(ep, tid);
        __syncthreads();
    }

    // ---- epilogue: lane owns token m and 16 consecutive channels ----------------
    const int h16 = (lane >> 5) * 16;
    if constexpr (ERR) {
        // the target of each fragment is loaded two fragments ahead of its use
        // (rows and columns past the edge read a clamped address and their
        // terms are left out)
        float yv[3][16];
        auto load_target = [&](auto sc) __attribute__((always_inline)) {
            constexpr int q = decltype(sc)::value, fn = q / C::FM, fm = q % C::FM;
            const int n0 = tn * C::BN + fn * 32 + h16, m = tm * C::BM + (wave * C::FM + fm) * 32 + (lane & 31);
            const float *yr = a.y0 + (int64_t)min(m, M - 1) * a.ldy0;
            if constexpr (!RAGGED) {   // 16-byte aligned rows of whole 16-channel pieces
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const v4f t = reinterpret_cast<const v4f *>(yr + min(n0, N - 16))[q4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) yv[q % 3][4 * q4 + e] = t[e];
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) yv[q % 3][v] = yr[min(n0 + v, N - 1)];
            }
        };
        double esum = 0.0;
        load_target(IC<0>{});
        load_target(IC<1>{});
        static_for<0, C::FN * C::FM>([&](auto sc) {
            constexpr int q = decltype(sc)::value, fn = q / C::FM, fm = q % C::FM;
            if constexpr (q + 2 < C::FN * C::FM) load_target(IC<q + 2>{});
            __builtin_amdgcn_sched_barrier(0);
            const int c0 = fn * 32 + h16, n0 = tn * C::BN + c0, r0 = (wave * C::FM + fm) * 32 + (lane & 31);
            if (tm * C::BM + r0 < M && n0 < N) {
                // d = Y0 - (sum * x_scale) * w_scale; the accumulator is 2^LOG times the sum
                const double xm = (double)ep[2 * C::BN + r0] * (1.0 / (double)(1 << FmtInfo<F>::LOG));
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    if (RAGGED && n0 + v >= N) continue;
                    const double d = __builtin_fma(-((double)acc[fn][fm][v] * xm), (double)ep[c0 + v], (double)yv[q % 3][v]);
                    esum = __builtin_fma(d, d, esum);
                }
            }
        });
        // fixed butterfly over the wave; lane 0 holds the wave's partial
        for (int off = 32; off > 0; off >>= 1) esum += __shfl_xor(esum, off);
        if (lane == 0) a.errp[cand * a.p_stride + (int64_t)tile * C::WM + wave] = esum;
        return;
    }
    static_for<0, C::FN>([&](auto fc) {
        static_for<0, C::FM>([&](auto mc) {
            constexpr int fn = decltype(fc)::value, fm = decltype(mc)::value;
            const int c0 = fn * 32 + h16, r0 = (wave * C::FM + fm) * 32 + (lane & 31);
            store_fragment<F, C::BN, I32OUT, RAGGED, BIAS>(a, acc[fn][fm], ep, c0, r0, tn * C::BN + c0, tm * C::BM + r0);
        });
    });
}

// ---- few tiles: the k loop split over the waves of a workgroup -----------------
// With few tiles the kernel above leaves most SIMDs without a wave, and what it
// takes is the length of one wave's k loop plus fixed latencies.  Here KS waves
// share one 128 x 64 tile: wave w runs stages w nks / KS .. (w + 1) nks / KS of
// it.  No operand is shared between waves, so operands go straight from memory
// (L2) to registers, kDepth stages ahead, with no LDS ring and no barrier in
// the loop.  The sums (exact integers) then meet in LDS by recursive halving:
// in each step a wave sends half of its fragments to a partner and adds the
// partner's other half, 16 and 8 KB a wave for KS = 4, so that every wave ends
// with 8 / KS summed fragments and runs their epilogue.
template <Fmt F, int KS_>
struct SplitCfg {
    static constexpr Fmt fmt = F;
    static constexpr int KS = KS_, NT = KS * 64, BN = 128, BM = 64;
    static constexpr int WU = FmtInfo<F>::WU, XU = FmtInfo<F>::XU;
    static constexpr int kDepth = F == Fmt::W8A8 || F == Fmt::F6 ? 2 : 3;
    static constexpr int EPN = 2 * BN + BM;
    static_assert(KS == 2 || KS == 4, "recursive halving over 8 fragments");
};

template <class C, bool I32OUT, bool RAGGED, bool BIAS>
__global__ void __launch_bounds__(C::NT, 2) split_gemm_kernel(Args a)
{
    static_assert(!(I32OUT && BIAS), "no bias on the integer output");
    constexpr Fmt F = C::fmt;
    constexpr int KS = C::KS, D = C::kDepth;
    __shared__ __align__(16) uint8_t exch[KS * 16384];   // a step: 16 KB a wave at most
    __shared__ float ep[C::EPN];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nks = a.K >> 6;
    int tm, tn;
    tile_coords(a, tile_of_block(), tm, tn);
    const int wunits = (int)(padded_rows(a.N) >> 5), xunits = (int)(padded_act_rows(a.M) >> 5);
    const int kb = wave * nks / KS, ke = (wave + 1) * nks / KS;
    const uint8_t *ws[4], *xs[2];
#pragma unroll
    for (int f = 0; f < 4; ++f) ws[f] = a.Wq + (int64_t)min(tn * 4 + f, wunits - 1) * nks * C::WU;
#pragma unroll
    for (int f = 0; f < 2; ++f) xs[f] = a.Xq + (int64_t)min(tm * 2 + f, xunits - 1) * nks * C::XU;

    EpilogueOperands<C::BN, C::BM, C::NT, BIAS> eo;
    if constexpr (!I32OUT) eo.load(a, tm, tn, tid);
    __builtin_amdgcn_sched_barrier(0);

    Acc<F> acc[4][2];
    static_for<0, 4>([&](auto fn) {
        static_for<0, 2>([&](auto fm) { acc[decltype(fn)::value][decltype(fm)::value] = Acc<F>{}; });
    });
    Operands<F> op[D];
    const int last = ke - 1;   // (loads past the end repeat the last stage; nks >= KS, so ke > kb)
    static_for<0, D>([&](auto dc) {
        op[decltype(dc)::value].load(ws, xs, min(kb + decltype(dc)::value, last), lane);
        __builtin_amdgcn_sched_barrier(0);   // (the loop's waits rely on this order)
    });
    // whole groups of D stages, then the rest one by one: one loop with one
    // exit, so that the compiler's waits count only the loads that matter
    const int groups = (ke - kb) / D, rest = (ke - kb) - groups * D;
    int k = kb;
    auto mma = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        if constexpr (F == Fmt::F6) {
            CLQ_STAGE_MMA_F6(op[P], acc)
        } else {
            stage_mma<F>(op[P], acc);
        }
    };
    for (int g = 0; g < groups; ++g)
        static_for<0, D>([&](auto dc) {
            constexpr int d = decltype(dc)::value;
            mma(dc);
            op[d].load(ws, xs, min(k + D, last), lane);
            __builtin_amdgcn_sched_barrier(0);   // (the loads would otherwise sink to their uses)
            ++k;
        });
    if (rest > 0) mma(IC<0>{});
    if constexpr (D > 2)
        if (rest > 1) mma(IC<1>{});

    if constexpr (!I32OUT) eo.store(ep, tid);   // (the exchange's barriers publish it)

    // one step's messages: fragments [fn0, fn0 + nf) x [fm0, fm0 + mf)
    using V4 = std::conditional_t<F == Fmt::F6, v4f, v4i>;
    auto send = [&](auto fn0, auto nf, auto fm0, auto mf, int to) __attribute__((always_inline)) {
        V4 *out = reinterpret_cast<V4 *>(exch + to * 16384) + lane;
        static_for<0, decltype(nf)::value>([&](auto i) {
            static_for<0, decltype(mf)::value>([&](auto j) {
                const Acc<F> &x = acc[decltype(fn0)::value + decltype(i)::value][decltype(fm0)::value + decltype(j)::value];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    out[((decltype(i)::value * decltype(mf)::value + decltype(j)::value) * 4 + q) * 64] =
                        V4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
            });
        });
    };
    auto receive = [&](auto fn0, auto nf, auto fm0, auto mf) __attribute__((always_inline)) {
        const V4 *in = reinterpret_cast<const V4 *>(exch + wave * 16384) + lane;
        static_for<0, decltype(nf)::value>([&](auto i) {
            static_for<0, decltype(mf)::value>([&](auto j) {
                Acc<F> &x = acc[decltype(fn0)::value + decltype(i)::value][decltype(fm0)::value + decltype(j)::value];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const V4 t = in[((decltype(i)::value * decltype(mf)::value + decltype(j)::value) * 4 + q) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[4 * q + e] += t[e];
                }
            });
        });
    };
    const int h16 = (lane >> 5) * 16;
    // the wave's summed fragments [fn0, fn0 + nf) x [fm0, fm0 + mf)
    auto finish = [&](auto fn0, auto nf, auto fm0, auto mf) __attribute__((always_inline)) {
        static_for<0, decltype(nf)::value>([&](auto i) {
            static_for<0, decltype(mf)::value>([&](auto j) {
                constexpr int fn = decltype(fn0)::value + decltype(i)::value, fm = decltype(fm0)::value + decltype(j)::value;
                const int c0 = fn * 32 + h16, r0 = fm * 32 + (lane & 31);
                store_fragment<F, C::BN, I32OUT, RAGGED, BIAS>(a, acc[fn][fm], ep, c0, r0, tn * C::BN + c0,
                                                              tm * C::BM + r0);
            });
        });
    };
    // step 1 halves by token fragment, step 2 by channel fragments.  The partner of
    // a step differs in one bit of the wave number; the barrier before a step's
    // sends keeps them behind the last step's receives.
    auto step2 = [&](auto fm0) __attribute__((always_inline)) {
        constexpr IC<1> one{};
        constexpr IC<2> two{};
        if constexpr (KS == 4) {
            __syncthreads();
            if ((wave & 1) == 0) {
                send(two, two, fm0, one, wave ^ 1);
                __syncthreads();
                receive(IC<0>{}, two, fm0, one);
                finish(IC<0>{}, two, fm0, one);
            } else {
                send(IC<0>{}, two, fm0, one, wave ^ 1);
                __syncthreads();
                receive(two, two, fm0, one);
                finish(two, two, fm0, one);
            }
        } else {
            finish(IC<0>{}, IC<4>{}, fm0, one);
        }
    };
    constexpr int top = KS / 2;
    if ((wave & top) == 0) {
        send(IC<0>{}, IC<4>{}, IC<1>{}, IC<1>{}, wave ^ top);
        __syncthreads();
        receive(IC<0>{}, IC<4>{}, IC<0>{}, IC<1>{});
        step2(IC<0>{});
    } else {
        send(IC<0>{}, IC<4>{}, IC<0>{}, IC<1>{}, wave ^ top);
        __syncthreads();
        receive(IC<0>{}, IC<4>{}, IC<1>{}, IC<1>{});
        step2(IC<1>{});
    }
}

// (token and channel counts reach 2^31 - 1)
inline int64_t tile_count(int64_t rows, int64_t tile) { return (rows + tile - 1) / tile; }

template <class C>
hipError_t launch_split(Args a, bool i32out, bool ragged, hipStream_t stream) {
    a.tiles_m = (int)tile_count(a.M, C::BM);
    a.tiles_n = (int)tile_count(a.N, C::BN);
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n)), block(C::NT);
    if (i32out && ragged) hipLaunchKernelGGL((split_gemm_kernel<C, true, true, false>), grid, block, 0, stream, a);
    else if (i32out) hipLaunchKernelGGL((split_gemm_kernel<C, true, false, false>), grid, block, 0, stream, a);
    else if (a.bias && ragged) hipLaunchKernelGGL((split_gemm_kernel<C, false, true, true>), grid, block, 0, stream, a);
    else if (a.bias) hipLaunchKernelGGL((split_gemm_kernel<C, false, false, true>), grid, block, 0, stream, a);
    else if (ragged) hipLaunchKernelGGL((split_gemm_kernel<C, false, true, false>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((split_gemm_kernel<C, false, false, false>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <class C>
hipError_t launch(Args a, bool i32out, bool ragged, hipStream_t stream) {
    a.tiles_m = (int)tile_count(a.M, C::BM);
    a.tiles_n = (int)tile_count(a.N, C::BN);
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n)), block(C::NT);
    if (i32out && ragged) hipLaunchKernelGGL((tile_gemm_kernel<C, true, true, false>), grid, block, 0, stream, a);
    else if (i32out) hipLaunchKernelGGL((tile_gemm_kernel<C, true, false, false>), grid, block, 0, stream, a);
    else if (a.bias && ragged) hipLaunchKernelGGL((tile_gemm_kernel<C, false, true, true>), grid, block, 0, stream, a);
    else if (a.bias) hipLaunchKernelGGL((tile_gemm_kernel<C, false, false, true>), grid, block, 0, stream, a);
    else if (ragged) hipLaunchKernelGGL((tile_gemm_kernel<C, false, true, false>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((tile_gemm_kernel<C, false, false, false>), grid, block, 0, stream, a);
    return hipGetLastError();
}

// ---- the kernel of a shape -------------------------------------------------------
// Counted in 128 x 64 wave tiles (t = M / 64 x N / 128, rounded up), c compute
// units; a workgroup of four waves fills half a compute unit's wave slots.
//   t <= 2 c                the k loop over four waves: every wave of the launch
//                           is resident at once and the k loop is a quarter as
//                           long (1024 x 4608 -> 1152: 11.3 us against 22.0 for two
//                           halves of the workgroup and 26.3 on 256-token tiles;
//                           1024 x 1152 -> 3456: 9.9 / 11.6 / 12.2;
//                           3584 x 1152 -> 1152, t = 1.97 c: 9.3, over two waves
//                           11.2; 3712, 2.04 c: 12.7 / 11.0);
//   2 c < t <= 3 c          still one round of two-wave workgroups: k over two
//                           waves (1280 x 1152 -> 3456: 11.8, over four 13.8,
//                           256-token tiles 12.3), or over four on long k loops,
//                           which hide the second round (1024 x 3072 -> 9216 is t =
//                           1152: 31.3 over four, 33.4 on 128-token tiles; 8192 x
//                           4608 -> 1152: 40.9 / 46.0; 2048 x 3072 -> 3072, t = 768: 21.6,
//                           22.2 over two), up to t = 5 c (2752 x 3072 -> 3072, 4.03 c:
//                           30.5, 128-token tiles 33.1; 3392, 4.97 c: 32.1 / 36.5; 3456,
//                           5.06 c: 35.7 / 36.1, W4A8 40.0 / 38.5);
//   3 c < t <= 4 c          256-token tiles, half a round (1536 x 1152 -> 4608: 13.4,
//                           k over two waves 13.9), while they are c at most:
//                           one more and a unit works through two (2688 x 3072
//                           -> 3072 is 264 of them: 37.7, k over two waves 24.6;
//                           7232 x 1152 -> 1152, 261: 18.7 / 14.5);
//   4 c < t <= 6 c          128-token tiles: 256-token ones would start a second
//                           round of a few (3072 x 1152 -> 3456: 18.9 against 19.8;
//                           4096 x 3072 -> 3072: 37.5 / 38.8; 10880 x 1152 -> 1152, 5.98
//                           c: 18.9 / 19.4; 10944, 6.01 c: 20.0 / 19.6); and up to
//                           8 c, where 256-token ones are more than the 2 c
//                           resident at once but 128-token ones no more than their
//                           4 c (1907 x 3072 -> 8605, 544 and 1020 tiles: 53.6 against
//                           42.3; 14464 x 1152 -> 1152 26.0 / 20.6, fp6 26.1 / 20.1; not
//                           of W8A8's, 3 c: 14464 x 4608 -> 1152 95.1 / 98.1);
//   t > 6 c                 256-token tiles, which move the fewest operand bytes
//                           (43200 x 1152 block: 590 us of GEMM against 690), up
//                           to 2^24 - 1 of them (a launch has under 2^32 lanes).
// Splits need a stage for every wave.  fp6 operands are half again as large,
// the matrix work half: four waves only pay up to t = c (2048 x 1152 -> 1152, t =
// 288: 9.1 over two waves, 10.1 over four; 1536, t = 216: 7.3 both; 1792, 0.98 c: 6.7
// both; 1856, 1.02 c: 8.3 / 9.3), two up to 2 c, and to 3 c on k loops under 48
// stages (1280 x 1152 -> 3456: 11.9, 256-token tiles 12.3; but 1536 x 3072 -> 3072: 21.2
// / 20.1; 5440 x 1152 -> 1152, 2.99 c: 11.9 / 12.1; 5504, 3.02 c: 13.5 / 12.1); up to 4 c
// more than c 256-token tiles give way to 128-token ones (2688 x 3072 -> 3072: 30.7 /
// 23.3, k over two waves 26.4).
enum Variant { kTile256, kTile128, kSplit4, kSplit2, kVariants };
// token tile, waves of a workgroup
constexpr int kVariantTokens[kVariants] = {256, 128, 64, 64};
constexpr int kVariantWaves[kVariants] = {4, 2, 4, 2};
template <Fmt F>
inline Variant pick_variant(int64_t M, int64_t N, int64_t K, int cus) {
    const int64_t t = tile_count(M, 64) * tile_count(N, 128), c = cus, nks = K >> 6;
    const int64_t t256 = tile_count(M, 256) * tile_count(N, 128);
    if (t256 >= (int64_t)1 << 24) return kTile128;
    const bool one_round = F != Fmt::W8A8 && t256 > 2 * c && tile_count(M, 128) * tile_count(N, 128) <= 4 * c;
    if constexpr (F == Fmt::F6) {
        if (nks >= 4 && t <= c) return kSplit4;
        if (nks >= 2 && (t <= 2 * c || (t <= 3 * c && nks < 48))) return kSplit2;
        return one_round || (t <= 6 * c && (t > 4 * c || t256 > c)) ? kTile128 : kTile256;
    }
    if (nks >= 4 && (t <= 2 * c || (nks >= 48 && t <= 5 * c && !(t > 3 * c && t <= 4 * c)))) return kSplit4;
    if (nks >= 2 && (t <= 3 * c || (t <= 4 * c && t256 > c))) return kSplit2;
    if (one_round || (t > 4 * c && t <= 6 * c)) return kTile128;
    return kTile256;
}

// ring depths: at least two workgroups (256 tokens) or three (128) per compute
// unit's 160 KB of LDS
template <Fmt F> constexpr int kRing256 = F == Fmt::W4A4 ? 5 : F == Fmt::F6 ? 4 : 3;
template <Fmt F> constexpr int kRing128 = F == Fmt::W4A4 ? 4 : 3;

template <Fmt F>
hipError_t launch_variant(Variant v, const Args &a, bool i32out, hipStream_t stream) {
    const bool ragged = a.N % 16 != 0;
    switch (v) {
        case kTile256: return launch<Cfg<F, 4, kRing256<F>>>(a, i32out, ragged, stream);
        case kTile128: return launch<Cfg<F, 2, kRing128<F>>>(a, i32out, ragged, stream);
        case kSplit4: return launch_split<SplitCfg<F, 4>>(a, i32out, ragged, stream);
        case kSplit2: return launch_split<SplitCfg<F, 2>>(a, i32out, ragged, stream);
        case kVariants: break;
    }
    return hipErrorInvalidValue;
}

template <Fmt F>
hipError_t launch_tiles(const Args &a, bool i32out, hipStream_t stream) {
    return launch_variant<F>(pick_variant<F>(a.M, a.N, a.K, compute_units()), a, i32out, stream);
}

constexpr int kGroupPanels = 4;   // token panels per tile group

}  // namespace tg
}  // namespace
}  // namespace clq
