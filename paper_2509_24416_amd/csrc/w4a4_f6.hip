// W4A4 GEMM on the fp6 matrix cores of gfx950, with the dequantising
// epilogue fused (CLQ, arXiv 2509.24416: the integer product of the W4A4
// codes, rescaled by the per-token activation scale and the per-channel
// weight scale of Eq. (1), plus bias).
//
// Codes carried as fp6.  gfx950 has no 4-bit integer matrix instruction.  Its
// fp6 format e2m3 (1 sign, 2 exponent, 3 mantissa bits, bias 1) holds every
// code of the 4-bit grid, -7..7, exactly, and v_mfma_f32_32x32x64_f8f6f4 on
// two fp6 operands multiplies them at twice the int8 instruction's rate.
// Each product of two codes is an integer of magnitude at most 49, and every
// partial sum of a k loop shorter than 2^24 / 49 codes is an integer below
// 2^24, which fp32 holds exactly: the accumulators are the exact integers
// sum_k qa * qw, whatever the order of the additions.
//
// fp6 code layout (weights and activations): the unit and lane map of the
// packed int4 layouts (32 rows x 64 codes per unit, lane l = 32h + rho
// holding codes 32h .. 32h+31 of fragment row rho; weights with their
// fragment-row order, so that accumulator element v of lane l is channel
// 16 (l / 32) + v of the fragment), 24 bytes per lane: code i of the lane's
// 32 at bits 6i .. 6i+5 of its 192 bits (f6_codes.h).  A unit is 1536
// bytes: lane l's first 16 bytes at 16 l, its last 8 after the first 1 KB
// (aligned LDS reads of 16 and 8 bytes; the transfer into LDS is one 16-byte
// load per lane for the first 1 KB and one 16-byte load on 32 lanes for the
// rest).  Units are stored [row unit][k unit].
//
// The product runs on the kernels of tile_gemm.h (one matrix instruction per
// fragment and 64-code stage, no operand widening).  This file keeps the
// two-halves kernel, for long k loops with few tiles, and the format
// conversion.  Against a persistent kernel with a branch-heavy stage loop the
// 16384-token block of width 1152 takes 246 us of GEMM instead of 283, the
// 4608-token one of width 3072 361 instead of 382.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "clq_internal.h"
#include "f6_codes.h"
#include "tile_gemm.h"

#define CLQ_LDS __attribute__((address_space(3)))

namespace clq {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
template <int Q> using IC = std::integral_constant<int, Q>;

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return (uint32_t)reinterpret_cast<size_t>((CLQ_LDS const void *)p);
}
template <int OFF>
__device__ __forceinline__ v4u lds_read16(uint32_t addr) {
    v4u v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ v2u lds_read8(uint32_t addr) {
    v2u v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// two fp16 outputs fma(p, w, bias) rounded once from fp32 operands and a
// packed fp16 bias pair (low half: first output)
__device__ __forceinline__ uint32_t fma_mix2(float p0, float w0, float p1, float w1, uint32_t b) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[0,0,1]\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, %3 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
        : "=&v"(r)
        : "v"(p0), "v"(w0), "v"(b), "v"(p1), "v"(w1));
    return r;
}

constexpr int kUnit = kF6Unit;  // bytes of a 32 x 64 fp6 unit
constexpr int kGroupM = 8;      // token panels per tile group (L2 reuse of channel panels)

// global -> LDS transfers of 16 and 4 bytes per lane (plain functions, so that
// the builtin's operands never depend on a template parameter, which the
// host compilation pass does not accept)
__device__ __forceinline__ void dma_lds16(const uint8_t *src, uint8_t *dst) {
    __builtin_amdgcn_global_load_lds(src, (CLQ_LDS void *)dst, 16, 0, 0);
}
__device__ __forceinline__ void dma_lds4(const uint8_t *src, uint8_t *dst) {
    __builtin_amdgcn_global_load_lds(src, (CLQ_LDS void *)dst, 4, 0, 0);
}

// waits for all but N outstanding transfers (and the LDS reads), then the
// workgroup barrier
template <int N>
__device__ __forceinline__ void wait_landed_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

struct F6Args {
    const uint8_t *Xq;
    const float *xs;
    const uint8_t *Wq;
    const float *ws;
    const uint16_t *bias;
    void *Y;
    int64_t ldy;
    int M, N, K, tiles_m, tiles_n;
};

// The LDS reads of one stage's operands have landed: one wait that names
// every destination register, so that no use is scheduled before it.
template <int FM>
__device__ __forceinline__ void wait_operands(v4u (&ra)[4], v4u (&rb)[FM], v2u (&sa)[4], v2u (&sb)[FM]) {
    static_assert(FM == 1 || FM == 2, "operand lists below");
    if constexpr (FM == 2)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(ra[0]), "+v"(ra[1]), "+v"(ra[2]), "+v"(ra[3]), "+v"(rb[0]), "+v"(rb[1]),
                       "+v"(sa[0]), "+v"(sa[1]), "+v"(sa[2]), "+v"(sa[3]), "+v"(sb[0]), "+v"(sb[1]));
    else
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(ra[0]), "+v"(ra[1]), "+v"(ra[2]), "+v"(ra[3]), "+v"(rb[0]),
                       "+v"(sa[0]), "+v"(sa[1]), "+v"(sa[2]), "+v"(sa[3]), "+v"(sb[0]));
}

// ---- few tiles with long k loops: the k loop in two halves ---------------------
// The two-halves scheme of the int4 GEMM on fp6 operands.  Each tile (128
// channels x BM tokens) gets two halves of NWH waves: half 0 runs the first
// half of the k-stages and half 1 the rest, each through its own NS-slot LDS
// ring (tile_gemm.h's ring protocol), in lockstep on the workgroup
// barrier; a second half one stage shorter idles on its last step.  At the
// end the halves swap their fp32 sums (exact integers, so exact sums) through
// the idle rings and each finishes two of the four channel fragments with
// the epilogue arithmetic of every other kernel.  One tile per workgroup, two
// workgroups per compute unit.
template <int NWH_, int NS_>
struct F6HalfTile {
    static constexpr int NWH = NWH_, NS = NS_, FN = 4, FM = 2;
    static constexpr int NT = 2 * NWH * 64;
    static constexpr int BN = FN * 32, BM = NWH * FM * 32;
    static constexpr int WUnits = BN / 32, XUnits = BM / 32, Units = WUnits + XUnits;
    static constexpr int UPW = Units / NWH;   // units per wave and stage, within a half
    static constexpr int VPW = 2 * UPW;       // transfers per wave and stage
    static constexpr int Slot = Units * kUnit;
    static constexpr int Exch = NWH * 16384;  // one half's outgoing sums: 2 fragments x 2 x 16 floats x 64 lanes per wave
    static constexpr int Pool = 2 * NS * Slot > 2 * Exch ? 2 * NS * Slot : 2 * Exch;
    static_assert(Units % NWH == 0, "units split evenly over a half's waves");
};
using F6Half128 = F6HalfTile<2, 3>;   // 128 x 128 tiles, 72 KB of rings
using F6Half64 = F6HalfTile<1, 4>;    // 128 x 64 tiles, 72 KB of rings

// the mixed fma of fma_mix2 with fp32 bias operands (each exactly an fp16 value)
__device__ __forceinline__ uint32_t fma_mix2f(float p0, float w0, float b0, float p1, float w1, float b1) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, %6"
        : "=&v"(r)
        : "v"(p0), "v"(w0), "v"(b0), "v"(p1), "v"(w1), "v"(b1));
    return r;
}

template <class C, bool I32OUT, bool RAGGED, bool BIAS>
__global__ void __launch_bounds__(C::NT, C::NWH == 1 ? 1 : 2) f6_gemm_halves_kernel(F6Args a)
{
    static_assert(!(I32OUT && BIAS), "no bias on the integer output");
    constexpr int NS = C::NS, kFN = C::FN, kFM = C::FM, kUPW = C::UPW, kVPW = C::VPW, kSlot = C::Slot;
    __shared__ __align__(16) uint8_t pool[C::Pool];
    // the tile's epilogue operands, staged after the k loop as floats:
    // channel scales, biases (fp16 widened, exact), token scales
    constexpr int EPN = 2 * C::BN + C::BM;
    __shared__ float ep[EPN];
    const float *ep_ws = ep, *ep_b = ep + C::BN, *ep_xs = ep + 2 * C::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = w8 / C::NWH, wm = w8 % C::NWH;
    const int M = a.M, N = a.N, nks = a.K >> 6;
    // one tile per workgroup: workgroups are dealt to the 8 XCDs
    // round-robin, and each XCD takes a contiguous run of the grouped order
    int L;
    {
        const int G = gridDim.x, x = blockIdx.x & 7, j = blockIdx.x >> 3;
        const int per = G >> 3, rem = G & 7;
        L = x * per + min(x, rem) + j;
    }
    int tm, tn;
    {
        const int gsz = kGroupM * a.tiles_n;
        const int g = L / gsz, r = L - g * gsz;
        const int m0 = g * kGroupM;
        const int gm = min(a.tiles_m - m0, kGroupM);
        tn = r / gm;
        tm = m0 + (r - tn * gm);
    }
    const int h0 = (nks + 1) >> 1;
    const int kb = half ? h0 : 0, len = half ? nks - h0 : h0;   // len >= 1 (nks >= 2)
    const int wunits_total = (int)(padded_rows(N) >> 5);
    const int xunits_total = (int)(padded_act_rows(M) >> 5);
    uint8_t *ring = pool + half * NS * kSlot;
    const uint8_t *usrc[C::UPW];
#pragma unroll
    for (int j = 0; j < kUPW; ++j) {
        const int u = wm * kUPW + j;
        if (u < C::WUnits) {
            const int ug = min(tn * C::WUnits + u, wunits_total - 1);
            usrc[j] = a.Wq + ((int64_t)ug * nks + kb) * kUnit;
        } else {
            const int ux = min(tm * C::XUnits + (u - C::WUnits), xunits_total - 1);
            usrc[j] = a.Xq + ((int64_t)ux * nks + kb) * kUnit;
        }
    }
    // stage k of this half into slot q; past the end the last stage is
    // loaded again (into a slot whose contents are never read), so every wave
    // issues the same transfers and the wait counts stay fixed
    auto produce = [&](int q, int k) {
        const uint32_t voff = (uint32_t)(min(k, len - 1) * kUnit + lane * 16);
        uint8_t *dst = ring + q * kSlot;
#pragma unroll
        for (int j = 0; j < kUPW; ++j) dma_lds16(usrc[j] + voff, dst + (wm * kUPW + j) * kUnit);
        if (lane < 32) {
#pragma unroll
            for (int j = 0; j < kUPW; ++j) dma_lds16(usrc[j] + voff + 1024, dst + (wm * kUPW + j) * kUnit + 1024);
        }
    };
    // two operand register sets used by alternate stages (the persistent
    // kernel's scheme; the ragged instances read into set 1 and copy it)
    constexpr bool kAlt = !RAGGED;
    v4u ra[2][kFN], rb[2][kFM];
    v2u sa[2][kFN], sb[2][kFM];
    const uint32_t wl0 = (uint32_t)(lane * 16), wl1 = (uint32_t)f6_tail_offset(lane);
    const uint32_t xo = (uint32_t)((C::WUnits + wm * kFM) * kUnit);
    auto read_stage = [&](int q, auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        uint32_t b16 = wl0, b8 = wl1;
        asm volatile("" : "+v"(b16), "+v"(b8));
        const uint32_t base = lds_addr(ring + q * kSlot);
        b16 += base;
        b8 += base;
        const uint32_t bx16 = b16 + xo, bx8 = b8 + xo;
        static_for<0, kFN>([&](auto f) {
            constexpr int o = decltype(f)::value * kUnit;
            ra[P][f] = lds_read16<o>(b16);
            sa[P][f] = lds_read8<o>(b8);
        });
        static_for<0, kFM>([&](auto f) {
            constexpr int o = decltype(f)::value * kUnit;
            rb[P][f] = lds_read16<o>(bx16);
            sb[P][f] = lds_read8<o>(bx8);
        });
    };
    auto stage_ready = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        wait_operands(ra[P], rb[P], sa[P], sb[P]);
    };
    v16f acc[kFN][kFM];
#pragma unroll
    for (int fn = 0; fn < kFN; ++fn)
#pragma unroll
        for (int fm = 0; fm < kFM; ++fm) acc[fn][fm] = v16f{};
    auto mma = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        v8i opa[kFN], opb[kFM];
#pragma unroll
        for (int f = 0; f < kFN; ++f)
            opa[f] = v8i{(int)ra[P][f][0], (int)ra[P][f][1], (int)ra[P][f][2], (int)ra[P][f][3],
                         (int)sa[P][f][0], (int)sa[P][f][1], 0, 0};
#pragma unroll
        for (int f = 0; f < kFM; ++f)
            opb[f] = v8i{(int)rb[P][f][0], (int)rb[P][f][1], (int)rb[P][f][2], (int)rb[P][f][3],
                         (int)sb[P][f][0], (int)sb[P][f][1], 0, 0};
#pragma unroll
        for (int fn = 0; fn < kFN; ++fn)
#pragma unroll
            for (int fm = 0; fm < kFM; ++fm)
                acc[fn][fm] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(opa[fn], opb[fm], acc[fn][fm], 2, 2, 0, 0, 0, 0);
    };

    // epilogue operands: loaded first (EPR per thread at clamped indices,
    // ahead of the transfers), held in registers through the k loop and
    // written to LDS after it, when no transfer into LDS is in flight
    constexpr int EPR = (EPN + C::NT - 1) / C::NT;
    float epv[EPR];
    _Float16 epb[EPR];
#pragma unroll
    for (int r = 0; r < EPR; ++r) {
        const int e = min(tid + r * C::NT, EPN - 1);
        const int ec = e & (C::BN - 1), er = max(e - 2 * C::BN, 0);
        const float *esrc = e < 2 * C::BN ? a.ws + min(tn * C::BN + ec, N - 1) : a.xs + min(tm * C::BM + er, M - 1);
        epv[r] = I32OUT ? 0.0f : *esrc;
        epb[r] = (_Float16)0.0f;
        if constexpr (BIAS) epb[r] = reinterpret_cast<const _Float16 *>(a.bias)[min(tn * C::BN + ec, N - 1)];
    }
    __builtin_amdgcn_sched_barrier(0);

    // stage s+1 has landed once at most the NS - 2 later productions are
    // outstanding (completion is in issue order)
    // prologue: stages 0..NS-1 in flight, stage 0 read into registers
    for (int q = 0; q < NS; ++q) produce(q, q);
    wait_vm_barrier<(NS - 1) * kVPW>();
    read_stage(0, IC<kAlt ? 0 : 1>{});
    stage_ready(IC<kAlt ? 0 : 1>{});
    // both halves take h0 steps; stage s in register set s & 1
    int q = 0, s = 0;
    auto step = [&](auto pc) __attribute__((always_inline)) -> bool {
        constexpr IC<kAlt ? decltype(pc)::value : 0> cur{};
        constexpr IC<kAlt ? 1 - decltype(pc)::value : 1> nxt{};
        const int nq = q + 1 == NS ? 0 : q + 1;
        const bool active = s < len;
        if constexpr (!kAlt) {
#pragma unroll
            for (int f = 0; f < kFN; ++f) {
                ra[0][f] = ra[1][f];
                sa[0][f] = sa[1][f];
            }
#pragma unroll
            for (int f = 0; f < kFM; ++f) {
                rb[0][f] = rb[1][f];
                sb[0][f] = sb[1][f];
            }
        }
        wait_landed_barrier<(NS - 2) * kVPW>();
        read_stage(nq, nxt);
        produce(q, s + NS);
        __builtin_amdgcn_sched_barrier(0);
        if (active) mma(cur);
        __builtin_amdgcn_sched_barrier(0);
        stage_ready(nxt);
        q = nq;
        ++s;
        return s < h0;
    };
    if (h0 > 0)
        while (step(IC<0>{}) && step(IC<1>{})) {
        }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // the epilogue operands into LDS (a thread past the end writes the last
    // value again); the barrier after the sends below publishes them
#pragma unroll
    for (int r = 0; r < EPR; ++r) {
        const int e = min(tid + r * C::NT, EPN - 1);
        ep[e] = e >= C::BN && e < 2 * C::BN ? (float)epb[r] : epv[r];
    }

    // the halves swap sums through the idle rings: half 0 finishes channel
    // fragments 0-1 and half 1 fragments 2-3, each adding the other's
    auto send = [&](auto f0c) {
        constexpr int f0 = decltype(f0c)::value;
        v4f *out = reinterpret_cast<v4f *>(pool + half * C::Exch + wm * 16384);
        static_for<0, 2>([&](auto fc) {
            constexpr int fn = f0 + decltype(fc)::value;
#pragma unroll
            for (int fm = 0; fm < kFM; ++fm)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const v16f &x = acc[fn][fm];
                    out[((decltype(fc)::value * kFM + fm) * 4 + q4) * 64 + lane] =
                        v4f{x[4 * q4], x[4 * q4 + 1], x[4 * q4 + 2], x[4 * q4 + 3]};
                }
        });
    };
    auto receive = [&](auto f0c) {
        constexpr int f0 = decltype(f0c)::value;
        const v4f *in = reinterpret_cast<const v4f *>(pool + (1 - half) * C::Exch + wm * 16384);
        static_for<0, 2>([&](auto fc) {
            constexpr int fn = f0 + decltype(fc)::value;
#pragma unroll
            for (int fm = 0; fm < kFM; ++fm)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const v4f y = in[((decltype(fc)::value * kFM + fm) * 4 + q4) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[fn][fm][4 * q4 + e] += y[e];
                }
        });
    };
    if (half == 0) send(IC<2>{});
    else send(IC<0>{});
    __syncthreads();
    if (half == 0) receive(IC<0>{});
    else receive(IC<2>{});

    // epilogue: lane owns token m and 16 consecutive channels; each half
    // its two channel fragments
    const int h16 = (lane >> 5) * 16;
    auto epilogue = [&](auto f0c) {
        static_for<0, 2>([&](auto fc) {
            constexpr int fn = decltype(f0c)::value + decltype(fc)::value;
            const int c0 = fn * 32 + h16, n0 = tn * C::BN + c0;
            float wsv[16], bw[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                wsv[v] = ep_ws[c0 + v];
                bw[v] = BIAS ? ep_b[c0 + v] : 0.0f;
            }
#pragma unroll
            for (int fm = 0; fm < kFM; ++fm) {
                const int r0 = (wm * kFM + fm) * 32 + (lane & 31), m = tm * C::BM + r0;
                const v16f &x = acc[fn][fm];
                if constexpr (I32OUT) {   // the exact integer sums
                    int32_t *dst = reinterpret_cast<int32_t *>(a.Y) + (int64_t)m * a.ldy + n0;
                    if (m < M && n0 < N) {
                        if (!RAGGED || n0 + 16 <= N) {
#pragma unroll
                            for (int q4 = 0; q4 < 4; ++q4)
                                reinterpret_cast<v4i *>(dst)[q4] =
                                    v4i{(int)x[4 * q4], (int)x[4 * q4 + 1], (int)x[4 * q4 + 2], (int)x[4 * q4 + 3]};
                        } else {
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                if (n0 + v < N) dst[v] = (int)x[v];
                        }
                    }
                    continue;
                }
                uint32_t hv[8];
                const float xsc = ep_xs[r0];
#pragma unroll
                for (int v = 0; v < 16; v += 2)
                    hv[v / 2] = fma_mix2f(x[v] * xsc, wsv[v], bw[v], x[v + 1] * xsc, wsv[v + 1], bw[v + 1]);
                uint16_t *dst = reinterpret_cast<uint16_t *>(a.Y) + (int64_t)m * a.ldy + n0;
                if (m < M && n0 < N) {
                    if (!RAGGED || n0 + 16 <= N) {
                        reinterpret_cast<v4u *>(dst)[0] = v4u{hv[0], hv[1], hv[2], hv[3]};
                        reinterpret_cast<v4u *>(dst)[1] = v4u{hv[4], hv[5], hv[6], hv[7]};
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            if (n0 + v < N) dst[v] = (uint16_t)(hv[v >> 1] >> (16 * (v & 1)));
                    }
                }
            }
        });
    };
    if (half == 0) epilogue(IC<0>{});
    else epilogue(IC<2>{});
}

// ---- format conversion: packed int4 units -> fp6 units ---------------------------
// One thread per lane slot: its 16 bytes (32 nibbles) become its six fp6
// dwords (the code order of f6_codes.h).
__global__ void repack_f6_kernel(const uint8_t *__restrict__ in, uint8_t *__restrict__ out, int64_t slots) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= slots) return;
    const int64_t unit = t >> 6;
    const int l = (int)(t & 63);
    const v4u src = *reinterpret_cast<const v4u *>(in + unit * 1024 + l * 16);
    const uint32_t d[4] = {src[0], src[1], src[2], src[3]};
    uint32_t w[6];
    f6_from_nibbles(d, w);
    f6_store(out + unit * kF6Unit, l, w);
}

}  // namespace

hipError_t launch_repack_f6(const uint8_t *in, int64_t units, uint8_t *out, hipStream_t stream) {
    const int64_t slots = units * 64;
    if (slots == 0) return hipSuccess;
    hipLaunchKernelGGL(repack_f6_kernel, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, stream, in, out, slots);
    return hipGetLastError();
}

namespace {

template <class C>
hipError_t launch_gemm_f6_halves(F6Args g, bool i32out, bool ragged, hipStream_t stream) {
    g.tiles_m = (g.M + C::BM - 1) / C::BM;
    g.tiles_n = (g.N + C::BN - 1) / C::BN;
    const dim3 gd((unsigned)(g.tiles_m * g.tiles_n)), bd(C::NT);   // one tile per workgroup
    if (i32out) {
        if (ragged) hipLaunchKernelGGL((f6_gemm_halves_kernel<C, true, true, false>), gd, bd, 0, stream, g);
        else hipLaunchKernelGGL((f6_gemm_halves_kernel<C, true, false, false>), gd, bd, 0, stream, g);
    } else if (ragged) {
        if (g.bias) hipLaunchKernelGGL((f6_gemm_halves_kernel<C, false, true, true>), gd, bd, 0, stream, g);
        else hipLaunchKernelGGL((f6_gemm_halves_kernel<C, false, true, false>), gd, bd, 0, stream, g);
    } else {
        if (g.bias) hipLaunchKernelGGL((f6_gemm_halves_kernel<C, false, false, true>), gd, bd, 0, stream, g);
        else hipLaunchKernelGGL((f6_gemm_halves_kernel<C, false, false, false>), gd, bd, 0, stream, g);
    }
    return hipGetLastError();
}

}  // namespace

int f6_schedule_force = 0;

// The kernel an M x N x K product gets, for the launch and for the query (the
// numbers of clq_w4a4_schedule_f6; 1, 2 and 3 are what the knob forces).
int f6_schedule(int64_t M, int64_t N, int K) {
    const int force = __atomic_load_n(&f6_schedule_force, __ATOMIC_RELAXED);
    if (force >= 1 && force <= 3) return force;
    // Long k loops (48 stages or more) with more than one and at most two 128 x
    // 64 wave tiles per compute unit stay on the two halves, whose four waves
    // share the operands through LDS (2048 x 4608 -> 1152: 18.8 us, 19.4 with the
    // k loop over two waves, 20.6 over four, 25.2 on 256-token tiles).
    const int64_t waves = (M + 63) / 64 * ((N + 127) / 128), cus = tg::compute_units();
    if ((K >> 6) >= 48 && waves > cus && waves <= 2 * cus) return 2;
    switch (tg::pick_variant<tg::Fmt::F6>(M, N, K, (int)cus)) {
        case tg::kTile128: return 6;
        case tg::kSplit4: return 4;
        case tg::kSplit2: return 5;
        default: return 1;
    }
}

hipError_t launch_gemm_f6(const uint8_t *Xq, const float *xs, const uint8_t *Wq, const float *ws,
                          const uint16_t *bias, int64_t M, int64_t N, int K, void *Y, int64_t ldy, bool i32out,
                          hipStream_t stream) {
    const int choice = f6_schedule(M, N, K);
    if (choice != 2 && choice != 3) {
        tg::Args t{};
        t.Xq = Xq;
        t.xs = xs;
        t.Wq = Wq;
        t.ws = ws;
        t.bias = bias;
        t.Y = Y;
        t.ldy = ldy;
        t.M = (int)M;
        t.N = (int)N;
        t.K = K;
        t.group_m = tg::kGroupPanels;
        const tg::Variant v = choice == 6 ? tg::kTile128 : choice == 4 ? tg::kSplit4 : choice == 5 ? tg::kSplit2 : tg::kTile256;
        return tg::launch_variant<tg::Fmt::F6>(v, t, i32out, stream);
    }
    F6Args g{};
    g.Xq = Xq;
    g.xs = xs;
    g.Wq = Wq;
    g.ws = ws;
    g.bias = bias;
    g.Y = Y;
    g.ldy = ldy;
    g.M = (int)M;
    g.N = (int)N;
    g.K = K;
    const bool ragged = N % 16 != 0 || (bias && reinterpret_cast<uintptr_t>(bias) % 4 != 0);
    return choice == 2 ? launch_gemm_f6_halves<F6Half128>(g, i32out, ragged, stream)
                       : launch_gemm_f6_halves<F6Half64>(g, i32out, ragged, stream);
}

}  // namespace clq
