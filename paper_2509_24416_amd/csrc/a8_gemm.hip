// W4A8 and W8A8 GEMM with the CLQ epilogue (arXiv 2509.24416, Sec. 4.1: the
// method is run at the bit settings W8A8, W4A8 and W4A4; Sec. 3.1 Eq. (1)
// with n = 8 for the activations, and for the weights of W8A8).
//
// Activations arrive as int8 codes in the int8 layout (clq_internal.h), one
// fp32 scale per token; weights as int4 (the packed weight layout of the W4A4
// path) or int8 codes (the int8 layout, fragment rows in the int4 weights'
// order), one fp32 scale per output channel with 1/b folded in.  Both feed
// v_mfma_i32_32x32x32_i8 directly, except that int4 weights are widened to
// int8 holding 16 q (so the int32 accumulator holds 16 * sum for W4A8).
//
// The kernels are tile_gemm.h's.  On 128-token tiles of two waves, each stage
// read and waited for right before its matrix instructions, the block linears
// took (us; 8192 and 43200 tokens of width 1152, 4608 of width 3072): W4A8 217,
// 816, 570, W8A8 231, 935, 688; now 176, 674, 462 and 201, 736, 497.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clq_internal.h"
#include "tile_gemm.h"

namespace clq {

hipError_t launch_a8_gemm(const uint8_t *Xq8, const float *xs, const uint8_t *Wq, int wbits,
                          const float *ws, const uint16_t *bias, int64_t M, int64_t N, int K,
                          void *Y, int64_t ldy, bool i32out, hipStream_t stream) {
    tg::Args t{};
    t.Xq = Xq8;
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
    if (wbits == 4) return tg::launch_tiles<tg::Fmt::W4A8>(t, i32out, stream);
    if (wbits == 8) return tg::launch_tiles<tg::Fmt::W8A8>(t, i32out, stream);
    return hipErrorInvalidValue;
}

}  // namespace clq
