"""GPU parity of the whole-tile GEMM kernels at the edges of their choice.

The kernel follows from t, the 128 x 64 wave tiles of the product (256 compute
units assumed): the k loop over four waves up to t = 512 (and to 1280 on k
loops of 48 stages of 64 codes or more), over two up to 768 (1024 where tiles
of 256 tokens would be more than 256), tiles of 256 tokens up to 1024, of 128 up
to 1536 (2048 where they are one round and tiles of 256 more), of 256 beyond;
fp6 codes take four waves to 256, two to 512 (768 under 48 stages), two halves
of a workgroup from 256 to 512 on longer k loops, and a persistent grid past
512 tiles of 256 tokens on k loops of at most 12 or 18 stages (one or two tiles a
workgroup, several); fewer stages than waves fall through to the next choice.
Shapes sit on both sides of each line, with ragged token and channel counts and stage counts that leave remainders, for
every code storage.  Sums are integers and exact.  An fp16 output is one
rounding of fma(p, w_scale, bias), p the fp32 rounding of sum * x_scale:
within 2^-11 of the value, plus 2^-24 |p w_scale| for p's rounding, plus half
of the smallest subnormal.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_24416_amd as m
    return m


SHAPES = [(1, 16, 128), (33, 130, 128), (65, 200, 192), (300, 1000, 256), (257, 1009, 448), (2000, 2040, 320),
          (2100, 2048, 256), (1500, 4000, 192), (2120, 3072, 320), (4000, 2050, 128), (2040, 3968, 3072),
          (1100, 3072, 256), (1100, 3000, 3072), (2100, 4090, 192), (2560, 3072, 3136), (6200, 2000, 256), (6208, 2050, 128),
          (8201, 2048, 128), (4900, 3456, 192), (16384, 1152, 320), (12800, 2176, 768), (2049, 8320, 448),
          (25700, 1024, 1152), (16400, 1008, 128), (16400, 1040, 128),
          (2688, 3072, 128), (520, 12000, 320), (840, 8605, 3072), (14464, 1152, 832)]


def _codes(clq, fmt, x, w, M, N, K, block):
    """(sums float64 [M, N], x_scale, w_scale, accum(), linear(bias))"""
    if fmt == "w4a4":
        q, s = clq.clq_rotate_quant_act(x, block)
        qw = clq.clq_quantize_weights(w, block)
        xc, wc = clq.clq_unswizzle_act(q, M, K), clq.clq_unswizzle_weights(qw)
        acc, lin = clq.clq_w4a4_accum_i32, clq.clq_w4a4_linear
    elif fmt == "f6":
        q, s = clq.clq_rotate_quant_act_f6(x, block)
        qw = clq.clq_quantize_weights_f6(w, block)
        xc, wc = clq.clq_unswizzle_f6(q, M, K, False), clq.clq_unswizzle_f6(qw.wq, N, K, True)
        acc, lin = clq.clq_w4a4_accum_f6, clq.clq_w4a4_linear_f6
    else:
        q, s = clq.clq_rotate_quant_act8(x, block)
        xc = clq.clq_unswizzle_act8(q, M, K)
        if fmt == "w4a8":
            qw = clq.clq_quantize_weights(w, block)
            wc = clq.clq_unswizzle_weights(qw)
        else:
            qw = clq.clq_quantize_weights8(w, block)
            wc = clq.clq_unswizzle_weights8(qw)
        acc, lin = clq.clq_a8_accum_i32, clq.clq_a8_linear

    def value(c, rows):   # packed nibbles (low first) or int8 codes -> float64
        if c.dtype == torch.uint8:
            c = c.reshape(rows, K // 2).to(torch.int16)
            c = torch.stack([c & 15, c >> 4], 2).reshape(rows, K)
            c = torch.where(c > 7, c - 16, c)
        return c.reshape(rows, K).double()

    return value(xc, M) @ value(wc, N).t(), s, qw.w_scale, lambda: acc(q, s, qw), lambda b: lin(q, s, qw, b)


@pytest.mark.parametrize("fmt", ["w4a4", "f6", "w4a8", "w8a8"])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_sums_and_outputs(clq, M, N, K, fmt):
    print(f"\n[gpu case] {fmt} {M} x {K} -> {N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    x[:, ::37] *= 30
    w = torch.randn((N, K), generator=g, device="cuda").half()
    bias = torch.randn(N, generator=g, device="cuda").half()
    sums, xs, ws, accum, linear = _codes(clq, fmt, x, w, M, N, K, 64)
    assert torch.equal(accum().double(), sums)
    p = sums * xs.double()[:, None] * ws.double()
    for b in (bias, None):
        y = p if b is None else p + b.double()
        bound = 2.0 ** -11 * y.abs() + 2.0 ** -23 * p.abs() + 2.0 ** -25
        got = linear(b).double()
        assert bool(((got - y).abs() <= bound).all())
    torch.cuda.synchronize()


@pytest.mark.parametrize("fmt", ["w4a4", "f6"])
@pytest.mark.parametrize("M,N,K", [(300, 1008, 256), (8201, 2048, 128)])
def test_bias_of_two_byte_alignment(clq, M, N, K, fmt):
    print(f"\n[gpu case] {fmt} {M} x {K} -> {N}, bias at an odd element", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    w = torch.randn((N, K), generator=g, device="cuda").half()
    bias = torch.randn(N + 1, generator=g, device="cuda").half()
    linear = _codes(clq, fmt, x, w, M, N, K, 64)[-1]
    assert torch.equal(linear(bias[1:]), linear(bias[1:].clone()))
    torch.cuda.synchronize()
