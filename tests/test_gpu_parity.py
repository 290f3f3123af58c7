"""GPU parity: the HIP path (through the C ABI binding) against the CPU oracle.

Integer results -- activation codes and scales, weight codes (after
unswizzling) and scales, int32 accumulators -- must match bit for bit; the
fp16 output must lie within 2e-3 of the oracle's fp64 dequantised result
(err = max |y - y64| / max(|p64| + |bias|, 2^-24)).  Small shapes span
several tiles and ragged tails; full-size layers are checked on sampled
token rows the oracle can afford.
"""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def clq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_24416_amd as m
    return m


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu case] {request.node.nodeid}", flush=True)
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# ---- rotate + quantize ---------------------------------------------------------

@pytest.mark.parametrize("M,K,block", [
    (1, 64, 32), (7, 128, 64), (255, 1152, 64), (257, 1152, 32), (64, 1152, 128),
    (33, 4608, 64), (20, 3072, 128), (5, 12288, 128), (3, 64, 64), (9, 256, 128)])
@pytest.mark.parametrize("law", ["L1", "L2"])
def test_rotate_quant_bitexact(clq, M, K, block, law):
    X = workloads.activations(M, K, law, seed=M + K + block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    ref_q, _, ref_s = oracle.quantize_act(X, block)
    assert np.array_equal(host(xs), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_act(Xq, M, K)), ref_q)
    # padding rows of the packed buffer hold zero codes
    assert Xq.numel() == clq.clq_act_bytes(M, K)


# Long rows (b = 64, 2048 <= K <= 5120) are handled in batches of 8 aligned
# rows; ragged row counts, a gather vector and a wider row stride included.
@pytest.mark.parametrize("M,K,ld,with_perm", [
    (1000, 4608, 4608, False), (777, 4608, 4672, True), (9, 2048, 2048, True), (1001, 5120, 5120, False),
    (8, 4608, 4608, False)])
def test_rotate_quant_long_rows(clq, M, K, ld, with_perm):
    X = workloads.activations(M, K, "L1", seed=M + K + 11)
    wide = np.zeros((M, ld), np.float16)
    wide[:, :K] = X
    perm = workloads.random_perm(K, seed=M) if with_perm else None
    Xq, xs = clq.clq_rotate_quant_act(dev(wide)[:, :K], 64, perm=None if perm is None else dev(perm))
    ref_q, _, ref_s = oracle.quantize_act(X, 64, perm)
    assert np.array_equal(host(xs), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_act(Xq, M, K)), ref_q)


@pytest.mark.parametrize("block", [32, 64, 128])
def test_rotate_quant_perm_and_stride(clq, block):
    M, K, ld = 37, 1152 if block != 128 else 1536, 2048
    X = workloads.activations(M, K, "L1", seed=block)
    wide = np.zeros((M, ld), np.float16)
    wide[:, :K] = X
    wide[:, K:] = np.float16(1000.0)          # must never be read
    perm = workloads.random_perm(K, seed=block + 1)
    Xd = dev(wide)[:, :K]
    Xq, xs = clq.clq_rotate_quant_act(Xd, block, dev(perm))
    ref_q, _, ref_s = oracle.quantize_act(X, block, perm)
    assert np.array_equal(host(xs), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_act(Xq, M, K)), ref_q)


def test_rotate_quant_adversarial_rows(clq):
    K, block = 256, 64
    X = np.zeros((8, K), np.float16)
    X[0, :] = np.float16(65504)
    X[1, ::2] = np.float16(-65504)
    X[2, :] = np.float16(-0.0)
    X[3, 17] = np.float16(6e-8)                   # one subnormal
    X[4, :] = np.float16(0.5)                     # exact ties after scaling
    X[4, 0] = np.float16(3.5)
    X[5, :64] = np.arange(64, dtype=np.float16) - np.float16(32)
    X[6, 3] = np.float16(-1.0)                    # single non-zero
    X[7, :] = workloads.activations(1, K, "L1", 3)[0]
    for block in (32, 64, 128):
        Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
        ref_q, _, ref_s = oracle.quantize_act(X, block)
        assert np.array_equal(host(xs), ref_s), block
        assert np.array_equal(host(clq.clq_unswizzle_act(Xq, 8, K)), ref_q), block


def test_act_padding_rows_are_zero(clq):
    M, K, block = 45, 256, 64                 # 45 rows -> 64 rows of storage
    X = workloads.activations(M, K, "L1", seed=4)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    assert Xq.numel() == 64 * K // 2
    full = host(clq.clq_unswizzle_act(Xq, 64, K))
    assert np.array_equal(full[:M], oracle.quantize_act(X, block)[0])
    assert not full[M:].any()


# ---- weights -------------------------------------------------------------------

@pytest.mark.parametrize("N,K,block,clip", [
    (1, 64, 32, 1.0), (8, 1152, 64, 1.0), (72, 1152, 64, 0.9), (200, 4608, 64, 1.0),
    (1152, 1152, 64, 1.0), (100, 3072, 128, 0.75), (3, 128, 128, 0.5)])
def test_quantize_weights_bitexact(clq, N, K, block, clip):
    W = workloads.weights(N, K, seed=N + K)
    qw = clq.clq_quantize_weights(dev(W), block, clip_ratio=clip)
    ref_q, _, ref_s = oracle.quantize_weights(W, block, None, clip)
    assert np.array_equal(host(qw.w_scale), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_weights(qw)), ref_q)


def test_quantize_weights_perm(clq):
    N, K, block = 96, 1152, 64
    W = workloads.weights(N, K, seed=5)
    perm = workloads.random_perm(K, seed=6)
    qw = clq.clq_quantize_weights(dev(W), block, dev(perm))
    ref_q, _, ref_s = oracle.quantize_weights(W, block, perm)
    assert np.array_equal(host(qw.w_scale), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_weights(qw)), ref_q)


# ---- GEMM: exact accumulators and the fp16 epilogue ------------------------------

# few tiles and at least 4 k-stages go through the two-halves kernel (the k
# loop split in two, the halves' sums added in LDS), including odd stage
# counts (one half a stage shorter) and ragged channels.  Its tiles have 128
# tokens, or 64 while the 128-token tiles would fill at most half the compute
# units: 64 for the small shapes, 128 for the last four (the last three at
# one to 2.5 tiles per compute unit, 8193 x 1030 in two rounds)
GEMM_SHAPES = [(1, 1, 64), (7, 8, 128), (129, 72, 192), (257, 200, 1152), (64, 1152, 1152),
               (300, 130, 640), (128, 128, 128), (513, 264, 4608), (257, 200, 576), (100, 1001, 320),
               (33, 48, 256), (5, 3, 256), (2049, 1030, 640), (4097, 1030, 640), (4000, 2000, 576),
               (8193, 1030, 576)]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("workspace", [None, False], ids=["ws", "nows"])
def test_accum_i32_bitexact(clq, M, N, K, workspace):
    block = 64
    X = workloads.activations(M, K, "L1", seed=M)
    W = workloads.weights(N, K, seed=N)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    acc = clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=workspace)
    _, xc, _ = oracle.quantize_act(X, block)
    _, wc, _ = oracle.quantize_weights(W, block)
    assert np.array_equal(host(acc), oracle.gemm_i32(xc, wc))


# Shapes whose schedule splits the k loop of its last rounds over
# every workgroup (clq_w4a4_schedule reports split stages), called repeatedly
# with one workspace: the split sums equal the whole-tile sums bit for bit
# and the oracle's on sampled rows.  (6400, 3072, 1536): 600 tiles, both
# rounds split; (6300, 3000, 1536): the same with ragged edges; (11264,
# 3200, 1536): one whole round, then 588 split tiles; (16384, 1152, 1920):
# 576 tiles of 30 stages, every stage split.
SPLIT_SHAPES = [(6400, 3072, 1536), (6300, 3000, 1536), (11264, 3200, 1536), (16384, 1152, 1920)]


@pytest.mark.parametrize("M,N,K", SPLIT_SHAPES)
def test_split_k_exact_and_repeatable(clq, M, N, K):
    block = 64
    plan = clq.clq_w4a4_schedule(M, N, K)
    assert plan["kernel"] == 0 and plan["split_stages"] > 0, plan
    assert clq.clq_w4a4_schedule(M, N, K, with_workspace=False)["split_stages"] == 0
    X = workloads.activations(M, K, "L1", seed=M + 7)
    W = workloads.weights(N, K, seed=N + 7)
    b = workloads.bias(N, seed=8)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    whole = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=False))
    Yw = host(clq.clq_w4a4_linear(Xq, xs, qw, dev(b), workspace=False))
    rows = np.unique(np.r_[0:3, M // 2 - 1:M // 2 + 2, M - 3:M, np.random.default_rng(M).choice(M, 10)])
    ref = oracle.linear(X[rows], W, b, block)
    assert np.array_equal(whole[rows], ref["acc"])
    ws = torch.zeros(clq.clq_w4a4_workspace_bytes(), dtype=torch.uint8, device="cuda")
    for rep in range(3):          # the workspace is left ready for the next call
        acc = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=ws))
        assert np.array_equal(acc, whole), rep
        Y = host(clq.clq_w4a4_linear(Xq, xs, qw, dev(b), workspace=ws))
        assert np.array_equal(Y.view(np.uint16), Yw.view(np.uint16)), rep
        assert oracle.err_metric(Y[rows].astype(np.float64), ref["y64"], ref["p64"], b) <= TOL, rep
    groups = clq.clq_w4a4_workspace_bytes() // (128 * 256 * 4 + 4 * 4)
    assert not host(ws[256:256 + groups * 4 * 4]).any()     # every flag back at zero
    assert clq.clq_w4a4_workspace_status(ws) == [0, 0, 0]   # no wait gave up


# Few tiles and a long k loop (no split, no workspace use): the automatic choice,
# and the two-halves kernel on 128- and 64-token tiles, which the schedule knob
# forces.
FEW_TILE_SHAPES = [(2048, 1152, 4608), (2000, 1000, 4608), (2048, 640, 8192), (1024, 1152, 4608), (300, 520, 8192)]


@pytest.mark.parametrize("M,N,K", FEW_TILE_SHAPES)
def test_few_tiles_long_k_exact(clq, M, N, K):
    block = 64
    assert clq.clq_w4a4_schedule(M, N, K)["kernel"] == 2    # k over four waves
    X = workloads.activations(M, K, "L1", seed=M + 7)
    W = workloads.weights(N, K, seed=N + 7)
    b = workloads.bias(N, seed=8)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    ref = oracle.linear(X, W, b, block)
    try:
        for force, kernel in ((0, 2), (3, 1), (4, 2)):
            clq.clq_debug_set(clq.CLQ_DEBUG_GEMM_SCHEDULE, force)
            assert clq.clq_w4a4_schedule(M, N, K)["kernel"] == kernel
            acc = clq.clq_w4a4_accum_i32(Xq, xs, qw)
            assert np.array_equal(host(acc), ref["acc"]), force
            Y = clq.clq_w4a4_linear(Xq, xs, qw, dev(b))
            assert oracle.err_metric(host(Y).astype(np.float64), ref["y64"], ref["p64"], b) <= TOL, force
            Y = clq.clq_w4a4_linear(Xq, xs, qw)
            assert oracle.err_metric(host(Y).astype(np.float64), ref["p64"], ref["p64"]) <= TOL, force
    finally:
        clq.clq_debug_set(clq.CLQ_DEBUG_GEMM_SCHEDULE, 0)


def test_split_k_wait_gives_up_is_reported(clq):
    # The split schedule's bounded wait, forced to run out from the host: a
    # short bound and contributors that never signal (a test-only switch).
    # Every kernel still exits; the owners leave the missing partials out and
    # the status words report it.  Then the knobs are restored, the
    # workspace zero-filled, and the same call is exact again.
    M, N, K, block = 6400, 3072, 1536, 64     # 600 tiles of 24 k-stages, all split
    assert clq.clq_w4a4_schedule(M, N, K)["split_stages"] > 0
    X = workloads.activations(M, K, "L1", seed=63)
    W = workloads.weights(N, K, seed=64)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    whole = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=False))
    ws = torch.zeros(clq.clq_w4a4_workspace_bytes(), dtype=torch.uint8, device="cuda")
    try:
        clq.clq_debug_set(clq.CLQ_DEBUG_SPLIT_SPIN_LIMIT, 16)
        clq.clq_debug_set(clq.CLQ_DEBUG_SPLIT_DROP_SIGNAL, 1)
        bad = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=ws))
    finally:
        clq.clq_debug_set(clq.CLQ_DEBUG_SPLIT_SPIN_LIMIT, 1 << 22)
        clq.clq_debug_set(clq.CLQ_DEBUG_SPLIT_DROP_SIGNAL, 0)
    gave_up, tile, rank = clq.clq_w4a4_workspace_status(ws)
    assert gave_up > 0
    assert 0 <= tile < 600 and 0 < rank < 8192
    assert not np.array_equal(bad, whole)            # the missing partials are visible
    ws.zero_()
    good = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=ws))
    assert np.array_equal(good, whole)
    assert clq.clq_w4a4_workspace_status(ws) == [0, 0, 0]


def test_default_workspace_per_stream(clq):
    # GEMMs on two streams with the binding's default workspace: each stream
    # gets its own, zero-filled on that stream.  Split-k launches of the two
    # streams alternate through events (a split launch needs its whole grid
    # resident); whole-tile launches run on both streams at once.
    M, N, K, block = 6400, 3072, 1536, 64
    assert clq.clq_w4a4_schedule(M, N, K)["split_stages"] > 0
    X = workloads.activations(M, K, "L1", seed=65)
    W = workloads.weights(N, K, seed=66)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    ref = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=False))
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    ev = None
    for i in range(4):
        s = s1 if i % 2 == 0 else s2
        with torch.cuda.stream(s):
            if ev is not None:
                s.wait_event(ev)
            outs.append(clq.clq_w4a4_accum_i32(Xq, xs, qw))
            ev = torch.cuda.Event()
            ev.record(s)
    torch.cuda.synchronize()
    w1, w2 = clq.default_workspace(stream=s1), clq.default_workspace(stream=s2)
    assert w1.data_ptr() != w2.data_ptr()
    for o in outs:
        assert np.array_equal(o.cpu().numpy(), ref)
    assert clq.clq_w4a4_workspace_status(stream=s1) == [0, 0, 0]
    assert clq.clq_w4a4_workspace_status(stream=s2) == [0, 0, 0]
    # whole-tile shapes on both streams at the same time
    Mw, Nw, Kw = 1024, 1024, 1152
    Xw = workloads.activations(Mw, Kw, "L1", seed=67)
    Ww = workloads.weights(Nw, Kw, seed=68)
    qww = clq.clq_quantize_weights(dev(Ww), block)
    Xqw, xsw = clq.clq_rotate_quant_act(dev(Xw), block)
    refw = host(clq.clq_w4a4_accum_i32(Xqw, xsw, qww, workspace=False))
    torch.cuda.synchronize()
    outs = []
    for i in range(6):
        with torch.cuda.stream(s1 if i % 2 == 0 else s2):
            outs.append(clq.clq_w4a4_accum_i32(Xqw, xsw, qww))
    torch.cuda.synchronize()
    for o in outs:
        assert np.array_equal(o.cpu().numpy(), refw)


def test_accum_i32_extremes(clq):
    """All codes +7 and alternating signs: |acc| reaches 49 K."""
    M, N, K, block = 48, 80, 4608, 64
    X = np.zeros((M, K), np.float16)
    X[:, 0] = np.float16(1.0)                 # a delta: every rotated entry is +-1
    X[1::2, 0] = np.float16(-1.0)
    W = np.zeros((N, K), np.float16)
    W[:, 0] = np.float16(1.0)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    acc = host(clq.clq_w4a4_accum_i32(Xq, xs, qw))
    _, xc, _ = oracle.quantize_act(X, block)
    _, wc, _ = oracle.quantize_weights(W, block)
    ref = oracle.gemm_i32(xc, wc)
    assert np.array_equal(acc, ref)
    assert np.abs(ref).max() == 49 * block


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("with_bias", [True, False])
def test_linear_fp16_tolerance(clq, M, N, K, with_bias):
    block = 64
    X = workloads.activations(M, K, "L1", seed=M + 1)
    W = workloads.weights(N, K, seed=N + 1)
    b = workloads.bias(N, seed=3) if with_bias else None
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    Y = clq.clq_w4a4_linear(Xq, xs, qw, None if b is None else dev(b))
    ref = oracle.linear(X, W, b, block)
    err = oracle.err_metric(host(Y).astype(np.float64), ref["y64"], ref["p64"], b)
    assert err <= TOL, err


def test_linear_row_stride_and_zero_rows(clq):
    M, N, K, block, ldy = 70, 136, 1152, 64, 256
    X = workloads.activations(M, K, "L1", seed=9)
    X[5] = 0
    X[66] = 0
    W = workloads.weights(N, K, seed=10)
    b = workloads.bias(N, seed=11)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    Ybig = torch.full((M, ldy), float("nan"), dtype=torch.float16, device="cuda")
    clq.clq_w4a4_linear(Xq, xs, qw, dev(b), out=Ybig[:, :N])
    Yh = host(Ybig)
    assert np.isnan(Yh[:, N:].astype(np.float32)).all()        # untouched padding
    ref = oracle.linear(X, W, b, block)
    assert oracle.err_metric(Yh[:, :N].astype(np.float64), ref["y64"], ref["p64"], b) <= TOL
    assert np.array_equal(Yh[5, :N], b) and np.array_equal(Yh[66, :N], b)   # zero rows -> bias


def test_linear_block128_perm(clq):
    M, N, K, block = 96, 192, 3072, 128
    X = workloads.activations(M, K, "L2", seed=12)
    W = workloads.weights(N, K, seed=13)
    b = workloads.bias(N, seed=14)
    perm = workloads.random_perm(K, seed=15)
    qw = clq.clq_quantize_weights(dev(W), block, dev(perm))
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block, dev(perm))
    acc = clq.clq_w4a4_accum_i32(Xq, xs, qw)
    Y = clq.clq_w4a4_linear(Xq, xs, qw, dev(b))
    ref = oracle.linear(X, W, b, block, perm)
    assert np.array_equal(host(acc), ref["acc"])
    assert oracle.err_metric(host(Y).astype(np.float64), ref["y64"], ref["p64"], b) <= TOL


# Rows too wide for the pipelined activation kernel (more than 256 blocks, or
# two staged copies beyond the LDS limit) go through the one-shot kernel.
@pytest.mark.parametrize("M,K,block", [(5, 12288, 32), (3, 32768, 128), (2, 32768, 64), (3, 17408, 64),
                                       (4, 32768, 32)])
def test_rotate_quant_wide_rows(clq, M, K, block):
    X = workloads.activations(M, K, "L1", seed=K + block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    ref_q, ref_c, ref_s = oracle.quantize_act(X, block)
    assert np.array_equal(host(xs), ref_s)
    assert np.array_equal(host(clq.clq_unswizzle_act(Xq, M, K)), ref_q)
    Xq8, xs8 = clq.clq_rotate_quant_act8(dev(X), block)
    _, ref_c8, ref_s8 = oracle.quantize_act(X, block, bits=8)
    assert np.array_equal(host(xs8), ref_s8)
    assert np.array_equal(host(clq.clq_unswizzle_act8(Xq8, M, K)), ref_c8)


def test_gemm_longest_rows(clq):
    # K = 32768, the largest accepted: |acc| <= 49 K and the widened
    # accumulators (256 x) stay within int32
    M, N, K, block = 40, 70, 32768, 128
    X = workloads.activations(M, K, "L1", seed=71)
    W = workloads.weights(N, K, seed=72)
    b = workloads.bias(N, seed=73)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    ref = oracle.linear(X, W, b, block)
    assert np.array_equal(host(clq.clq_w4a4_accum_i32(Xq, xs, qw)), ref["acc"])
    Y = clq.clq_w4a4_linear(Xq, xs, qw, dev(b))
    assert oracle.err_metric(host(Y).astype(np.float64), ref["y64"], ref["p64"], b) <= TOL


# ---- the single-linear configuration: 256 tokens x 1152 -> 1152, block 64 ----------

@pytest.mark.parametrize("with_bias", [True, False], ids=["bias", "nobias"])
@pytest.mark.parametrize("swap", ["none", "obs"])
def test_single_linear_config(clq, with_bias, swap):
    layer = workloads.C1.layers[0]
    M, K, N, block = layer.M, layer.K, layer.N, layer.block
    X, W, b = workloads.layer_inputs(layer)
    if not with_bias:
        b = None
    perm = perm_d = None
    if swap == "obs":
        # the swap vector derived from a separate calibration draw of the
        # same law (Sec. 3.3 outlier detection, abs-max metric), on the GPU,
        # checked against the oracle's derivation first
        from oracle import obs as oobs
        cal = workloads.calibration(4, M, K, "L1", seed=layer.seed + 3)
        sc = clq.clq_obs_channel_scores(dev(cal), "absmax")
        perm_d = clq.clq_obs_permutation(sc)
        perm = oobs.obs(cal, "absmax")[2]
        assert np.array_equal(host(perm_d), perm)
    qw = clq.clq_quantize_weights(dev(W), block, perm_d)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block, perm_d)
    Y = clq.clq_w4a4_linear(Xq, xs, qw, None if b is None else dev(b))
    acc = clq.clq_w4a4_accum_i32(Xq, xs, qw)
    ref = oracle.linear(X, W, b, block, perm)
    assert np.array_equal(host(xs), ref["x_scale"])
    assert np.array_equal(host(clq.clq_unswizzle_act(Xq, M, K)), ref["xq"])
    assert np.array_equal(host(qw.w_scale), ref["w_scale"])
    assert np.array_equal(host(clq.clq_unswizzle_weights(qw)), ref["wq"])
    assert np.array_equal(host(acc), ref["acc"])
    assert oracle.err_metric(host(Y).astype(np.float64), ref["y64"], ref["p64"], b) <= TOL


# ---- full-size layers (the shapes the benchmark times), sampled rows --------------

FULL = [l for w in (workloads.C2, workloads.C3, workloads.C4) for l in w.layers]


@pytest.mark.parametrize("layer", FULL, ids=[l.name for l in FULL])
def test_full_size_layer_sampled(clq, layer):
    X, W, b = workloads.layer_inputs(layer)
    qw = clq.clq_quantize_weights(dev(W), layer.block)
    Xd = dev(X)
    Xq, xs = clq.clq_rotate_quant_act(Xd, layer.block)
    Y = clq.clq_w4a4_linear(Xq, xs, qw, dev(b))
    rng = np.random.default_rng(layer.seed)
    rows = np.unique(np.concatenate([[0, layer.M - 1], rng.choice(layer.M, 30, replace=False)]))
    rows_t = torch.from_numpy(rows).cuda()
    Xq_s = host(clq.clq_unswizzle_act(Xq, layer.M, layer.K)[rows_t])
    xs_s, Y_s = host(xs[rows_t]), host(Y[rows_t])
    ref_xq, xc, ref_xs = oracle.quantize_act(X[rows], layer.block)
    assert np.array_equal(xs_s, ref_xs)
    assert np.array_equal(Xq_s, ref_xq)
    wq_ref, wc, ws_ref = oracle.quantize_weights(W, layer.block)
    assert np.array_equal(host(qw.w_scale), ws_ref)
    acc = oracle.gemm_i32(xc, wc)
    y64, p64 = oracle.epilogue(acc, ref_xs, ws_ref, b)
    assert oracle.err_metric(Y_s.astype(np.float64), y64, p64, b) <= TOL
    # the exact accumulators on the same rows, through the int32 variant
    acc_gpu = clq.clq_w4a4_accum_i32(Xq, xs, qw)
    assert np.array_equal(host(acc_gpu[rows_t]), acc)


# ---- serialised quantized weights ------------------------------------------------

def test_qweight_save_load_roundtrip(clq, tmp_path):
    N, K, block = 200, 1152, 64
    W = workloads.weights(N, K, seed=91)
    perm = workloads.random_perm(K, seed=92)
    qw = clq.clq_quantize_weights(dev(W), block, dev(perm), clip_ratio=0.9)
    path = str(tmp_path / "w.safetensors")
    clq.save_qweight(path, qw)
    back = clq.load_qweight(path)
    assert (back.N, back.K, back.block, back.bits, back.clip_ratio) == (N, K, block, 4, qw.clip_ratio)
    assert torch.equal(back.wq.cpu(), qw.wq.cpu()) and torch.equal(back.w_scale.cpu(), qw.w_scale.cpu())
    assert torch.equal(back.perm.cpu(), qw.perm.cpu())
    # the reloaded weight drives the linear exactly as the original
    X = workloads.activations(64, K, "L1", seed=93)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block, dev(perm))
    assert np.array_equal(host(clq.clq_w4a4_accum_i32(Xq, xs, back)), host(clq.clq_w4a4_accum_i32(Xq, xs, qw)))


# Every schedule the GEMM can take (the debug knob forces one: 256-token tiles
# with and without the split rule, the two-halves kernel on 128- and
# 64-token tiles) gives the same exact integer sums, and fp16 outputs within
# the tolerance of the oracle, on shapes that the automatic choice sends to
# each of them: few tiles, a ragged channel edge, a split-k shape and a
# large one.
FORCED_SHAPES = [(1024, 1152, 1152), (300, 1000, 640), (4096, 3456, 1152), (16384, 1152, 4608), (8192, 4608, 1152)]


@pytest.mark.parametrize("M,N,K", FORCED_SHAPES)
def test_forced_schedules_agree(clq, M, N, K):
    block = 64
    X = workloads.activations(M, K, "L1", seed=M + 1)
    W = workloads.weights(N, K, seed=N + 1)
    b = workloads.bias(N, seed=N + 2)
    qw = clq.clq_quantize_weights(dev(W), block)
    Xq, xs = clq.clq_rotate_quant_act(dev(X), block)
    rows = np.unique(np.r_[0:3, M // 2, M - 3:M])
    r = oracle.linear(X[rows], W, b, block)
    ref = None
    try:
        for force in (0, 1, 2, 3, 4):
            clq.clq_debug_set(3, force)
            plan = clq.clq_w4a4_schedule(M, N, K)
            expect = {1: 0, 2: 0, 3: 1, 4: 2}.get(force)
            assert expect is None or plan["kernel"] == expect, (force, plan)
            ws = torch.zeros(clq.clq_w4a4_workspace_bytes(), dtype=torch.uint8, device="cuda")
            acc = host(clq.clq_w4a4_accum_i32(Xq, xs, qw, workspace=ws))
            Y = host(clq.clq_w4a4_linear(Xq, xs, qw, dev(b), workspace=ws))
            assert clq.clq_w4a4_workspace_status(ws) == [0, 0, 0]
            if ref is None:
                ref, refY = acc, Y
                assert np.array_equal(acc[rows], r["acc"])
            else:
                assert np.array_equal(acc, ref), force
                # every kernel rounds the same products with the same
                # instruction: the fp16 outputs agree bit for bit too
                assert np.array_equal(Y.view(np.uint16), refY.view(np.uint16)), force
            assert oracle.err_metric(Y[rows].astype(np.float64), r["y64"], r["p64"], b) <= TOL, force
    finally:
        clq.clq_debug_set(3, 0)
