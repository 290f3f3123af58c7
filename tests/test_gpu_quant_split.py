"""GPU parity of the rotate+quantize kernel at the edges of its split.

A lane owns 8 columns of four rows; the widths below change how many four-row
groups share a workgroup (1, 2, 4, 8, groups that end inside a wave), how many
chunks a lane holds (one up to 8192 columns, two up to 16384, none beyond), where
a gathered row is staged, and which few rows take a workgroup each, or
run in batches of 8.  Codes and scales match the CPU oracle bit for bit, padding
rows hold zero codes.
"""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_24416_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("with_perm", [False, True])
@pytest.mark.parametrize("M,K,block", [
    (1, 64, 32), (2049, 64, 64), (4100, 192, 32), (1030, 576, 64), (2100, 1152, 64), (4100, 1152, 128),
    (35, 8192, 128), (33, 8256, 64), (31, 8320, 128), (5, 16384, 32), (3, 16448, 64), (2, 32768, 128),
    # the last row counts with a workgroup each, and the first without
    (128, 4160, 32), (192, 4160, 32), (193, 4160, 32), (128, 6208, 32), (256, 8256, 32), (257, 8256, 32),
    (128, 8256, 64), (192, 8256, 64), (193, 8256, 64), (64, 12416, 128), (65, 12416, 128),
    # fp6 rows in batches of 8: the first row count of 256 compute units' second
    # round that takes them and the last that does not, ragged last batches
    (3393, 4160, 64), (3392, 4160, 64), (4070, 5120, 64), (6001, 4544, 64), (4096, 4608, 64), (4096, 5184, 64)])
def test_codes_and_scales(clq, M, K, block, with_perm):
    print(f"\n[gpu case] {M} x {K}, block {block}, perm {with_perm}", flush=True)
    X = workloads.activations(M, K, "L1", seed=M + K + block)
    perm = workloads.random_perm(K, seed=K) if with_perm else None
    pd = None if perm is None else dev(perm)
    for bits, act, uns in ((4, clq.clq_rotate_quant_act, lambda q, R: clq.clq_unswizzle_act(q, R, K)),
                           (6, clq.clq_rotate_quant_act_f6, lambda q, R: clq.clq_unswizzle_f6(q, R, K, False)),
                           (8, clq.clq_rotate_quant_act8, lambda q, R: clq.clq_unswizzle_act8(q, R, K))):
        rows = (M + 31) // 32 * 32
        q, s = act(dev(X), block, perm=pd)
        ref_q, ref_c, ref_s = oracle.quantize_act(X, block, perm, bits=8 if bits == 8 else 4)
        got = host(uns(q, rows))
        assert np.array_equal(host(s), ref_s), bits
        assert np.array_equal(got[:M], ref_c if bits == 8 else ref_q), bits
        assert not got[M:].any(), bits


# weights have a row order of their own, a clamp and a clip ratio: groups per
# workgroup, one and two chunks per lane, a workgroup per row for few rows and
# past 16384 columns, ragged row counts
@pytest.mark.parametrize("with_perm", [False, True])
@pytest.mark.parametrize("N,K,block", [
    (1, 64, 32), (2090, 192, 64), (2090, 1152, 128), (1100, 1792, 64), (600, 8192, 128), (33, 8192, 64), (300, 8256, 64),
    (290, 8320, 128), (129, 8256, 32), (270, 16384, 32), (200, 16384, 64), (70, 16384, 128), (97, 16448, 64),
    (40, 16448, 32), (35, 32768, 128), (20, 32768, 32)])
def test_weight_codes_and_scales(clq, N, K, block, with_perm):
    print(f"\n[gpu case] weights {N} x {K}, block {block}, perm {with_perm}", flush=True)
    W = workloads.weights(N, K, seed=N + K + block)
    W[N // 2] = 0
    perm = workloads.random_perm(K, seed=K) if with_perm else None
    pd = None if perm is None else dev(perm)
    rows = (N + 63) // 64 * 64
    for bits, quant, uns in (
            (4, clq.clq_quantize_weights, clq.clq_unswizzle_weights),
            (6, clq.clq_quantize_weights_f6, lambda q: clq.clq_unswizzle_f6(q.wq, rows, K, True)),
            (8, clq.clq_quantize_weights8, clq.clq_unswizzle_weights8)):
        for clip in (1.0, 0.71875):
            qw = quant(dev(W), block, perm=pd, clip_ratio=clip)
            ref_q, ref_c, ref_s = oracle.quantize_weights(W, block, perm, clip, bits=8 if bits == 8 else 4)
            got = host(uns(qw))
            assert np.array_equal(host(qw.w_scale), ref_s), (bits, clip)
            assert np.array_equal(got[:N], ref_c if bits == 8 else ref_q), (bits, clip)
            assert not got[N:].any(), (bits, clip)
