"""GPU parity of the CLPS search at the edges of its batches and row splits.

Candidates are quantized and multiplied in batches of nearly equal size, at
most 8; row ratios run on one wave per row with 1, 2, 3, 4, 6 or 8 chunks per
lane up to 4096 columns and on a workgroup per row beyond.  Clip ratios match
the CPU oracle bit for bit (order statistics and fp32 arithmetic); errors are
sums of M N fp64 squares in another order, each term within a few 2^-53 of the
oracle's, so 1e-12 relative holds them with a wide margin.
"""
import numpy as np
import pytest

import oracle
from oracle import clps
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


@pytest.mark.parametrize("M,N,K,block,G,perm,gamma", [
    (40, 70, 512, 32, 7, False, 0.01), (300, 30, 576, 64, 8, True, 0.01), (33, 129, 1024, 128, 9, False, 0.2),
    (33, 300, 1152, 64, 17, True, 0.0), (20, 18, 2048, 128, 3, True, 0.5), (17, 33, 2560, 64, 2, False, 0.01),
    (9, 40, 4096, 32, 10, True, 0.01), (9, 20, 4160, 64, 9, True, 0.01), (300, 260, 128, 64, 256, False, 0.05),
    # two chunks per lane, many and few rows
    (9, 20, 8256, 64, 9, False, 0.01), (9, 300, 8320, 128, 17, True, 0.01), (9, 20, 16384, 32, 10, True, 0.01)])
def test_batches_and_widths(clq, M, N, K, block, G, perm, gamma):
    print(f"\n[gpu case] {M} x {N} x {K}, block {block}, {G} candidates, perm {perm}", flush=True)
    X = workloads.activations(M, K, "L1", seed=M + G)
    W = workloads.weights(N, K, seed=N + G)
    W[N // 2] = 0                              # a zero row counts as ratio 1
    W[N // 3, 1:] = 0                          # one value: every magnitude of its block is equal
    p = workloads.random_perm(K, seed=G) if perm else None
    Y0 = oracle.linear_fp64(X, W).astype(np.float32)
    al, er, best = clq.clq_clps_search(dev(X), dev(W), dev(Y0), block, perm=None if p is None else dev(p),
                                       gamma=gamma, grid=G)
    ral, rer, rbest = clps.search(X, W, Y0, block, p, gamma, G)
    torch.cuda.synchronize()
    assert np.array_equal(al.cpu().numpy(), ral)
    e = er.cpu().numpy()
    assert np.allclose(e, rer, rtol=1e-12, atol=0)
    b = int(best.cpu()[0])
    assert b == int(np.argmin(e))
    assert b == rbest or abs(rer[b] - rer[rbest]) <= 1e-12 * rer[rbest]
