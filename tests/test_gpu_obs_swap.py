"""GPU parity of the OBS swap at the edges of its kernel: one, two, eight, 16 and 64
channels per thread, ragged last threads, all scores equal, signed zeros,
infinities and the type's largest and smallest values.  The swap is integer
arithmetic on an order, so it matches the CPU oracle exactly; NaN scores, which
the oracle does not rank, must still give a permutation with them on the left.
"""
import numpy as np
import pytest

from oracle import obs

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_24416_amd as m
    return m


def swap(clq, sc):
    out = clq.clq_obs_permutation(torch.from_numpy(sc).cuda())
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("D", [2, 6, 1022, 1152, 2046, 2048, 2050, 8192, 8194, 16384, 16386, 32770, 65534])
def test_swap_values(clq, D):
    print(f"\n[gpu case] D = {D}", flush=True)
    rng = np.random.default_rng(D)
    cases = [rng.standard_normal(D).astype(np.float32), np.full(D, 3.5, np.float32),
             rng.integers(-2, 3, size=D).astype(np.float32) * np.float32(0.0),      # both zeros: all equal
             rng.choice(np.array([np.inf, -np.inf, 3.4028235e38, -3.4028235e38, 1e-45, 0.0], np.float32), size=D)]
    for sc in cases:
        assert np.array_equal(swap(clq, sc), obs.permutation(sc))
    sc = rng.standard_normal(D).astype(np.float32)
    nan = rng.choice(D, size=max(1, D // 4), replace=False)
    sc[nan] = np.nan
    p = swap(clq, sc)
    assert np.array_equal(np.sort(p), np.arange(D))
    assert set(nan.tolist()) <= set(p[:D // 2].tolist()) if len(nan) <= D // 2 else True
