"""Counting a ring range into a histogram: at the edges of a workgroup's share
and of the grid, odd length caps, ranges that wrap."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cap,begin,L", [(1, 1, 0, 1), (4095, 5000, 4000, 33), (4096, 4096, 1, 32768), (4097, 9001, 7000, 32767),
                                           (65537, 70001, 69999, 2), (262144, 262144, 5, 4099), (262145, 300000, 299999, 32766)])
def test_window_histogram(n, cap, begin, L):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(n)
    ring = np.exp(rng.uniform(-1, 11, cap)).astype(np.int32) - 1  # below 1 and above 32,768 too
    ring[rng.integers(0, cap, 3)] = [-5, 2**31 - 1, 0]
    print(f"window histogram n={n} cap={cap} begin={begin} L={L}", flush=True)
    want = np.bincount(np.clip(ring[(begin + np.arange(n)) % cap], 1, L), minlength=L + 1)
    hist = E.window_histogram(torch.from_numpy(ring).cuda(), L, begin=begin, n=n)
    assert np.array_equal(hist.cpu().numpy()[:L + 1], want)
