"""The routing lut and its compact map, as a table upload builds them: word and
workgroup edges, one queue and the largest number, both readings."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _bounds(kind, k, L, rng):
    if kind == "first":  # rises at the lowest lengths
        return np.arange(1, k) + 1
    if kind == "last":   # ... and at the highest
        return np.arange(L - k + 2, L + 1)
    return np.sort(rng.choice(np.arange(2, L + 1), k - 1, replace=False))


# max_len around 32 (a map word), 64 (a wave), 256 (a workgroup), and the largest
@pytest.mark.parametrize("kind", ["spread", "first", "last"])
@pytest.mark.parametrize("L,k", [(1, 1), (31, 5), (32, 32), (33, 7), (63, 2), (65, 64), (255, 9), (256, 256), (257, 200),
                                 (5000, 64), (32767, 256), (32768, 1), (32768, 256)])
def test_lut_and_map(L, k, kind):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(L + k)
    b = _bounds(kind, k, L, rng)
    print(f"lut L={L} k={k} {kind}", flush=True)
    g = E.read_table(E.upload_table(b, np.ones(k), L))
    want = np.searchsorted(b, np.arange(1, L + 1), side="right")
    assert np.array_equal(g["lut"][1:], want)
    assert np.array_equal(E.route_map_queues(g["route"], L)[1:], want)


@pytest.mark.parametrize("L,k", [(33, 2), (257, 20), (5000, 40), (32768, 100)])
def test_gapped_lut_and_map(L, k):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(L)
    ends = np.sort(rng.choice(np.arange(2, L + 1), 2 * k, replace=False))  # disjoint intervals, gaps between them
    lo, hi = ends[0::2], ends[1::2]
    print(f"gapped lut L={L} k={k}", flush=True)
    g = E.read_table(E.upload_table(lo[1:], np.ones(k), L, lo, hi, gapped=True))

    def queue(x):  # the Dispatcher's rule for lengths between queues i and i + 1
        i = int(np.searchsorted(lo, x, side="right")) - 1
        if i < 0 or i == k - 1 or x <= hi[i]:
            return max(i, 0)
        if 10 * x <= 11 * (hi[i] + 1):
            return i
        if 10 * x >= 9 * lo[i + 1]:
            return i + 1
        return i if x - hi[i] <= lo[i + 1] - x else i + 1

    want = np.array([queue(x) for x in range(1, L + 1)])
    assert np.array_equal(g["lut"][1:], want)
    assert np.array_equal(E.route_map_queues(g["route"], L)[1:], want)
