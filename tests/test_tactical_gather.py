"""Algorithm 1 with its age thresholds: the rule's edges,
equal and NaN arrivals, arrival order and its reverse, rows of whole queues,
pools whose queues follow the sample's and the workgroups' periods, and one
whose sample misses the queue (the exact slow path); and which path answered."""
import numpy as np
import pytest

import oracle
import plan_util
from paper_2601_21758_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pool(kind, n, rng):
    L = W._lengths(rng, n, W.MIX_TWO)
    A = (rng.random(n) * 100).astype(np.float32)
    if kind == "oldest_first":
        A = np.sort(A)
    elif kind == "oldest_last":
        A = np.sort(A)[::-1].copy()
    elif kind == "equal":
        A[:] = 3.0
    elif kind == "nan":
        A[rng.random(n) < 0.3] = np.nan
        A[rng.random(n) < 0.1] = -0.0
    elif kind == "one_length":  # one queue holds everything
        L[:] = 40
        A = np.sort(A)
    elif kind == "long_only":   # the top queue is small
        L[:] = np.where(rng.random(n) < 0.02, L, 0)
    elif kind.startswith("every"):  # the short requests, the oldest of all, sit in every so-many-th chunk
        c = np.arange(n) // 256
        short = (L < 2048) & (c % int(kind[5:]) == 3)
        L[(L < 2048) & ~short] = 0
        A[short] *= 0.01
    elif kind == "unsampled":   # the sampled slots are empty, everything else is one queue
        L[:] = 40
        c = np.arange((n + 255) // 256, dtype=np.uint64)
        at = ((c * 0x9E3779B1) & 0xFFFFFFFF) >> 25
        for half in (0, 128):
            ids = (c * 256 + half + at).astype(np.int64)
            L[ids[ids < n]] = 0
    return L, A


# every queue fits one list up to 9,088 requests; the thresholds are taken up to B = 1,962, beyond 16,777,216 requests
# up to 443, and beyond 33,554,432 not at all
CASES = [(1, 3, "mixed"), (9088, 4096, "mixed"), (9089, 4096, "mixed"), (65536, 64, "mixed"), (65537, 1500, "oldest_first"), (300001, 1962, "mixed"), (300001, 1963, "mixed"),
         (1 << 20, 1024, "oldest_first"), (1 << 20, 1024, "oldest_last"), (200003, 700, "equal"), (150000, 300, "nan"),
         (500000, 1024, "one_length"), (400000, 1024, "long_only"), (100000, 500, "unsampled"),
         (4194304 + 513, 256, "mixed"),
         # periods of the sample's places and of the workgroups' shares, more than one share holds
         (1 << 21, 700, "every128"), (1 << 22, 1024, "every256"), ((1 << 22) + 3, 200, "every64"), (1 << 20, 1900, "every16"),
         (3000001, 1500, "every256"),
         # every second chunk sampled; and the size whose last chunk starts a pair by itself
         (16777216 + 77, 443, "mixed"), (16777216 + 300, 444, "mixed"), (33554432 + 5, 100, "mixed")]


@pytest.mark.parametrize("n,B,kind", CASES)
def test_tactical_gather(n, B, kind):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(n + B)
    L, A = _pool(kind, n, rng)
    print(f"tactical gather n={n} B={B} {kind}", flush=True)
    t = oracle.partition(np.clip(W._lengths(rng, 30000, W.MIX_TWO), 1, None), init_queues=32, max_queues=32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tab = E.upload_table(t.bounds, t.mean, 32768, t.lo, t.hi, t.count, t.sum)
    ec = E.new_empty_counters("cuda")
    Ld = dev(L)
    ws = E.Workspace("cuda")
    ids, nsel, qp, hs, rm = E.tactical_step(Ld, dev(A), 100.0, tab, dev(W.THETA_MID), B, 1 << 30, ec, tombstone=True,
                                            ws=ws)
    r = oracle.tactical_step(L, A, 100.0, t, np.zeros(t.k, np.int32), W.THETA_MID, B, 1 << 30)
    m = r.ids.size
    assert int(qp[0]) == r.q_prim and int(nsel[0]) == m
    got = ids.cpu().numpy()
    assert np.array_equal(got[:m], r.ids) and np.all(got[m:] == -1)
    left = L.copy()
    left[got[:m]] = 0
    assert np.array_equal(Ld.cpu().numpy(), left)
    # the rows came from their lists, but for the pool whose sample is empty
    p = plan_util.tactical(n, B)
    assert (p["rank"] > 0) == (n <= 9088 or B <= 1962 and n <= 1 << 24 or B <= 443 and n <= 1 << 25)
    if p["rank"] > 0:
        count = ws.buf[p["count_at"]:p["count_at"] + 12].view(torch.int32).cpu().numpy()
        assert (count > p["list_cap"]).any() == (kind == "unsampled")
        assert kind == "unsampled" or count.sum() >= m
