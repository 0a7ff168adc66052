"""Pools whose shares take more than one pass per workgroup (beyond 4,194,304
requests): chunk counts at their edges, data whose high keys fill one wave's
region, and the merge's two widths, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2601_21758_amd import workloads as W
from parity_util import check_admission

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FULL = 256 * 64 * 256  # requests of one full pass


# n, B, kind: G M is 4,096 slots up to B = 1,024 and 8,192 above
CASES = [(FULL + 1, 1024, "mixed"), (FULL + 256 * 256 * 16 - 1, 1025, "arrival"), (2 * FULL + 77, 4096, "mixed"),
         (FULL + 300, 40, "oldest_first"), (FULL + 999, 300, "all_equal"), (FULL + 12345, 2000, "hot_blocks"),
         (FULL + 5, 64, "rising"), (FULL + 70000, 256, "tombstones")]


def _pool(kind, n):
    if kind in W.ADVERSARIAL_KINDS:
        return W.adversarial(kind, n, 9)
    if kind == "rising":  # each chunk's scores above all before it: every pass raises the bars
        return np.full(n, 500, np.int32), np.linspace(400.0, 0.0, n).astype(np.float32), 500.0
    p = W.make_pool("three", n, 23, arrivals="poisson" if kind == "arrival" else "uniform", horizon=300.0, K=64)
    return p.length, p.arrival, p.now


@pytest.mark.parametrize("n,B,kind", CASES)
def test_step_beyond_one_pass(n, B, kind):
    from paper_2601_21758_amd import ewsjf as E
    L, A, now = _pool(kind, n)
    print(f"multi-pass step n={n} B={B} {kind}", flush=True)
    t = oracle.partition(np.clip(L[:50000], 1, None), init_queues=64, max_queues=64)
    cost = (0.01, 1e-4, 2e-9)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tab = E.upload_table(t.bounds, t.mean, 32768, t.lo, t.hi, t.count, t.sum)
    ids, top, nsel = (x.cpu().numpy() for x in E.step(dev(L), dev(A), now, tab, dev(W.THETA_MID), B, cost))
    rids, rtop, rnsel, rs = oracle.step(L, A, now, t, W.THETA_MID.reshape(1, 6), B, cost)
    check_admission(ids[0], top[0], nsel[0], rids[0], rtop[0], rnsel[0], rs[0])
    # the same scores through ewsjf_select, bit for bit against a sort
    s = E.score(dev(L), dev(A), now, tab, dev(W.THETA_MID), cost)
    i2, t2, n2 = (x.cpu().numpy() for x in E.select(s, B))
    assert np.array_equal(i2, ids) and np.array_equal(t2.view(np.int32), top.view(np.int32)) and n2[0] == nsel[0]
