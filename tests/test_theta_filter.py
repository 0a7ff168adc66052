"""The many-vector step's filter: at the edges of its rule, and on pools where
it has to leave vectors to the plain kernels, every vector against the
oracle; and which path answered the ordinary ones."""
import numpy as np
import pytest

import oracle
import plan_util
from paper_2601_21758_amd import _lib as L_
from paper_2601_21758_amd import workloads as W
from parity_util import check_admission

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _thetas(kind, n, rng):
    th = rng.uniform(W.THETA_LO, W.THETA_HI, (n, 6))
    if kind == "wide":        # some weights negative
        th = W.THETA_MID * rng.uniform(0.3, 3.0, (n, 6))
        th[::3, 2] = -1e-3
    if kind == "fair_only":   # scores that do not depend on the wait
        th[:, :4] = 0.0
    if kind == "mixed":       # vectors that order the pool in opposite ways, and one that scores everything 0
        th[1::2, 2:4] = 0.0
        th[2] = 0.0
        th[4, 1] = -5.0
    return th.astype(np.float32)


def _pool(kind, n, rng):
    if kind in W.ADVERSARIAL_KINDS:
        return W.adversarial(kind, n, 5)
    p = W.make_pool("three" if n % 2 else "two", n, 17, arrivals="poisson" if kind == "arrival" else "uniform", K=64)
    length, arrival = p.length.copy(), p.arrival.copy()
    if kind in ("few_live", "some_live", "none_live"):  # fewer live requests than B, and more
        keep = rng.choice(n, {"few": 100, "some": 500, "none": 0}[kind[:-5]], replace=False)
        live = np.zeros(n, bool)
        live[keep] = True
        length[~live] = 0
    if kind == "one_run":     # every live request in one run of slots
        length[:] = np.where((np.arange(n) >= n // 3) & (np.arange(n) < n // 3 + 2500), length, 0)
    if kind == "always_waiting":  # arrivals of -inf: infinite scores
        arrival[rng.choice(n, 40, replace=False)] = -np.inf
    if kind == "just_arrived":  # no wait at all
        arrival[:] = p.now
    if kind == "hidden":      # the highest scores all sit between the sample's places
        length[:] = 4000
        stride = (n // 512) & ~3
        at = (np.arange(300) * stride + 24)
        length[at], arrival[at] = 3, 0.0
    return length, arrival, p.now


LIVE = ("few_live", "some_live", "none_live", "one_run")  # too few live requests for thresholds
# n, vectors, B: one workgroup's pool (8,192 requests, the sample's size) and, for fewer than 6 vectors,
# 262,144 requests are the rule's edges
CASES = [(8192, 3, 40, "uniform", ""), (8193, 3, 40, "uniform", ""), (8195, 64, 200, "arrival", ""),
         (12001, 2, 128, "uniform", ""), (262144, 2, 64, "uniform", ""), (262144, 2, 65, "uniform", ""), (131072, 3, 33, "arrival", ""), (262145, 5, 64, "uniform", ""),
         (262145, 6, 1000, "arrival", ""), (30000, 9, 4096, "uniform", ""), (65537, 63, 64, "uniform", ""),
         (100003, 48, 700, "arrival", "wide"), (70001, 64, 300, "just_arrived", ""), (65536, 64, 256, "few_live", ""),
         (300001, 6, 200, "some_live", ""), (1 << 20, 33, 256, "some_live", "wide"), (65536, 9, 64, "none_live", ""),
         (200000, 7, 256, "one_run", ""), (100001, 12, 64, "always_waiting", ""), (100001, 12, 64, "always_waiting", "mixed"),
         (300001, 17, 256, "hidden", ""), (131072, 40, 100, "tombstones", "mixed"), (90000, 64, 64, "uniform", "fair_only"),
         (65536, 70, 64, "uniform", "mixed"), (80000, 64, 500, "all_equal", ""), (120000, 40, 256, "hot_blocks", ""),
         (100000, 64, 64, "oldest_first", "wide"), (100001, 64, 64, "future_arrivals", "")]


@pytest.mark.parametrize("n,nt,B,kind,tk", CASES)
def test_filtered_step(n, nt, B, kind, tk):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(n + nt)
    L, A, now = _pool(kind, n, rng)
    theta = _thetas(tk, nt, rng)
    print(f"filtered step n={n} vectors={nt} B={B} {kind} {tk}", flush=True)
    t = oracle.partition(np.clip(L[:20000], 1, None), init_queues=64, max_queues=64)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tab = E.upload_table(t.bounds, t.mean, 32768, t.lo, t.hi, t.count, t.sum)
    ws = E.Workspace("cuda")
    ids, top, nsel = (x.cpu().numpy() for x in E.step(dev(L), dev(A), now, tab, dev(theta), B, ws=ws))
    plan = plan_util.plan(L_.OP_STEP, n, nt, B)
    if plan["filter"] > 0 and (kind in ("uniform", "arrival") and tk == "" or kind in LIVE):
        # answered from the survivors (a vector that the plain kernels answer overwrites these, the first one all)
        found = int(ws.buf[:4].view(torch.int32)[0])
        tau = ws.buf[256:256 + 4 * nt].view(torch.float32).cpu().numpy()
        live = int((L > 0).sum())
        few = kind in LIVE
        assert (found == live and (tau == -1).all()) if few else (B <= found <= plan["room"] and (tau > 0).all())
    rids, rtop, rnsel, rs = oracle.step(L, A, now, t, theta, B)
    if (theta >= 0).all() or tk == "":  # (with negative weights cancellation can exceed the score tolerance)
        for ti in range(nt):
            check_admission(ids[ti], top[ti], nsel[ti], rids[ti], rtop[ti], rnsel[ti], rs[ti])
    # each vector by itself (the one-vector kernels form the same keys)
    for ti in range(0, nt, 5):
        i1, t1, n1 = (x.cpu().numpy() for x in E.step(dev(L), dev(A), now, tab, dev(theta[ti]), B))
        assert np.array_equal(ids[ti], i1[0]) and nsel[ti] == n1[0]
        assert np.array_equal(top[ti].view(np.int32), t1[0].view(np.int32))
