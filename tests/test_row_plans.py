"""Several rows at once: scores of a group of vectors with rows at every
alignment, selection with one to four chunks per wave, trials with shares of
one pass and of more and the statistics their merge keeps."""
import numpy as np
import pytest

import oracle
from paper_2601_21758_amd import workloads as W
from parity_util import check_admission, check_scores

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _pool(n, seed):
    p = W.make_pool("three", n, seed, arrivals="uniform", horizon=300.0, K=32)
    L = p.length.copy()
    L[::11] = 0
    t = oracle.partition(np.clip(L, 1, None), init_queues=32, max_queues=32)
    from paper_2601_21758_amd import ewsjf as E
    return L, p.arrival, p.now, t, E.upload_table(t.bounds, t.mean, 32768, t.lo, t.hi, t.count, t.sum)


# vectors: a group of 8, its edges, two groups; sizes of every remainder mod 4
@pytest.mark.parametrize("n,nt", [(1, 8), (4098, 7), (8195, 9), (4097, 17), (300004, 3)])
def test_score_rows(n, nt):
    from paper_2601_21758_amd import ewsjf as E
    L, A, now, t, tab = _pool(n, 3)
    th = np.random.default_rng(n).uniform(W.THETA_LO, W.THETA_HI, (nt, 6)).astype(np.float32)
    print(f"score rows n={n} vectors={nt}", flush=True)
    g = E.score(dev(L), dev(A), now, tab, dev(th), (0.01, 1e-4, 2e-9))
    check_scores(g.cpu().numpy(), oracle.score(L, A, now, t, th, (0.01, 1e-4, 2e-9)))
    assert np.array_equal(E.route(dev(L), tab).cpu().numpy(), oracle.route(L, t))


# chunks per wave: 1 (one round of the chip), 2, 4, and rows beyond one round; more of the B than larger shares hold
@pytest.mark.parametrize("n,rows,B", [(65536, 4, 64), (300001, 6, 700), (524287, 4, 256), (1000003, 4, 4096),
                                      (700001, 9, 33), (20000, 100, 4096), (9000, 256, 2048)])
def test_select_rows(n, rows, B):
    from paper_2601_21758_amd import ewsjf as E
    rng = np.random.default_rng(rows)
    s = rng.standard_normal((rows, n)).astype(np.float32)
    s[1] = np.round(s[1], 2)           # many equal scores
    s[2, : n // 2] = np.nan            # half not admissible
    s[3] = np.sort(s[3])[::-1]         # the highest first: clustered
    print(f"select rows n={n} rows={rows} B={B}", flush=True)
    ids, top, nsel = (x.cpu().numpy() for x in E.select(dev(s), B))
    for r in range(rows):
        key = np.where(np.isnan(s[r]), -np.inf, s[r])
        want = np.argsort(-key, kind="stable")[:B]
        assert nsel[r] == B and np.array_equal(ids[r], want)
        assert np.array_equal(top[r], s[r][want])


# capacity, pools, B: shares of one pass, of two, of many; few workgroups per pool; one pool past a round of the chip
@pytest.mark.parametrize("cap,pools,B", [(65536, 3, 64), (262144, 40, 100), (1 << 20, 16, 512), (1 << 19, 100, 64),
                                         (100004, 70, 300), (262144, 17, 513), (131072, 257, 32), (65536, 129, 64)])
def test_trial_shares(cap, pools, B):
    from paper_2601_21758_amd import ewsjf as E
    from paper_2601_21758_amd.trial import Trial
    L, A, now, t, tab = _pool(cap, 5)
    th = np.random.default_rng(cap).uniform(W.THETA_LO, W.THETA_HI, (pools, 6)).astype(np.float32)
    tr = Trial(cap, th, B, tab)
    tr.start(L, A)
    new = _pool(777, 6)
    print(f"trial capacity={cap} pools={pools} B={B}", flush=True)
    tr.pos = cap - 300  # the arrivals wrap
    ids, top, nsel = (x.cpu().numpy() for x in tr.step(dev(new[0]), dev(new[1]), now))
    L2, A2 = L.copy(), A.copy()
    at = (cap - 300 + np.arange(777)) % cap
    L2[at], A2[at] = new[0], new[1]
    for p in sorted({0, 1, pools // 2, pools - 1}):
        rids, rtop, rnsel, rs = oracle.step(L2, A2, now, t, th[p:p + 1], B)
        check_admission(ids[p], top[p], nsel[p], rids[0], rtop[0], rnsel[0], rs[0])
        left = L2.copy()
        left[ids[p][:nsel[p]]] = 0
        assert np.array_equal(tr.len[p].cpu().numpy(), left)
        assert np.array_equal(tr.arr[p].cpu().numpy(), A2)
        # the statistics of the admitted requests, which the merge keeps: whole numbers exactly, the sums of at most
        # B terms within B roundings of binary64
        i = ids[p][:nsel[p]]
        wait = np.maximum(0.0, np.float64(np.float32(now)) - A2[i].astype(np.float64))
        st = tr.stats[p].cpu().numpy()
        assert st[0] == nsel[p] and st[1] == L2[i].astype(np.int64).sum() and st[7] == 1 and st[4] == wait.max()
        assert np.allclose(st[2:4], [wait.sum(), (wait * wait).sum()], rtol=B * 2.3e-16, atol=0)
        assert np.array_equal(tr.queue_admits[p].cpu().numpy()[:t.k], np.bincount(oracle.route(L2[i], t), minlength=t.k))
