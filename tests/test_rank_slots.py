"""The rank merge's own slots: every count of slots per thread, lists longer
and shorter than a workgroup's own slots, slot counts that are no multiple of
them, and the largest slot count; waves whose keys overflow their region."""
import numpy as np
import pytest

import oracle
from paper_2601_21758_amd import workloads as W
from parity_util import check_admission

torch = pytest.importorskip("torch")


def own_slot(w, k, nwg, per):
    return k * nwg + (w + k * (nwg // per + 1)) % nwg


@pytest.mark.parametrize("slots", [16, 384, 1024, 2048, 4080, 4096, 4112, 8190, 8192, 8200, 8960, 9088])
def test_every_slot_has_one_owner(slots):
    nr = -(-slots // 1024)
    per = 16 if nr <= 4 else 32 if nr <= 8 else 36
    nwg = -(-slots // per)
    assert nwg <= 256
    own = [own_slot(w, k, nwg, per) for w in range(nwg) for k in range(per)]
    assert sorted(own) == list(range(nwg * per)) and nwg * per >= slots


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["mixed", "arrival", "oldest_first", "all_equal"])
@pytest.mark.parametrize("n,B", [(8195, 64), (12001, 500), (50000, 16), (131072, 2048), (262144, 1024), (262144, 4096),
                                 (524288, 3000), (1048577, 3000), (1048576, 4096)])
def test_rank_of_many_slots(n, B, kind):
    from paper_2601_21758_amd import ewsjf as E
    if kind in ("oldest_first", "all_equal"):
        L, A, now = W.adversarial(kind, n, 6)
    else:
        p = W.make_pool("three", n, 6, arrivals="uniform", horizon=300.0, K=16)
        L, A, now = p.length, p.arrival, p.now
        if kind == "arrival":
            A = np.sort(A)
    print(f"rank slots n={n} B={B} {kind}", flush=True)
    t = oracle.partition(np.clip(L, 1, None), init_queues=16, max_queues=16)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tab = E.upload_table(t.bounds, t.mean, 32768, t.lo, t.hi, t.count, t.sum)
    theta = W.THETA_MID.reshape(1, 6).astype(np.float32)
    ids, top, nsel = (x.cpu().numpy() for x in E.step(dev(L), dev(A), now, tab, dev(theta), B))
    rids, rtop, rnsel, rs = oracle.step(L, A, now, t, theta, B)
    check_admission(ids[0], top[0], nsel[0], rids[0], rtop[0], rnsel[0], rs[0])
