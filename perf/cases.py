"""The workloads this framework's speed is measured on.

Each case is one call (or one short chain of calls) that a program using the
scheduler makes: the scheduling step over pools of every size, the step under
many parameter vectors, the streaming scheduler's step, Refine-and-Prune from
a window and from its histogram, Algorithm 1's batch rule, proposal trials,
and the separate route / score / select calls.  Sizes and length mixtures are
those of the seeded workloads (workloads.py), the benchmark and the tests.

`prepare` draws the inputs on the GPU from the seed and builds what such a
program keeps between calls (the queue table, output buffers, workspaces, the
streaming scheduler); `run` is one pass; `exact` evaluates the same
definitions in plain numpy / torch in 64 bits, without the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_21758_amd import ewsjf as E
from paper_2601_21758_amd import workloads as W
from paper_2601_21758_amd.streaming import StreamingScheduler
from paper_2601_21758_amd.trial import Trial

MAX_LEN = 32768
RATE = 1e4           # arrivals per second
STREAM_BATCHES = 2048  # distinct arrival batches a streaming state holds
TRIAL_BATCHES = 256
ALPHA, EPS, MIN_WIDTH = 2.0, 1e-6, 16


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # A small deployment's step: 4,096 pending requests, 16 queues, 64 admissions.
        dict(name="step_4k", kind="step", n=4096, theta=1, B=64, K=16, mix="two", order="mixed", holes=0.0, c2=0.0),
        # An ordinary step: a quarter of a million pending requests of three length modes, 64 queues.
        dict(name="step_256k", kind="step", n=262144, theta=1, B=256, K=64, mix="three", order="mixed", holes=0.0,
             c2=0.0),
        # The headline step: 4M pending requests in arrival order, 256 queues, 1,024 admissions.
        dict(name="step_4m", kind="step", n=4194304, theta=1, B=1024, K=256, mix="two", order="arrival", holes=0.0,
             c2=0.0),
        # The largest pool, of a size that divides nothing, a tenth of its slots empty, a quadratic prefill cost.
        dict(name="step_9m", kind="step", n=9437189, theta=1, B=1500, K=64, mix="three", order="mixed", holes=0.1,
             c2=2e-9),
        # The meta-optimizer's scan: one 1M pool under 256 parameter vectors.
        dict(name="theta_256x1m", kind="step", n=1048576, theta=256, B=256, K=64, mix="three", order="mixed",
             holes=0.0, c2=0.0),
        # The streaming scheduler's step: a 1M ring, 4,096 arrivals in, 512 admitted and emptied.
        dict(name="stream_1m", kind="stream", n=1048576, per=4096, B=512, K=64, window=65536, bubbles=0),
        # The strategic loop over a large window: a 1M window into 256 queues.
        dict(name="partition_1m", kind="partition", W=1048576, K=256, mix="two", init=0, hist=0),
        # The streaming scheduler's repartition: recount the 65,536-length window from the length log, then
        # Refine-and-Prune from the histogram, 64 queues.
        dict(name="repartition_64k", kind="partition", W=65536, K=64, mix="two", init=0, hist=1),
        # The paper's own Stage 1 (k-means, k = 3) over a window of three length modes.
        dict(name="kmeans3_256k", kind="partition", W=262144, K=64, mix="three", init=1, hist=0),
        # Algorithm 1's batch rule (queue heads, ArgMax, fill, backfill) over the 4M pool.
        dict(name="tactical_4m", kind="tactical", n=4194304, B=1024, K=256, mix="two", order="arrival"),
        # Trials of 16 parameter proposals, each on its own 1M ring with common arrivals.
        dict(name="trial_16x1m", kind="trial", n=1048576, pools=16, per=4096, B=512, K=64),
        # Route, score and select as separate calls: an odd pool size, four parameter vectors.
        dict(name="parts_1m", kind="parts", n=1000003, theta=4, B=256, K=64, mix="three", order="mixed", holes=0.1,
             c2=0.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "theta", "stream", "partition", "partition", "tactical", "trial",
                       "parts"])
    mix, order = rng.choice(["two", "three"]), rng.choice(["mixed", "arrival"])
    K = rng.choice([16, 32, 64, 128, 256])
    holes, c2 = rng.choice([0.0, 0.0, 0.1, 0.5]), rng.choice([0.0, 0.0, 2e-9])
    if kind == "step":
        n = _log(rng, 1000, 9400000)
        return dict(kind="step", n=n, theta=1, B=min(_log(rng, 16, 4096), max(16, n // 64)), K=K, mix=mix, order=order,
                    holes=holes, c2=c2)
    if kind == "theta":
        return dict(kind="step", n=_log(rng, 4096, 1048576), theta=_log(rng, 2, 256), B=_log(rng, 16, 256), K=K,
                    mix=mix, order=order, holes=holes, c2=c2)
    if kind == "stream":
        n = _log(rng, 65536, 1048576)
        return dict(kind="stream", n=n, per=_log(rng, 64, 4096), B=_log(rng, 32, 512), K=rng.choice([16, 64]),
                    window=_log(rng, 4096, 65536), bubbles=rng.choice([0, 1]))
    if kind == "partition":
        init = rng.choice([0, 0, 1])
        return dict(kind="partition", W=_log(rng, 1000, 262144 if init else 1048576), K=K if K >= 64 else 64, mix=mix,
                    init=init, hist=rng.choice([0, 1]))
    if kind == "tactical":
        n = _log(rng, 16384, 4194304)
        return dict(kind="tactical", n=n, B=min(_log(rng, 16, 1024), n // 64), K=K, mix=mix, order=order)
    if kind == "trial":
        return dict(kind="trial", n=4 * _log(rng, 4096, 262144), pools=_log(rng, 2, 16), per=_log(rng, 64, 4096),
                    B=_log(rng, 32, 512), K=rng.choice([16, 64]))
    return dict(kind="parts", n=_log(rng, 1000, 1048576), theta=_log(rng, 1, 4), B=_log(rng, 16, 256), K=K, mix=mix,
                order=order, holes=holes, c2=c2)


# ---------------------------------------------------------------------------
# Inputs, on the GPU, from the seed
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def _lengths(g, n, mix, p_short=None):
    """Prompt lengths of a workload's mixture (p_short: the weight of the first mode, a number or one per request)."""
    comps = W.MIX_TWO if mix == "two" else W.MIX_THREE
    u = torch.rand(n, generator=g, device="cuda")
    z = torch.randn(n, generator=g, device="cuda")
    if p_short is None:
        cum = torch.cumsum(torch.tensor([c[0] for c in comps], device="cuda"), 0)[:-1].contiguous()
        c = torch.searchsorted(cum, u, right=True)
    else:
        c = (u >= p_short).long()
    t = torch.tensor([[math.log(m), s, lo, hi] for _, m, s, lo, hi in comps], device="cuda")[c]
    x = torch.round(torch.exp(t[:, 0] + t[:, 1] * z))
    return torch.minimum(torch.maximum(x, t[:, 2]), t[:, 3]).to(torch.int32)


def _arrivals(g, n, order, horizon):
    """Uniform arrivals over the horizon; in arrival order they are a Poisson process given its count."""
    a = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * horizon
    if order == "arrival":
        a = torch.sort(a).values
    return a.to(torch.float32)


def _thetas(g, n):
    lo, hi = (torch.tensor(x, device="cuda") for x in (W.THETA_LO, W.THETA_HI))
    if n == 1:
        return torch.from_numpy(W.THETA_MID.reshape(1, 6).copy()).cuda()
    return (lo + (hi - lo) * torch.rand(n, 6, generator=g, device="cuda", dtype=torch.float64)).to(torch.float32)


def _cost(case):
    return (0.01, 1e-4, float(case.get("c2", 0.0)))


def _pool(case, seed):
    """length, arrival, now, theta and partition window of a pool case."""
    g = _gen(seed)
    n = case["n"]
    horizon = n / RATE if case["order"] == "arrival" else 300.0
    length = _lengths(g, n, case["mix"])
    arrival = _arrivals(g, n, case["order"], horizon)
    window = length[-max(1, n // 4):].clone()
    if case.get("holes", 0.0) > 0.0:
        length[torch.rand(n, generator=g, device="cuda") < case["holes"]] = 0
    now = float(np.float32(horizon))
    return length, arrival, now, _thetas(g, case.get("theta", 1)), window


def _stream_inputs(case, seed, batches, order="arrival"):
    """A full ring and the arrival batches that follow it, the share of short requests falling from 0.9 to 0.3."""
    g = _gen(seed)
    C, per = case["n"], case["per"]
    n = C + batches * per
    p = torch.full((n,), 0.9, device="cuda")
    p[C:] = torch.linspace(0.9, 0.3, batches, device="cuda").repeat_interleave(per)
    length = _lengths(g, n, "two", p)
    arrival = _arrivals(g, n, order, n / RATE)
    return length[:C], arrival[:C], length[C:].view(batches, per), arrival[C:].view(batches, per)


def _params(K, init=0):
    return E.params(init_mode=init, init_queues=K, max_queues=K, min_width=MIN_WIDTH, max_len=MAX_LEN, alpha=ALPHA,
                    eps=EPS)


def _proposals(g, P):
    mid = torch.from_numpy(W.THETA_MID).cuda().double()
    return (mid * (0.3 + 2.7 * torch.rand(P, 6, generator=g, device="cuda", dtype=torch.float64))).float()


def _window(case, seed):
    """The window as the last W entries of a length log of 2 W, and the place in it where the window begins."""
    g = _gen(seed)
    n = case["W"]
    p = 0.6 if case["hist"] else None  # a streaming window is drawn in mid-drift
    window = _lengths(g, n, case["mix"], p if case["mix"] == "two" else None)
    if not case["hist"]:
        return window, 0
    begin = n + n // 3  # the window wraps around the log's end
    log = torch.zeros(2 * n, dtype=torch.int32, device="cuda")
    log[(begin + torch.arange(n, device="cuda")) % (2 * n)] = window
    return log, begin


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind in ("step", "tactical", "parts"):
        length, arrival, now, theta, window = _pool(case, seed)
        s.update(len=length, arr=arrival, now=now, theta=theta, B=case["B"], cost=E.cost(*_cost(case)),
                 table=E.partition(window, _params(case["K"])), ws=E.Workspace(length.device))
        s["out"] = (torch.empty((theta.shape[0], case["B"]), dtype=torch.int32, device="cuda"),
                    torch.empty((theta.shape[0], case["B"]), dtype=torch.float32, device="cuda"),
                    torch.empty((theta.shape[0],), dtype=torch.int32, device="cuda"))
        if kind == "tactical":
            s["k"] = E.read_table(s["table"])["k"]
            s["empty"] = E.new_empty_counters("cuda")
        if kind == "parts":
            s["qid"] = torch.empty_like(length)
            s["score"] = torch.empty((theta.shape[0], case["n"]), dtype=torch.float32, device="cuda")
    elif kind == "stream":
        L0, A0, dl, da = _stream_inputs(case, seed, STREAM_BATCHES)
        sched = StreamingScheduler(case["n"], case["window"], case["B"], _params(case["K"]), W.THETA_MID,
                                   device="cuda", bubbles=(64, 2 * case["K"]) if case["bubbles"] else None)
        sched.fill(L0, A0)
        s.update(sched=sched, len=list(dl.unbind(0)), arr=list(da.unbind(0)), now=da[:, -1].tolist(), i=0)
    elif kind == "trial":
        L0, A0, dl, da = _stream_inputs(case, seed, TRIAL_BATCHES)
        table = E.partition(L0[-min(65536, case["n"]):].contiguous(), _params(case["K"]))
        theta = _proposals(_gen(seed + 1), case["pools"])
        trial = Trial(case["n"], theta.cpu().numpy(), case["B"], table, device="cuda")
        trial.start(L0, A0)
        s.update(trial=trial, len=list(dl.unbind(0)), arr=list(da.unbind(0)), now=da[:, -1].tolist(), i=0)
    else:
        window, begin = _window(case, seed)
        s.update(window=window, begin=begin, W=case["W"], hist=None, params=_params(case["K"], case["init"]),
                 table=E.new_table("cuda"), ws=E.Workspace("cuda"))
        if case["hist"]:
            s["hist"] = torch.empty(MAX_LEN + 1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    return s


def run(s):
    kind = s["kind"]
    if kind == "step":
        ids, top, n_sel = E.step(s["len"], s["arr"], s["now"], s["table"], s["theta"], s["B"], s["cost"],
                                 out=s["out"], ws=s["ws"])
        return {"ids": ids, "top": top, "n_sel": n_sel}
    if kind == "stream":
        i = s["i"]
        s["i"] = (i + 1) % len(s["now"])
        sched = s["sched"]
        ids, top, n_sel = sched.step(s["now"][i], True, s["len"][i], s["arr"][i])
        return {"ids": ids, "top": top, "n_sel": n_sel, "ring_len": sched.len, "ring_arrival": sched.arr,
                "log": sched.log}
    if kind == "partition":
        if s["hist"] is None:
            return {"table": E.partition(s["window"], s["params"], table=s["table"], ws=s["ws"])}
        E.window_histogram(s["window"], MAX_LEN, hist=s["hist"], begin=s["begin"], n=s["W"])
        return {"table": E.partition_hist(s["hist"], s["params"], table=s["table"], ws=s["ws"]), "hist": s["hist"]}
    if kind == "tactical":
        ids, n_sel, q_prim, head, removed = E.tactical_step(
            s["len"], s["arr"], s["now"], s["table"], s["theta"], s["B"], 1 << 30, s["empty"], cost_=s["cost"],
            ws=s["ws"])
        k = s["k"]  # the entries past the table's queues are not written
        return {"ids": ids, "n_sel": n_sel, "q_prim": q_prim, "head_score": head[:k], "removed": removed[:k],
                "table": s["table"], "empty": s["empty"]}
    if kind == "trial":
        i = s["i"]
        s["i"] = (i + 1) % len(s["now"])
        t = s["trial"]
        ids, top, n_sel = t.step(s["len"][i], s["arr"][i], s["now"][i])
        return {"ids": ids, "top": top, "n_sel": n_sel, "stats": t.stats, "queue_admits": t.queue_admits,
                "len": t.len, "arrival": t.arr}
    qid = E.route(s["len"], s["table"], out=s["qid"])
    score = E.score(s["len"], s["arr"], s["now"], s["table"], s["theta"], s["cost"], out=s["score"])
    ids, top, n_sel = E.select(score, s["B"], out=s["out"], ws=s["ws"])
    return {"qid": qid, "score": score, "ids": ids, "top": top, "n_sel": n_sel}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
TABLE_BYTES = 49 * 1024   # a queue table, written or read
MAP_BYTES = 12 * 1024     # the routing map and the queue means a step reads
PHI_FLOPS = 14            # one score of one request
TERM_FLOPS = 5            # one more score of it (its per-request terms are shared)


def work(case):
    kind = case["kind"]
    if kind in ("step", "parts"):
        n, t, B = case["n"], case["theta"], case["B"]
        by = 8 * n + MAP_BYTES + 24 * t + 8 * t * B + 4 * t
        if kind == "parts":
            by = 4 * n + 4 * n + 8 * n + 2 * 4 * n * t + 8 * t * B + 4 * t + 3 * MAP_BYTES
        return {"bytes": by, "flops": n * (PHI_FLOPS - TERM_FLOPS + TERM_FLOPS * t)}
    if kind == "stream":
        n, per, B = case["n"], case["per"], case["B"]
        return {"bytes": 8 * n + 8 * per + 4 * per + MAP_BYTES + 12 * B, "flops": n * PHI_FLOPS}
    if kind == "tactical":
        return {"bytes": 8 * case["n"] + MAP_BYTES + 4 * case["B"] + 8 * 256, "flops": 2 * case["n"]}
    if kind == "trial":
        n, P, per, B = case["n"], case["pools"], case["per"], case["B"]
        return {"bytes": P * (8 * n + 12 * B + 64 + 8 * 256) + 8 * per + MAP_BYTES, "flops": P * n * PHI_FLOPS}
    return {"bytes": 4 * case["W"] + TABLE_BYTES + (4 * (MAX_LEN + 1) if case["hist"] else 0), "flops": 2 * case["W"]}


def tolerance(case):
    if case["kind"] == "partition":
        return "exact"
    # Scores in binary32 (a reciprocal, a log2 and about eight rounded operations): measured up to 9.5e-8 (norm) and
    # 3.1e-7 (one value) against 64 bits.  Requests whose scores differ by less trade places in the admitted order:
    # up to 0.13% of the ids.  Four times each.
    return {"rel": 4e-7, "max": 1.2e-6, "differ": 0.005}


# ---------------------------------------------------------------------------
# The same definitions in plain numpy / torch, in 64 bits
# ---------------------------------------------------------------------------
TABLE_DTYPE = np.dtype([("head", "<i4", 6), ("n_window", "<i8"), ("bounds", "<i4", 256), ("lo", "<i4", 256),
                        ("hi", "<i4", 256), ("count", "<i8", 256), ("sum", "<i8", 256), ("mean", "<f8", 256),
                        ("lut", "u1", MAX_LEN + 16), ("route", "<u8", MAX_LEN // 32 + 2)])


def _kmeans3(PN, PS, V):
    """The split (i, j) of V distinct values into three clusters of least squared error, ties to the smallest."""
    n, s = PN.astype(np.float64), PS.astype(np.float64)
    best = (-1.0, 0, 0)
    for i in range(1, V - 1):
        a, b = n[i + 1:V] - n[i], s[i + 1:V] - s[i]
        c, d = n[V] - n[i + 1:V], s[V] - s[i + 1:V]
        F = ((s[i] * s[i]) / n[i] + (b * b) / a) + (d * d) / c
        j = int(np.argmax(F))
        if F[j] > best[0]:
            best = (float(F[j]), i, i + 1 + j)
    return best[1], best[2]


def _refine_and_prune(window, K, init):
    """Refine-and-Prune of a window of lengths: the queues' (lo, hi, count, sum), and the stage sizes."""
    v, c = np.unique(np.clip(window, 1, MAX_LEN), return_counts=True)
    v, V = v.astype(np.int64), v.size
    PN = np.concatenate([[0], np.cumsum(c)])
    PS = np.concatenate([[0], np.cumsum(c * v)])
    if init == 0:
        b = (v - v[0]) * K // (v[-1] - v[0] + 1)
        starts = np.concatenate([[0], 1 + np.flatnonzero(np.diff(b))])
    elif V <= 3:
        starts = np.arange(V)
    else:
        starts = np.array([0, *_kmeans3(PN, PS, V)])
    n_coarse = starts.size
    while True:  # every gap above alpha times its cluster's mean gap is cut, until none is
        ends = np.append(starts[1:], V)
        seg = np.repeat(np.arange(starts.size), ends - starts)[:-1]
        last = np.isin(np.arange(V - 1), ends - 1)
        size, span = (ends - starts)[seg], (v[ends - 1] - v[starts])[seg]
        cut = ~last & (size >= 3) & (span >= MIN_WIDTH) & (np.diff(v) * (size - 1.0) > ALPHA * span)
        if not cut.any():
            break
        starts = np.sort(np.concatenate([starts, 1 + np.flatnonzero(cut)]))
    ends = np.append(starts[1:], V)
    lo, hi = list(v[starts]), list(v[ends - 1])
    n, s = list(PN[ends] - PN[starts]), list(PS[ends] - PS[starts])
    n_leaves = len(lo)

    def utility(i):
        ra, rb = float(n[i]) / float(hi[i] - lo[i] + 1), float(n[i + 1]) / float(hi[i + 1] - lo[i + 1] + 1)
        return (ra + rb) / (abs(float(s[i + 1]) / float(n[i + 1]) - float(s[i]) / float(n[i])) + EPS)

    u = [utility(i) for i in range(len(lo) - 1)]
    while len(lo) > K:
        i = int(np.argmin(u))
        hi[i], n[i], s[i] = hi[i + 1], n[i] + n[i + 1], s[i] + s[i + 1]
        for x in (lo, hi, n, s):
            del x[i + 1]
        del u[i]
        if i < len(u):
            u[i] = utility(i)
        if i > 0:
            u[i - 1] = utility(i - 1)
    return tuple(np.array(x, np.int64) for x in (lo, hi, n, s)), V, n_coarse, n_leaves


def _table(window, K, init=0):
    """The queue table as the library lays it out."""
    (lo, hi, n, s), V, n_coarse, n_leaves = _refine_and_prune(window, K, init)
    k = lo.size
    t = np.zeros(1, TABLE_DTYPE)[0]
    t["head"] = [k, MAX_LEN, V, n_coarse, n_leaves, 0]
    t["n_window"] = window.size
    t["bounds"][:k - 1], t["lo"][:k], t["hi"][:k], t["count"][:k], t["sum"][:k] = lo[1:], lo, hi, n, s
    t["mean"][:k] = s.astype(np.float64) / n.astype(np.float64)
    q = np.searchsorted(lo[1:], np.arange(MAX_LEN + 64), side="right")
    q[0] = 0
    q[MAX_LEN + 1:] = q[MAX_LEN]
    t["lut"][:MAX_LEN + 1] = q[:MAX_LEN + 1]
    rise = np.diff(q, prepend=0).astype(np.uint64)[:32 * (MAX_LEN // 32 + 2)].reshape(-1, 32)
    base = q[np.maximum(32 * np.arange(MAX_LEN // 32 + 2) - 1, 0)].astype(np.uint64)
    t["route"] = (base << np.uint64(32)) | (rise << np.arange(32, dtype=np.uint64)).sum(1, dtype=np.uint64)
    return t


def _host(x):
    return x.cpu().numpy()


def _queues(length, table):
    bounds = torch.from_numpy(table["bounds"][:table["head"][0] - 1].astype(np.int64)).cuda()
    return torch.searchsorted(bounds, length.long().clamp(1, MAX_LEN), right=True)


def _phi(length, arrival, now, table, q, theta, cost):
    """Phi of every request (NaN where the slot is empty), binary64."""
    mean = torch.from_numpy(table["mean"].copy()).cuda()[q]
    th = theta.double()
    b = length.double()
    c = cost[0] + cost[1] * b + cost[2] * b * b
    wait = torch.clamp(float(np.float32(now)) - arrival.double(), min=0.0)
    phi = (q + 1).double() / (b + 1.0) * ((th[0] * mean + th[1]) + (th[2] * mean + th[3]) * (wait / c)
                                          + (th[4] * mean + th[5]) * torch.log(b + 1.0))
    return torch.where(length > 0, phi, torch.full_like(phi, math.nan))


def _top(phi, B):
    """The B highest scores, their ids and how many there are."""
    live = torch.isfinite(phi)
    m = min(B, int(live.sum()))
    x = torch.where(live, phi, torch.full_like(phi, -math.inf))
    val, idx = torch.topk(x, m, sorted=True)
    ids = torch.full((B,), -1, dtype=torch.int64, device="cuda")
    top = torch.full((B,), math.nan, dtype=torch.float64, device="cuda")
    ids[:m], top[:m] = idx, val
    return ids, top, m


def _stack(rows):
    ids, top, m = zip(*rows)
    return torch.stack(ids), torch.stack(top), torch.tensor(m)


def exact(case, seed):
    kind = case["kind"]
    if kind == "partition":
        w, begin = _window(case, seed)
        w = _host(w)
        if case["hist"]:
            w = w[(begin + np.arange(case["W"])) % w.size]
        t = {"table": np.frombuffer(_table(w, case["K"], case["init"]).tobytes(), np.uint8).copy()}
        if case["hist"]:
            t["hist"] = np.bincount(w, minlength=MAX_LEN + 1).astype(np.int32)
        return t
    if kind in ("step", "parts"):
        length, arrival, now, theta, window = _pool(case, seed)
        t = _table(_host(window), case["K"])
        q = _queues(length, t)
        phi = [_phi(length, arrival, now, t, q, th, _cost(case)) for th in theta] if kind == "parts" else None
        rows = phi if phi is not None else (_phi(length, arrival, now, t, q, th, _cost(case)) for th in theta)
        ids, top, m = _stack([_top(p, case["B"]) for p in rows])
        out = {"ids": ids, "top": top, "n_sel": m}
        if phi is not None:
            out["qid"] = torch.where(length > 0, q, torch.full_like(q, -1))
            out["score"] = torch.stack(phi)
        return out
    if kind == "tactical":
        length, arrival, now, theta, window = _pool(case, seed)
        t = _table(_host(window), case["K"])
        k = int(t["head"][0])
        q = _queues(length, t)
        order = torch.sort(arrival, stable=True).indices  # arrival, equal arrivals by id
        by_q = order[torch.sort(q[order], stable=True).indices]
        cnt = torch.bincount(q, minlength=k)
        first = torch.cumsum(cnt, 0) - cnt
        head_id = by_q[first.clamp(max=case["n"] - 1)]
        phi = _phi(length[head_id], arrival[head_id], now, t, torch.arange(k, device="cuda"), theta[0], _cost(case))
        phi = torch.where(cnt > 0, phi, torch.full_like(phi, math.nan))
        h = _host(torch.nan_to_num(phi, nan=-math.inf))
        prim = int(np.argmax(h))
        near = sorted([x for x in (prim - 1, prim + 1) if 0 <= x < k and int(cnt[x]) > 0], key=lambda x: (-h[x], x))
        ids = torch.cat([by_q[int(first[x]):int(first[x]) + int(cnt[x])] for x in [prim] + near])[:case["B"]]
        full = torch.full((case["B"],), -1, dtype=torch.int64, device="cuda")
        full[:ids.numel()] = ids
        return {"ids": full, "n_sel": torch.tensor([ids.numel()]), "q_prim": torch.tensor([prim]), "head_score": phi,
                "removed": torch.zeros(k, dtype=torch.int64), "table": None, "empty": None}
    if kind == "stream":
        if case["bubbles"]:
            return None
        L0, A0, dl, da = _stream_inputs(case, seed, STREAM_BATCHES)
        t = _table(_host(L0[-case["window"]:]), case["K"])
        ln, ar = L0.clone(), A0.clone()
        ln[:case["per"]], ar[:case["per"]] = dl[0], da[0]
        theta = torch.from_numpy(W.THETA_MID.copy()).cuda()
        phi = _phi(ln, ar, float(da[0, -1]), t, _queues(ln, t), theta, W.DEFAULT_COST)
        ids, top, m = _stack([_top(phi, case["B"])])
        return {"ids": ids, "top": top, "n_sel": m, "ring_len": None, "ring_arrival": ar.double(), "log": None}
    L0, A0, dl, da = _stream_inputs(case, seed, TRIAL_BATCHES)
    t = _table(_host(L0[-min(65536, case["n"]):]), case["K"])
    theta = _proposals(_gen(seed + 1), case["pools"])
    ln, ar = L0.clone(), A0.clone()
    ln[:case["per"]], ar[:case["per"]] = dl[0], da[0]
    now = float(da[0, -1])
    q = _queues(ln, t)
    rows = [_top(_phi(ln, ar, now, t, q, th, W.DEFAULT_COST), case["B"]) for th in theta]
    ids, top, m = _stack(rows)
    stats = torch.zeros((case["pools"], 8), dtype=torch.float64, device="cuda")
    for p, (i, _, k) in enumerate(rows):
        i = i[:k]
        wait = torch.clamp(now - ar[i].double(), min=0.0)
        stats[p] = torch.stack([torch.tensor(float(k), dtype=torch.float64, device="cuda"), ln[i].double().sum(),
                                wait.sum(), wait.square().sum(), wait.max(), *torch.zeros(2, device="cuda").double(),
                                torch.tensor(1.0, dtype=torch.float64, device="cuda")])
    return {"ids": ids, "top": top, "n_sel": m, "stats": stats, "queue_admits": None, "len": None,
            "arrival": ar.double().expand(case["pools"], -1)}
