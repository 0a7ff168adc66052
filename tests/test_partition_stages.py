"""Refine-and-Prune's kernels at the sizes and shapes where their paths change,
bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2601_21758_amd import workloads as W
from parity_util import check_table

torch = pytest.importorskip("torch")


def _window(name):
    rng = np.random.default_rng(sum(map(ord, name)))
    if name == "two_modes":        # one long chain of merges
        return W._lengths(rng, 65536, W.MIX_TWO)
    if name == "three_modes":      # chains on both sides
        return W._lengths(rng, 30000, W.MIX_THREE)
    if name == "scattered":        # isolated pairs all over the axis: no chains
        base = np.arange(1, 900) * 36
        return np.repeat(np.concatenate([base, base + rng.integers(8, 16, base.size)]),
                         rng.integers(1, 50, 2 * base.size)).astype(np.int32)
    if name == "equal_gaps":       # every pair of leaves has the same utility
        return np.repeat(np.arange(1, 1200, dtype=np.int32) * 27, 3)
    if name == "scattered_many":   # no chains, more leaves than LDS holds
        base = np.arange(1, 2400) * 13
        return np.repeat(np.concatenate([base, base + rng.integers(3, 6, base.size)]),
                         rng.integers(1, 50, 2 * base.size)).astype(np.int32)
    if name == "many_leaves":      # chains over more leaves than LDS holds
        return np.sort(rng.choice(np.arange(1, 32769), 9000, replace=False)).astype(np.int32)
    if name == "all_lengths":      # every length once: the largest number of leaves
        return np.arange(1, 32769, dtype=np.int32)
    raise ValueError(name)


# name, init_queues, max_queues, min_width, expected range of Stage-3 leaves
STAGE3 = [
    ("two_modes", 64, 64, 16, (300, 2048)),
    ("two_modes", 64, 1, 16, (300, 2048)),
    ("three_modes", 16, 16, 16, (300, 2048)),
    ("scattered", 32768, 200, 0, (1500, 2048)),
    ("equal_gaps", 32768, 37, 0, (1199, 1199)),
    ("scattered_many", 32768, 256, 0, (2049, 32768)),
    ("many_leaves", 32768, 50, 0, (2049, 32768)),
    ("all_lengths", 32768, 256, 0, (32768, 32768)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,K,mq,mw,leaves", STAGE3)
def test_stage3_merges(name, K, mq, mw, leaves):
    from paper_2601_21758_amd import ewsjf as E
    win = _window(name)
    print(f"stage 3 {name} W={win.size} max_queues={mq}", flush=True)
    ref = oracle.partition(win, init_queues=K, max_queues=mq, min_width=mw)
    assert leaves[0] <= ref.n_leaves <= leaves[1]
    prm = E.params(init_queues=K, max_queues=mq, min_width=mw)
    check_table(E.read_table(E.partition(torch.from_numpy(win).cuda(), prm)), ref)


# Windows for the 3-means splits: one value tile and its edges (63, 64, 65
# distinct values), a few, the most; ties between splits; one far value.
KMEANS3 = {
    "v2": lambda r: np.array([5, 9, 9], np.int32),
    "v3": lambda r: np.array([5, 9, 700], np.int32),
    "v4": lambda r: np.array([1, 2, 3, 4], np.int32),
    "v63": lambda r: r.permutation(np.arange(1, 64, dtype=np.int32)),
    "v64": lambda r: np.repeat(np.arange(100, 164, dtype=np.int32), 2),
    "v65": lambda r: np.arange(1, 66, dtype=np.int32) * 500,
    "v129_symmetric": lambda r: np.concatenate([np.arange(1, 65), [16384], 32768 - np.arange(1, 65)]).astype(np.int32),
    "far_value": lambda r: np.concatenate([r.integers(1, 400, 5000), [32768]]).astype(np.int32),
    "three_modes": lambda r: W._lengths(r, 20000, W.MIX_THREE),
    "uniform": lambda r: r.integers(1, 32769, 60000).astype(np.int32),
    "all_lengths": lambda r: np.arange(1, 32769, dtype=np.int32),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(KMEANS3))
def test_kmeans3_split(name):
    from paper_2601_21758_amd import ewsjf as E
    win = KMEANS3[name](np.random.default_rng(7))
    print(f"3-means {name} W={win.size}", flush=True)
    ref = oracle.partition(win, init_mode=oracle.KMEANS3, max_queues=32)
    prm = E.params(init_mode=1, max_queues=32)
    check_table(E.read_table(E.partition(torch.from_numpy(win).cuda(), prm)), ref)


def _stage2_window(name):
    rng = np.random.default_rng(sum(map(ord, name)))
    if name.startswith("v"):  # that many distinct values, irregular gaps, repeated counts
        n = int(name[1:])
        v = np.sort(rng.choice(np.arange(1, 32769), n, replace=False))
        return np.repeat(v, rng.integers(1, 4, n)).astype(np.int32)
    if name == "clusters":    # gaps inside gaps: several levels of refinement
        v = [a * 8192 + b * 512 + c * 32 + d for a in range(4) for b in (0, 1, 2, 9) for c in (0, 1, 5) for d in (0, 1, 2)]
        return (np.array(v) + 1).astype(np.int32)
    if name == "on_the_line":  # gaps equal to alpha times the mean gap are not cut
        return np.cumsum([1] + [1, 1, 4, 1, 1, 4, 1, 1, 2] * 40).astype(np.int32)
    raise ValueError(name)


STAGE2 = [f"v{n}" for n in (1, 2, 3, 63, 64, 65, 128, 1023, 1025, 4097, 32768)] + ["clusters", "on_the_line"]


@pytest.mark.gpu
@pytest.mark.parametrize("gap_mode", [0, 1])
@pytest.mark.parametrize("name", STAGE2)
def test_stage2_cuts(name, gap_mode):
    """Segment words and their edges, one and several levels, both gap readings, three ratios alpha."""
    from paper_2601_21758_amd import ewsjf as E
    win = _stage2_window(name)
    for alpha, K, mw in ((2.0, 16, 16), (1.01, 1, 0), (3.7, 200, 3)):
        print(f"stage 2 {name} gap_mode={gap_mode} alpha={alpha} K={K}", flush=True)
        ref = oracle.partition(win, init_queues=K, max_queues=256, min_width=mw, alpha=alpha, gap_mode=gap_mode)
        prm = E.params(init_queues=K, max_queues=256, min_width=mw, alpha=alpha, gap_mode=gap_mode)
        check_table(E.read_table(E.partition(torch.from_numpy(win).cuda(), prm)), ref)
