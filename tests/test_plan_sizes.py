"""The selection plans that the host chooses: what the kernels assume of them,
and the rules that keep the merge away from the pool."""
import os

import pytest

import plan_util
from paper_2601_21758_amd import _lib as L
from paper_2601_21758_amd.build import LIB_STAMPS

pytestmark = pytest.mark.skipif(not os.path.exists(LIB_STAMPS), reason="instrumented library not built")

WAVES, REGION = 16, 64


@pytest.mark.parametrize("n,B", [(9000, 2048), (16384, 4096), (20000, 4096), (40000, 2048), (65536, 64), (9000, 4096),
                                 (1 << 22, 4096)])
@pytest.mark.parametrize("op", [L.OP_SELECT, L.OP_STEP])
def test_regions_are_filled_where_the_admissions_need_them(op, n, B):
    p = plan_util.plan(op, n, 1, B)
    share = B / (p["G"] * WAVES)
    need = share + 2 * share ** 0.5
    if share > REGION:
        assert p["fit"] < REGION  # no list holds it
    else:
        assert p["fit"] >= min(need, REGION - 1)


@pytest.mark.parametrize("n,rows,B", [(20000, 100, 4096), (9000, 256, 2048), (32768, 64, 4096), (65536, 256, 4096),
                                      (100003, 64, 4096), (65536, 64, 64), (1 << 20, 4, 1024), (1 << 20, 4, 2048),
                                      (262144, 16, 512), (1000003, 4, 256), (65536, 64, 512)])
def test_rows_keep_room_for_the_admissions(n, rows, B):
    """Several rows take larger shares per workgroup, but the slots and the waves' regions hold the B where one chunk
    per wave would hold them, and short lists stay short."""
    p = plan_util.plan(L.OP_SELECT, n, rows, B)
    G1 = min(256, -(-n // 4096))  # one chunk per wave
    slots1 = G1 * min(1024, 9088 // G1)
    if slots1 >= B:
        assert p["G"] * p["M"] >= B
    assert B / (p["G"] * WAVES) <= max(40, B / (G1 * WAVES))
    if -(-B // G1) <= 12:
        assert p["lg"] <= 3 and B <= 12 * p["G"]


@pytest.mark.parametrize("cap", [4, 16384, 65536, 262144, 1 << 20, 1 << 23])
@pytest.mark.parametrize("B", [1, 32, 512, 2048, 4096])
def test_trials_run_in_whole_rounds(cap, B):
    """One pass per workgroup, or rounds of the chip that are at least three quarters full, with a region's room for
    every wave's share of the B."""
    full = min(256, -(-cap // 16384))
    for pools in (1, 2, 15, 16, 17, 33, 64, 65, 100, 129, 160, 200, 255, 256, 257, 300, 511, 513, 1000, 1024):
        G = plan_util.plan(L.OP_TRIAL, cap, pools, B)["G"]
        assert 1 <= G <= full
        if G < full:
            rounds = -(-G * pools // 256)
            assert G * pools >= 0.75 * 256 * rounds, (pools, G)
            assert B <= 64 * G


@pytest.mark.parametrize("n,nt,B,filtered", [(262144, 2, 64, False), (262144, 3, 64, False), (262144, 4, 64, True),
                                             (262144, 2, 65, True), (24000, 2, 8, False), (24000, 2, 9, True),
                                             (131072, 2, 128, True), (524288, 2, 128, False), (1 << 20, 6, 128, True)])
def test_few_vectors_are_filtered_where_lists_are_long(n, nt, B, filtered):
    assert (plan_util.plan(L.OP_STEP, n, nt, B)["filter"] > 0) == filtered
