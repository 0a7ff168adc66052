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
