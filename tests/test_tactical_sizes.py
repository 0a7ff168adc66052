"""The sizes of Algorithm 1's sample, which the kernels index without a bound:
every sample has a place and every place lies in the buffers, for pool sizes
at the edges where more chunks are left out."""
import os

import pytest

import plan_util
from paper_2601_21758_amd.build import LIB_STAMPS

pytestmark = pytest.mark.skipif(not os.path.exists(LIB_STAMPS), reason="instrumented library not built")

CHUNK = 256
EDGES = sorted({c + d for k in range(0, 8) for c in (65536 << k, (65536 << k) + (1 << k)) for d in (-1, 0, 1)})


@pytest.mark.parametrize("chunks", [1, 2, 3, 100, 4096, *EDGES])
@pytest.mark.parametrize("B", [1, 100, 443])
def test_sample_fits(chunks, B):
    for n in (chunks * CHUNK - CHUNK + 1, chunks * CHUNK):
        if n > 2**31 - 1:
            continue
        s = plan_util.tactical(n, B)
        sampled = (chunks + (1 << s["lg_step"]) - 1) >> s["lg_step"]
        assert s["samples"] == 2 * sampled
        assert s["samples"] <= s["places"] <= s["room"], (n, s)
