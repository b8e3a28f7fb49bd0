"""The extracting pass from mask words with as many selected elements in a part as its lists in LDS hold, one more
and one less, with regions that end inside a list, and with the elements crowded into one end of the part: bit for bit
what the oracle computes, ascending, the lowest indices where a region is full.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu

PART = 32768
EXACT = B.DGC_FLAG_EXACT_SELECT | B.DGC_FLAG_SORTED_OUTPUT


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("crowded", [False, True])
@pytest.mark.parametrize("k", [165, 2048, 2049, 4095, 4096, 4097, 8191, 8193, 9215, 9216, 9217, 18432, 18433, 32767])
def test_windows_of_a_part(staged, crowded, k):
    rng = np.random.default_rng([k, crowded])
    g = rng.standard_normal(PART + 5).astype(np.float32)
    if crowded:
        g[:PART] = np.sort(np.abs(g[:PART])) * np.where(rng.random(PART) < 0.5, -1, 1)
    for cap in (PART, k, k - 1, max(1, k // 2)):
        # the second tensor shares the first one's last tile, or starts a ragged one of its own
        for first in (PART, PART - 700):
            p = Pair([0, first, PART + 5], warmup_workspace=staged, capacities=[min(cap, first), PART + 5 - first],
                     momentum=0.9, density=min(1.0, (min(k, first - 1) - 0.5) / first), flags=EXACT, seed=3)
            res = p.step(g, 0, label=f"windows k={k} staged={staged} crowded={crowded} cap={cap} first={first}")
            assert res.counts[0] == min(k, first - 1)
            p.close()
