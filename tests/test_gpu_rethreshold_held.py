"""The re-threshold and the settling of exact thresholds with the records' keys in registers: tensors of as many tiles as two
threads to a tile hold, and one more, tensors that share their first and last tiles with neighbours, tiles with more
elements than a record holds (few, and so many that they are listed), and ties at the threshold.  As the oracle's.  Run
with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu

TILE = 1024
MOST = 4096 * TILE


@pytest.mark.parametrize("lead", [0, 300])                      # the large tensor shares its first and last tiles, or not
@pytest.mark.parametrize("n", [TILE * 511, TILE * 512, TILE * 513, TILE * 1536 + 77])
@pytest.mark.parametrize("crowd", [0, 40, 700])                 # tiles with dozens of large values each
def test_rethreshold(n, lead, crowd):
    """One value in a thousand is wanted, and the sample misses most of the large ones, which so pass."""
    p = Pair(np.concatenate([[0], np.cumsum(([lead] if lead else []) + [n, 500])]), momentum=0.5, density=0.001, seed=4,
             refine_alpha=1.0, sample_min=4096, sample_max=4096)
    rng = np.random.default_rng([n, lead, crowd])
    for it in range(2):
        g = rng.standard_t(3, p.n).astype(np.float32)
        for t in rng.choice(n // TILE, min(crowd, n // TILE), replace=False):
            at = lead + t * TILE + rng.choice(TILE, 6 if crowd > 100 else 30, replace=False)
            g[at] = rng.choice(np.float32([20.0, 30.0, -30.0, 44.5]), at.size)
        p.step(g, it, label=f"re-threshold n={n} lead={lead} crowd={crowd}")
    p.close()


@pytest.mark.parametrize("n", [MOST - 1, MOST, MOST + TILE])
def test_tensors_around_the_limit(n):
    p = Pair(np.array([0, n, n + 90]), momentum=0.5, density=0.001, seed=4, refine_alpha=1.0, sample_min=4096, sample_max=4096)
    g = np.random.default_rng(n).standard_t(3, p.n).astype(np.float32)
    g[5 * TILE:5 * TILE + 3000] *= 40.0
    p.step(g, 0, label=f"re-threshold n={n}")
    p.close()


@pytest.mark.parametrize("sizes", [[70000] * 3, [2500000] * 4 + [200], [4300000, 4500000, 777]])
@pytest.mark.parametrize("ties", [False, True])
def test_exact_floor(sizes, ties):
    p = Pair(np.concatenate([[0], np.cumsum(sizes)]), momentum=0.5, density=0.001, seed=4, flags=B.DGC_FLAG_EXACT_SELECT)
    g = np.random.default_rng(len(sizes)).standard_t(3, p.n).astype(np.float32)
    if ties:
        g = (np.round(4 * g) / 4).astype(np.float32)
    g[11] = np.nan
    p.step(g, 0, label=f"exact {sizes[0]} ties={ties}")
    p.close()
