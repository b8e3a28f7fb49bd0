"""The re-threshold where its ranking takes another way: more elements than a workgroup lists, bins that
hold hundreds of equal keys, magnitudes beyond the histogram's last bin, regions too small for the list.
Bit for bit against the oracle.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from oracle import dgc_oracle as O
from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu


def values(kind, rng, n, density):
    """More large elements than are wanted, so that a threshold below them lets too many pass."""
    if kind == "tail":
        return rng.standard_t(3, n)
    share = rng.random(n)
    small = 0.1 * rng.random(n)
    if kind == "levels":                                   # a few magnitudes: thousands of equal keys
        return np.where(share < 1.1 * density, -8.0, np.where(share < 8 * density, 2.0, small))
    if kind == "close":                                    # one bin of the histogram holds them all
        return np.where(share < 2 * density, 1.0 + 1e-6 * rng.integers(0, 1000, n), small)
    return np.where(share < 2 * density, np.exp(rng.uniform(0.0, 60.0, n)), small)    # "wide": far beyond four octaves


@pytest.mark.parametrize("density,tight", [(0.001, False), (0.004, False), (0.004, True), (0.03, False), (0.03, True)])
@pytest.mark.parametrize("kind", ["tail", "levels", "close", "wide"])
def test_rethreshold_forms(kind, density, tight):
    sizes = [700, 650001, 3, 40000]                        # 650001: at 3 % more pass than a workgroup lists
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    caps = [O.topk_count(density, s) for s in sizes] if tight else None
    kw = dict(momentum=0.0, density=density, seed=8, sample_min=512, sample_max=512, refine_alpha=1.0,
              flags=B.DGC_FLAG_SORTED_OUTPUT)
    p = Pair(offsets, **({"capacities": caps} if tight else {"layout_density": 0.25}), **kw)
    rng = np.random.default_rng([len(kind), int(density * 1e6)])
    refined = 0
    for it in range(6):
        g = values(kind, rng, p.n, density).astype(np.float32)
        p.set_state(np.zeros(p.n, np.float32), np.zeros(p.n, np.float32))
        res = p.step(g, it, label=f"rethreshold {kind} d={density} tight={tight} it{it}")
        refined += sum(res.refined)
    assert refined > 0
    p.close()
