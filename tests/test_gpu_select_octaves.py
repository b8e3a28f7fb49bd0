"""Threshold selection at ranks that are not ranked from a short list: values spread over as many octaves as the first
histogram covers, and over more, a key below what was guessed, in the bin that takes everything above, in a crowd of nearly
equal values and of equal ones, and a handful of values beyond all others.  Thresholds and index sets as the oracle's.
Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu


def values(kind, n, rng):
    x = rng.standard_normal(n)
    if kind == "octaves":                     # evenly over forty octaves
        x = np.exp2(rng.uniform(-20, 20, n)) * np.sign(x)
    elif kind == "two heights":               # nine in ten far below the largest
        x = np.where(rng.random(n) < 0.9, 1e-6 * x, 1e3 * x)
    elif kind == "outliers":
        x[rng.choice(n, 20, replace=False)] *= 1e20
    elif kind == "nearly equal":
        x = 1.0 + 1e-6 * x
    elif kind == "equal":
        x = np.sign(x) * rng.choice([0.5, 1.0, 2.0], n)
    elif kind == "mostly zero":
        x = np.where(rng.random(n) < 0.8, 0.0, x)
    elif kind == "denormal":
        x = 1e-42 * x
    elif kind == "not numbers":
        x[rng.choice(n, n // 50, replace=False)] = np.nan
        x[rng.choice(n, n // 50, replace=False)] = np.inf
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["normal", "octaves", "two heights", "outliers", "nearly equal", "equal", "mostly zero",
                                  "denormal", "not numbers"])
@pytest.mark.parametrize("n,sample", [(500000, 32768), (90000, 8192), (20000, 20000), (1500, 4096)])
@pytest.mark.parametrize("density", [0.006, 0.25, 0.97])
def test_ranks(kind, n, sample, density):
    rng = np.random.default_rng([n, int(density * 1000)])
    p = Pair(np.array([0, 9, 9 + n]), momentum=0.0, density=density, seed=6, sample_min=sample, sample_max=max(sample, 32),
             flags=B.DGC_FLAG_SORTED_OUTPUT)
    p.step(values(kind, p.n, rng), 0, label=f"{kind} n={n} d={density}")
    p.close()
