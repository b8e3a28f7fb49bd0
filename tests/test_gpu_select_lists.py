"""Threshold selection at the sizes where its short way changes: candidates that fill one to eight of a thread's
groups of four and leave the last one partly empty, lists around the 256 keys that have four threads each, several
large values in one thread's hands, and ties in the list.  Thresholds and index sets as the oracle's.
Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 1023, 1025, 4096, 4097, 5119, 12289, 20477, 28671, 32767, 32768])
@pytest.mark.parametrize("rank", [0.0005, 0.003, 0.0035])
def test_whole_tensors(n, rank):
    """Candidates are the tensor: a single load each."""
    p = Pair(np.array([0, 40, 40 + n]), momentum=0.5, density=rank, seed=3, sample_min=32768)
    rng = np.random.default_rng(n)
    g = rng.standard_t(3, p.n).astype(np.float32)
    p.step(g, 0, label=f"whole {n}")
    g = np.round(g * 2) / 2                       # many ties
    p.step(g.astype(np.float32), 1, label=f"whole {n}, ties")
    p.close()


@pytest.mark.parametrize("sample", [4096, 4128, 8192, 12320, 20480, 28672, 32768])
@pytest.mark.parametrize("density", [0.001, 0.0035, 0.02])
@pytest.mark.parametrize("clip", [0.0, 0.7])
def test_samples(sample, density, clip):
    """Sampled blocks, four candidates to a load; a row of large neighbours puts several into one thread."""
    p = Pair(np.array([0, 7, 7 + 400000]), momentum=0.5, density=density, seed=9, sample_min=sample, sample_max=sample,
             clip_threshold=clip, num_workers=2)
    rng = np.random.default_rng(sample)
    for it in range(2):
        g = rng.standard_t(3, p.n).astype(np.float32)
        g[1000:1000 + 64 * 900] *= 30.0           # about a seventh of the blocks: clusters
        p.step(g, it, label=f"sample {sample} d={density}")
    p.close()
