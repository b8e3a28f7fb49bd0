"""Decoding short payloads in one launch: numbers of entries around a workgroup's share and around the longest payload that
goes this way, payloads of different lengths beside each other, streams that start anywhere, runs that reach behind the
vector's end or past 2**32.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from tests.test_gpu_wire_forms import run_case

pytestmark = pytest.mark.gpu

GROUP, LONGEST = 4096, 32768


def stream(rng, entries, most):
    runs = rng.integers(0, most + 1, entries).astype(np.uint16)
    vals = rng.standard_normal(entries).astype(np.float32)
    return runs, vals, np.cumsum(runs.astype(np.int64) + 1) - 1


@pytest.mark.parametrize("shift", [0, 1, 5])
@pytest.mark.parametrize("entries", [1, 7, 8, 9, 511, 513, GROUP - 1, GROUP, GROUP + 1, 3 * GROUP + 8, LONGEST - 1, LONGEST,
                                     LONGEST + 1])
def test_entries_around_a_workgroups_share(entries, shift):
    rng = np.random.default_rng([entries, shift])
    streams = [stream(rng, e, 400) for e in (entries, max(1, entries // 3), 0, min(entries, GROUP + 5))]
    n = int(max(s[2][-1] for s in streams if s[2].size)) + 1
    run_case(n, streams, 0, shift=shift)
    run_case(max(1, n - 3), streams, 0, shift=shift)          # the last entries lie behind the end


def test_runs_past_two_to_the_32():
    rng = np.random.default_rng(1)
    runs = np.full(LONGEST, 65535, np.uint16)
    vals = np.ones(LONGEST, np.float32)
    far = (runs, vals, np.cumsum(runs.astype(np.int64) + 1) - 1)
    run_case(5_000_000, [far, stream(rng, 9000, 200), far], 0)
