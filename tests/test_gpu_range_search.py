"""The searches of the range kernel (densities up to 0.5 %) in lists around the lengths at which their first round
changes shape, with pairs on both sides of the ranges' bounds, fresh and previous lists of different lengths, no previous
ones at all, and empty ones: the worker-ordered sum bit for bit.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B

pytestmark = pytest.mark.gpu

RANGE = 131072
SIZES = [900, 8 * RANGE + 777, 5]
LENGTHS = [0, 1, 31, 33, 63, 64, 65, 127, 129, 2111, 2112, 2113, 4223, 4224, 4225, 4300]


def payload(m, rng, crowded, layout, offsets):
    import torch
    lo, hi = int(offsets[1]), int(offsets[2])
    if crowded:                                     # around the bounds of the ranges, which start at the tensor's tile
        start = lo // 1024 * 1024
        bounds = np.arange(start + RANGE, hi, RANGE)
        near = np.unique(np.concatenate([b + np.arange(-400, 400) for b in bounds]))
        pos = np.sort(rng.choice(near[(near >= lo) & (near < hi)], m, replace=False))
    else:
        pos = np.sort(rng.choice(hi - lo, m, replace=False)) + lo
    val = rng.standard_normal(m).astype(np.float32)
    idx_all, val_all = np.zeros(layout[-1], np.int32), np.zeros(layout[-1], np.float32)
    counts = np.array([1 if m else 0, m, 0], np.int32)
    at = layout[1]
    idx_all[at:at + m], val_all[at:at + m] = pos, val
    if m:
        idx_all[0], val_all[0] = 7, 0.5
        pos, val = np.concatenate([[7], pos]), np.concatenate([np.float32([0.5]), val])
    return (pos, val), tuple(torch.from_numpy(t).cuda() for t in (idx_all, val_all, counts))


@pytest.mark.parametrize("crowded", [False, True])
@pytest.mark.parametrize("workers,previous", [(1, 0), (3, 5), (8, 8), (12, 9)])
def test_lists_of_every_shape(workers, previous, crowded):
    import torch
    rng = np.random.default_rng([workers, previous, crowded])
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    n = int(offsets[-1])
    layout = [0, 900, 900 + 4400, 900 + 4400 + 5]
    for turn in range(len(LENGTHS)):
        dgc = B.Dgc(B.make_config(density=0.003, num_workers=workers), offsets)
        dgc.set_layout(layout)
        new = [payload(LENGTHS[(turn + 5 * w) % len(LENGTHS)], rng, crowded, layout, offsets) for w in range(workers)]
        old = [payload(LENGTHS[(turn + 3 + 7 * w) % len(LENGTHS)], rng, crowded, layout, offsets) for w in range(previous)]
        lists = tuple([d[i] for _, d in new] for i in range(3))
        was = np.zeros(n, np.float32)
        for (pos, val), _ in old:
            was[pos] += val
        expect = np.zeros(n, np.float32)
        for (pos, val), _ in new:
            expect[pos] = (expect[pos] + val).astype(np.float32)
        dense = torch.from_numpy(was).cuda()
        dgc.dgc_decompress_replace_regions(dense, *lists, [d[0] for _, d in old], [d[2] for _, d in old])
        assert np.array_equal(dense.cpu().numpy(), expect), turn
        dgc.dgc_decompress_accumulate_regions(dense, *lists)
        for (pos, val), _ in new:
            expect[pos] = (expect[pos] + val).astype(np.float32)
        assert np.array_equal(dense.cpu().numpy(), expect), turn
        dgc.close()


@pytest.mark.parametrize("new,old", [(2113, 8600), (4224, 17000), (3000, 20000), (900, 9000), (8600, 2500), (20000, 4224), (2112, 4225), (40, 3000)])
def test_new_and_previous_lists_of_very_different_lengths(new, old):
    """As after a change of density: the two are searched together, each with its own number of probes."""
    import torch
    rng = np.random.default_rng([new, old])
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    n = int(offsets[-1])
    layout = [0, 900, 900 + 20500, 900 + 20500 + 5]
    dgc = B.Dgc(B.make_config(density=0.003, num_workers=3), offsets)
    dgc.set_layout(layout)
    fresh = [payload(m, rng, False, layout, offsets) for m in (new, new, 0)]
    last = [payload(m, rng, False, layout, offsets) for m in (old, 7, old)]
    was, expect = np.zeros(n, np.float32), np.zeros(n, np.float32)
    for (pos, val), _ in last:
        was[pos] += val
    for (pos, val), _ in fresh:
        expect[pos] = (expect[pos] + val).astype(np.float32)
    dense = torch.from_numpy(was).cuda()
    lists = tuple([d[i] for _, d in fresh] for i in range(3))
    dgc.dgc_decompress_replace_regions(dense, *lists, [d[0] for _, d in last], [d[2] for _, d in last])
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.close()
