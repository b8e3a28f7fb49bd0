"""The sparse clear by tensors: lists around the 256 indices that a workgroup takes at a time and the 1024 of a chunk, more
pairs than the density let expect (a workgroup then strides), counts beyond the region, tensors without a pair, and numbers of
tensors and payloads on both sides of the line to the launch that numbers the pairs.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 255, 256, 257, 1023, 1024, 1025, 4097]


def clear(sizes, lengths, workers, density, over=0, seed=0):
    """`lengths(tensor, worker)` pairs each; `over`: what the counts claim beyond the region."""
    import torch
    rng = np.random.default_rng([seed, workers, len(sizes)])
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    most = [max(max(lengths(j, w) for w in range(workers)), 1) for j in range(len(sizes))]
    layout = np.concatenate([[0], np.cumsum(most)]).tolist()
    dgc = B.Dgc(B.make_config(density=density, num_workers=workers), offsets)
    dgc.set_layout(layout)
    start = rng.standard_normal(n).astype(np.float32)
    expect, idx_list, count_list = start.copy(), [], []
    for w in range(workers):
        idx = np.full(layout[-1], n, np.int32)       # behind the pairs: no element of the set
        counts = np.zeros(len(sizes), np.int32)
        for j, size in enumerate(sizes):
            m = lengths(j, w)
            e = offsets[j] + np.sort(rng.choice(size, m, replace=False))
            idx[layout[j]:layout[j] + m] = e
            expect[e] = 0.0
            counts[j] = m + (over if m == most[j] else 0)
        idx_list.append(torch.from_numpy(idx).cuda())
        count_list.append(torch.from_numpy(counts).cuda())
    dense = torch.from_numpy(start).cuda()
    dgc.dgc_dense_clear_regions(dense, idx_list, count_list)
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.close()


@pytest.mark.parametrize("workers", [1, 5, 64])
@pytest.mark.parametrize("density", [0.001, 0.2])
def test_lists_of_every_length(workers, density):
    clear([5000, 4097, 4500, 6000, 4097], lambda j, w: LENGTHS[(j + 2 * w) % len(LENGTHS)], workers, density, over=3)


@pytest.mark.parametrize("tensors,workers", [(8192, 2), (16384, 1), (16385, 1), (5462, 3)])
def test_both_sides_of_the_line(tensors, workers):
    clear([3] * tensors, lambda j, w: (j + w) % 4, workers, 0.004)


@pytest.mark.parametrize("long", [4000, 70000])
def test_one_long_tensor_among_many_short(long):
    """Eight workgroups, then one, for each of 1001 tensors: the long one takes several chunks, or too many."""
    clear([4] * 1000 + [200000], lambda j, w: long if j == 1000 else (j + w) % 3, 2, 0.25)
