"""The receive side of sets of few parts, a word of LDS per element: parts that are whole tensors and parts of long ones,
numbers of pairs on both sides of what a workgroup takes into registers, numbers of payloads on both sides of the change
of its width, fresh and previous payloads that share indices, and the same payloads in sets with so many more tensors
that the range and the part kernels take them.  The worker-ordered sum bit for bit.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B

pytestmark = pytest.mark.gpu

PART = 32768
SIZES = [700, 3 * PART + 513, PART, 1, PART + 1023]
TILE = 1024


def payload(share, rng, offsets, layout, crowd):
    """A share of every tensor's elements (of the second tensor's `crowd` elements around a part's bound as well)."""
    import torch
    idx, val = np.zeros(layout[-1], np.int32), np.zeros(layout[-1], np.float32)
    counts = np.zeros(len(offsets) - 1, np.int32)
    pairs = []
    for j in range(len(offsets) - 1):
        lo, hi = int(offsets[j]), int(offsets[j + 1])
        e = lo + rng.choice(hi - lo, int(round(share * (hi - lo))), replace=False)
        if j == 1 and crowd:
            bound = lo // TILE * TILE + PART
            e = np.concatenate([e, bound - crowd // 3 + np.arange(crowd)])
        e = np.unique(e)
        x = rng.standard_normal(e.size).astype(np.float32)
        idx[layout[j]:layout[j] + e.size], val[layout[j]:layout[j] + e.size] = e, x
        counts[j] = e.size
        pairs.append((e, x))
    flat = tuple(np.concatenate(z) for z in zip(*pairs))
    return flat, tuple(torch.from_numpy(t).cuda() for t in (idx, val, counts))


@pytest.mark.parametrize("more", [0, 246, 247])       # tensors of one element: 10 parts, 256, 257
@pytest.mark.parametrize("workers,share,crowd", [(1, 0.02, 0), (1, 0.0, 9000), (8, 0.003, 600), (9, 0.002, 1400),
                                                 (2, 0.04, 2047), (64, 0.0004, 90)])
def test_direct_merge(workers, share, crowd, more):
    import torch
    rng = np.random.default_rng([workers, more, crowd])
    sizes = SIZES + [1] * more
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    layout = np.concatenate([[0], np.cumsum([min(s, 12000) for s in sizes])]).tolist()
    dgc = B.Dgc(B.make_config(density=max(share, 0.0005), num_workers=workers), offsets)
    dgc.set_layout(layout)
    new = [payload(share, rng, offsets, layout, crowd) for _ in range(workers)]
    old = [payload(share, rng, offsets, layout, crowd // 2) for _ in range(max(1, workers - 1))]
    lists = tuple([d[i] for _, d in new] for i in range(3))
    old_lists = [d[0] for _, d in old], [d[2] for _, d in old]

    def ordered(dense, step):
        for (e, x), _ in new:
            dense[e] = (dense[e] + np.float32(step) * x).astype(np.float32)
        return dense

    start = rng.standard_normal(n).astype(np.float32)
    dense = torch.from_numpy(start).cuda()
    dgc.dgc_decompress_accumulate_regions(dense, *lists)
    assert np.array_equal(dense.cpu().numpy(), ordered(start.copy(), 1.0))
    theta = torch.from_numpy(start).cuda()
    dgc.dgc_sparse_sgd_apply_regions(theta, 0.5, *lists)
    assert np.array_equal(theta.cpu().numpy(), ordered(start.copy(), -0.5))
    was = np.zeros(n, np.float32)
    for (e, x), _ in old:
        was[e] += x
    expect = ordered(np.zeros(n, np.float32), 1.0)
    dense = torch.from_numpy(was).cuda()
    dgc.dgc_decompress_replace_regions(dense, *lists, *old_lists)
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.dgc_decompress_replace_regions(dense, *lists, lists[0], lists[2])      # itself again
    assert np.array_equal(dense.cpu().numpy(), expect)
    dense.zero_()
    dgc.dgc_decompress_replace_regions(dense, *lists)                          # nothing before
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.close()


@pytest.mark.parametrize("first,then", [(0.25, 0.001), (0.001, 0.25)])
def test_replacing_across_a_change_of_density(first, then):
    """Long previous lists, and long new ones, on the way from a warm-up density to the lowest and back."""
    import torch
    rng = np.random.default_rng(5)
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    layout = offsets.tolist()
    dgc = B.Dgc(B.make_config(density=first, num_workers=3), offsets)
    dgc.set_layout(layout)
    dense = torch.zeros(int(offsets[-1]), device="cuda")
    previous = ()
    for density in (first, then, then, first):
        dgc.dgc_set_density(density)
        new = [payload(density, rng, offsets, layout, 0) for _ in range(3)]
        lists = tuple([d[i] for _, d in new] for i in range(3))
        dgc.dgc_decompress_replace_regions(dense, *lists, *previous)
        expect = np.zeros(dense.numel(), np.float32)
        for (e, x), _ in new:
            expect[e] = (expect[e] + x).astype(np.float32)
        assert np.array_equal(dense.cpu().numpy(), expect)
        previous = (lists[0], lists[2])
    dgc.close()


@pytest.mark.parametrize("share,workers,then", [(0.01, 2, 0.01), (0.02, 1, 0.02), (0.01, 2, 0.001), (0.02, 1, 0.004)])
def test_replacing_above_half_a_percent_reads_nothing(share, workers, then):
    """The whole of `dense` is written whatever it holds and whatever the previous payloads name, and so it is in the call
    behind such a one."""
    import torch
    rng = np.random.default_rng([workers, int(1000 * then)])
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    layout = offsets.tolist()
    dgc = B.Dgc(B.make_config(density=share, num_workers=workers), offsets)
    dgc.set_layout(layout)
    dense = torch.empty(int(offsets[-1]), device="cuda")
    stale = [torch.zeros(layout[-1], dtype=torch.int32, device="cuda")], [torch.zeros(len(SIZES), dtype=torch.int32, device="cuda")]
    for density in (share, then):
        dgc.dgc_set_density(density)
        new = [payload(density, rng, offsets, layout, 0) for _ in range(workers)]
        expect = np.zeros(dense.numel(), np.float32)
        for (e, x), _ in new:
            expect[e] = (expect[e] + x).astype(np.float32)
        dense.fill_(7.0)
        dgc.dgc_decompress_replace_regions(dense, *(tuple([d[i] for _, d in new] for i in range(3))), *stale)
        assert np.array_equal(dense.cpu().numpy(), expect), density
    dgc.close()


@pytest.mark.parametrize("workers,more", [(7, 0), (64, 0), (64, 25)])
def test_part_kernel_that_searches_and_that_looks_up(workers, more):
    """Dense payloads, parts times payloads on both sides of the line between one launch and two."""
    import torch
    rng = np.random.default_rng([workers, more])
    sizes = SIZES + [3] * more                       # 10 parts, 35
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    dgc = B.Dgc(B.make_config(density=0.25, num_workers=workers), offsets)
    layout = offsets.tolist()
    dgc.set_layout(layout)
    new = [payload(0.25 if w % 3 else 0.01, rng, offsets, layout, 0) for w in range(workers)]
    lists = tuple([d[i] for _, d in new] for i in range(3))
    start = rng.standard_normal(int(offsets[-1])).astype(np.float32)
    expect, fresh = start.copy(), np.zeros_like(start)
    for (e, x), _ in new:
        expect[e] = (expect[e] + x).astype(np.float32)
        fresh[e] = (fresh[e] + x).astype(np.float32)
    dense = torch.from_numpy(start).cuda()
    dgc.dgc_decompress_accumulate_regions(dense, *lists)
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.dgc_decompress_replace_regions(dense, *lists)
    assert np.array_equal(dense.cpu().numpy(), fresh)
    dgc.close()
