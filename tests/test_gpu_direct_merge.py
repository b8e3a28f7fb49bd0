"""The receive side of sets of few parts, a word of LDS per element: parts that are whole tensors and parts of long ones,
numbers of pairs on both sides of what a workgroup takes into registers, numbers of payloads on both sides of the change
of its width, fresh and previous payloads that share indices, and the same payloads in sets with so many more tensors
that the range and the part kernels take them.  The worker-ordered sum bit for bit.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B
from tests.parity import capture

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


@pytest.mark.parametrize("workers", [1, 3, 8, 9, 64])       # at density 0.001: 64 of them 0.064 pairs per element
@pytest.mark.parametrize("taken", [2048, 2049, 4096, 4097, 8193, 16385, 31001])
def test_parts_that_pairs_crowd(workers, taken):
    """Parts that start anywhere and end behind any quad, in one of which the payloads together have `taken` pairs and in
    another each of them has as many: on both sides of what a workgroup takes into registers, and of the rounds of chunks."""
    import torch
    rng = np.random.default_rng([workers, taken])
    sizes = [703, 31001, 2 * PART, 31002, 513, 1]              # (one part each, but for the third)
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    layout = offsets.tolist()
    dgc = B.Dgc(B.make_config(density=0.001, num_workers=workers), offsets)
    dgc.set_layout(layout)

    def lists_of(number):
        pairs, out = [], ([], [], [])
        shares = np.diff(np.linspace(0, taken, number + 1).astype(int))
        for w in range(number):
            idx, val, counts = np.zeros(layout[-1], np.int32), np.zeros(layout[-1], np.float32), np.zeros(len(sizes), np.int32)
            for j, crowd in ((0, 9), (1, shares[w]), (3, min(taken, sizes[3])), (4, sizes[4] if w == number - 1 else 0)):
                e = layout[j] + np.sort(rng.choice(sizes[j], crowd, replace=False))
                idx[layout[j]:layout[j] + crowd], val[layout[j]:layout[j] + crowd] = e, rng.standard_normal(crowd)
                counts[j] = crowd
                pairs.append((e, val[layout[j]:layout[j] + crowd]))
            for to, x in zip(out, (idx, val, counts)):
                to.append(torch.from_numpy(x).cuda())
        return pairs, out

    def ordered(dense, pairs, step):
        for e, x in pairs:
            dense[e] = (dense[e] + np.float32(step) * x).astype(np.float32)
        return dense

    pairs, lists = lists_of(workers)
    old_pairs, old = lists_of(max(1, workers // 2))
    start = rng.standard_normal(layout[-1]).astype(np.float32)
    dense = torch.from_numpy(start).cuda()
    dgc.dgc_decompress_accumulate_regions(dense, *lists)
    assert np.array_equal(dense.cpu().numpy(), ordered(start.copy(), pairs, 1.0))
    theta = torch.from_numpy(start).cuda()
    dgc.dgc_sparse_sgd_apply_regions(theta, 0.5, *lists)
    assert np.array_equal(theta.cpu().numpy(), ordered(start.copy(), pairs, -0.5))
    dense = torch.from_numpy(ordered(np.zeros_like(start), old_pairs, 1.0)).cuda()
    dgc.dgc_decompress_replace_regions(dense, *lists, old[0], old[2])
    assert np.array_equal(dense.cpu().numpy(), ordered(np.zeros_like(start), pairs, 1.0))
    few_pairs, few = lists_of(1)
    few[2][0].zero_()                                            # long previous lists, and nothing new
    dgc.dgc_decompress_replace_regions(dense, *few, lists[0], lists[2])
    assert not dense.any()
    dgc.close()


@pytest.mark.parametrize("workers", [2, 9])                   # 512 threads, 1024
@pytest.mark.parametrize("scale", [None, 0.5])
def test_elements_that_no_pair_names_are_another_streams(workers, scale):
    """Two streams add to one vector, one to elements of even and one to elements of odd numbers of parts that pairs crowd."""
    import torch
    rng = np.random.default_rng(workers)
    n, taken, calls = 3 * PART + 513, 9001, 40
    expect = rng.standard_normal(n).astype(np.float32)
    dense = torch.from_numpy(expect).cuda()
    sides = []
    for odd in (0, 1):
        dgc = B.Dgc(B.make_config(density=0.001, num_workers=workers), [0, n])
        dgc.set_layout([0, taken])
        lists = [[], [], []]
        pairs = []
        for _ in range(workers):
            e = 2 * np.sort(rng.choice(3 * PART // 4, taken, replace=False)).astype(np.int32) + odd
            x = rng.standard_normal(taken).astype(np.float32)
            pairs.append((e, x if scale is None else np.float32(-scale) * x))
            for to, t in zip(lists, (e, x, np.array([taken], np.int32))):
                to.append(torch.from_numpy(t).cuda())
        for _ in range(calls):
            for e, x in pairs:
                expect[e] = (expect[e] + x).astype(np.float32)
        sides.append((dgc, lists, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(calls):
        for dgc, lists, stream in sides:
            with torch.cuda.stream(stream):
                if scale is None:
                    dgc.dgc_decompress_accumulate_regions(dense, *lists)
                else:
                    dgc.dgc_sparse_sgd_apply_regions(dense, scale, *lists)
    torch.cuda.synchronize()
    assert np.array_equal(dense.cpu().numpy(), expect)
    for dgc, _, _ in sides:
        dgc.close()


def best_of(call, turns=8, calls=20):
    """Time of a call in us, of the fastest of several rows of them in a captured graph."""
    import time

    import torch
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with capture(graph):
        for _ in range(calls):
            call()
    best = float("inf")
    for _ in range(turns):
        torch.cuda.synchronize()
        start = time.perf_counter()
        graph.replay()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - start)
    return best / calls * 1e6


@pytest.mark.parametrize("n,density,workers,crowded", [(1 << 20, 0.008, 4, 8), (7000001, 0.01, 8, 50)])
def test_crowded_parts_are_no_slower_than_in_the_part_kernel(n, density, workers, crowded):
    """All pairs in an eighth or a fiftieth of the tensor, against the same in a set with so many more tensors that the part
    kernels take them.  Each pair by itself took 1.4 and 6 times as long as they do, their way through the pairs takes 0.6 and
    0.8: the bound lies where noise does not reach it from either side."""
    import torch
    rng = np.random.default_rng(crowded)
    k = int(density * n)
    chosen = [np.sort(rng.choice(n // crowded, k, replace=False)).astype(np.int32) for _ in range(workers)]
    took = []
    for more in (0, 257):
        offsets = np.concatenate([[0], np.cumsum([n] + [1] * more)])
        dgc = B.Dgc(B.make_config(density=density, num_workers=workers), offsets)
        layout = [0] + [k + i for i in range(more + 1)]
        dgc.set_layout(layout)
        lists = [[], [], []]
        for e in chosen:
            lists[0].append(torch.from_numpy(np.concatenate([e, np.zeros(more, np.int32)])).cuda())
            lists[1].append(torch.ones(k + more, device="cuda"))
            lists[2].append(torch.tensor([k] + [0] * more, dtype=torch.int32, device="cuda"))
        dense = torch.zeros(n + more, device="cuda")
        took.append(best_of(lambda: dgc.dgc_decompress_accumulate_regions(dense, *lists)))
        dgc.close()
    assert took[0] <= 1.1 * took[1], took


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


@pytest.mark.parametrize("sizes,workers", [([PART + 5] * 21 + [77], 24), ([PART + 5] * 22 + [77], 24), ([PART + 5] * 3, 25),
                                           ([PART] * 3 + [77], 25), ([PART] * 3 + [77], 64)])
def test_part_kernel_by_lists_and_payloads(sizes, workers):
    """Lists that are searched, and payloads, on both sides of where a launch of its own finds the pairs; nothing to search."""
    import torch
    rng = np.random.default_rng([len(sizes), workers])
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    layout = offsets.tolist()
    dgc = B.Dgc(B.make_config(density=0.25, num_workers=workers), offsets)
    dgc.set_layout(layout)
    new = [payload(0.02 + 0.01 * (w % 5), rng, offsets, layout, 0) for w in range(workers)]
    lists = tuple([d[i] for _, d in new] for i in range(3))
    start = rng.standard_normal(layout[-1]).astype(np.float32)
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
