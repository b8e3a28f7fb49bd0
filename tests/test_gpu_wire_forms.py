"""The forms of the wire-format kernels at the sizes where they change over: encoder with and without a
scan launch, decoder entry by entry and by range, blocks of 512 entries and more, streams that are not
16-byte aligned, ends of blocks and ranges.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from oracle import dgc_oracle as O
from paper_1712_01887_amd import binding as B
from tests.parity import Pair

pytestmark = pytest.mark.gpu

DET = B.DGC_FLAG_DETERMINISTIC_ACCUMULATE


def random_stream(rng, n, density, trailing=0):
    """Entries of a random sparse vector of n - trailing elements: (runs, vals, positions)."""
    idx = np.flatnonzero(rng.random(n - trailing) < density)
    gap = np.diff(idx, prepend=-1) - 1
    need = 1 + (gap >> 16)
    end = np.cumsum(need)
    runs = np.full(int(end[-1]) if idx.size else 0, 65535, np.int64)
    runs[end - 1] = gap & 65535
    vals = np.zeros(runs.size, np.float32)
    vals[end - 1] = rng.standard_normal(idx.size).astype(np.float32)
    return runs.astype(np.uint16), vals, np.cumsum(runs + 1) - 1


def run_case(n, streams, flags, handle_n=None, shift=0, seed=0):
    """Decodes onto a random vector; compares with the worker-ordered binary32 sum."""
    import torch
    rng = np.random.default_rng(seed)
    dgc = B.Dgc(B.make_config(flags=flags), [0, handle_n or n])
    start = rng.standard_normal(n).astype(np.float32)
    start[:: 7] = -0.0
    dense = torch.from_numpy(start).cuda()
    dev_runs, dev_vals = [], []
    for runs, vals, _ in streams:
        r = torch.zeros(runs.size + 8, dtype=torch.int16, device="cuda")[shift:]
        x = torch.zeros(vals.size + 8, device="cuda")[shift:]
        r[: runs.size] = torch.from_numpy(runs.view(np.int16)).cuda()
        x[: vals.size] = torch.from_numpy(vals).cuda()
        dev_runs.append(r)
        dev_vals.append(x)
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    dgc.dgc_decode_accumulate(dense, dev_runs, dev_vals, [s[0].size for s in streams], bad)
    expect = start.copy()
    exact = start.astype(np.float64)
    mags = np.abs(exact)
    beyond = False
    for runs, vals, pos in streams:
        ok = pos < n
        beyond |= not ok.all()
        expect[pos[ok]] = expect[pos[ok]] + vals[ok]      # positions of one stream are distinct
        exact[pos[ok]] += vals[ok]
        mags[pos[ok]] += np.abs(vals[ok])
    got = dense.cpu().numpy()
    assert bool(bad.item() & B.DGC_DIAG_BAD_INDEX) == beyond
    if flags & DET:
        assert np.array_equal(got.view(np.uint32), expect.view(np.uint32))
    else:
        # a sum of N + 1 binary32 terms in any order: within N * 2**-24 of the exact one, relative to the terms
        assert np.all(np.abs(got - exact) <= len(streams) * 2.0 ** -24 * mags)
    dgc.close()


@pytest.mark.parametrize("flags", [0, DET])
@pytest.mark.parametrize("n,density,workers,shift", [
    (1, 1.0, 1, 0), (7, 1.0, 3, 1), (511, 1.0, 2, 0), (513, 1.0, 2, 3), (8191, 0.5, 5, 0), (8193, 0.5, 5, 0),
    (100001, 0.001, 2, 0), (100001, 0.9, 2, 1), (300000, 0.07, 1, 0), (300000, 0.03, 4, 0), (300000, 0.2, 16, 1),
    (1000003, 0.0001, 3, 0), (1000003, 0.25, 4, 0), (3000001, 0.003, 64, 0),
])
def test_decode_forms(n, density, workers, shift, flags):
    rng = np.random.default_rng([n, workers])
    streams = [random_stream(rng, n, density, trailing=min(n - 1, 40 * (w % 2))) for w in range(workers)]
    if workers > 2:
        streams[1] = streams[1][0][:0], streams[1][1][:0], streams[1][2][:0]    # a worker that sends nothing
    run_case(n, streams, flags, shift=shift)


@pytest.mark.parametrize("flags", [0, DET])
@pytest.mark.parametrize("n", [3000, 4000000])
def test_decode_blocks_of_more_than_512_entries(n, flags):
    """64 payloads with every element sent: the workspace holds one position per 2048 entries; summed into a
    vector of the handle's size (range form) and into a long one (entry by entry, unless in order)."""
    rng = np.random.default_rng(n)
    run_case(n, [random_stream(rng, 3000, 1.0) for _ in range(64)], flags, handle_n=3000)


@pytest.mark.parametrize("flags", [0, DET])
@pytest.mark.parametrize("density", [0.002, 0.4])
def test_decode_skips_and_flags_what_lies_behind_the_end(density, flags):
    rng = np.random.default_rng(3)
    streams = [random_stream(rng, 20000, density), random_stream(rng, 25000, density), random_stream(rng, 20000, density)]
    run_case(20000, streams, flags, handle_n=25000)
    # runs that add up to more than 2**32: nothing wraps round
    runs = np.full(70000, 65535, np.uint16)
    vals = np.ones(70000, np.float32)
    run_case(70000, [(runs, vals, np.cumsum(runs.astype(np.int64) + 1) - 1)], flags)


@pytest.mark.parametrize("sizes,density,layout_density", [
    ([4097, 3, 66000, 8192], 0.5, 1.0),        # a few workgroups: block sums added up without a scan
    ([5, 4600000, 77], 0.02, 1.0),             # some thousand of them, most without a pair
    ([900001, 1], 0.00002, 0.0001),            # gaps of more than 65535 zeros in most rounds
])
def test_encode_forms(sizes, density, layout_density):
    import torch
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    p = Pair(offsets, layout_density=layout_density, momentum=0.0, density=density, seed=6, flags=B.DGC_FLAG_SORTED_OUTPUT)
    g = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    res = p.step(g, 0, label=f"encode {sizes}")
    want_runs, want_vals = O.encode(*O.flatten_payload(res))
    runs = torch.zeros(want_runs.size + 4, dtype=torch.int16, device="cuda")
    vals = torch.zeros(want_runs.size + 4, device="cuda")
    num = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    p.dgc.dgc_encode(p.out_idx, p.out_val, p.out_counts, runs[:-4], vals[:-4], num)
    assert int(num.item()) == want_runs.size
    assert np.array_equal(runs.cpu().numpy()[:-4].view(np.uint16), want_runs) and not runs[-4:].any().item()
    assert np.array_equal(vals.cpu().numpy()[:-4], want_vals) and not vals[-4:].any().item()
    p.close()


def test_encode_with_more_block_sums_than_a_workgroup_adds_up():
    """Regions of 70 M pairs between them, nearly empty: 17090 workgroup slots, so a scan launch."""
    import torch
    sizes = [69000001, 1000003]
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dgc = B.Dgc(B.make_config(), offsets)
    dgc.set_layout(offsets.tolist())
    rng = np.random.default_rng(1)
    per = [np.sort(rng.choice(s, k, replace=False)).astype(np.int64) + o for s, k, o in zip(sizes, (9000, 300), offsets)]
    idx = torch.zeros(int(offsets[-1]), dtype=torch.int32, device="cuda")
    val = torch.zeros(int(offsets[-1]), device="cuda")
    x = [rng.standard_normal(p.size).astype(np.float32) for p in per]
    for o, p, v in zip(offsets, per, x):
        idx[o:o + p.size] = torch.from_numpy(p.astype(np.int32)).cuda()
        val[o:o + p.size] = torch.from_numpy(v).cuda()
    counts = torch.tensor([p.size for p in per], dtype=torch.int32, device="cuda")
    want_runs, want_vals = O.encode(np.concatenate(per).astype(np.int32), np.concatenate(x))
    runs = torch.zeros(want_runs.size, dtype=torch.int16, device="cuda")
    vals = torch.zeros(want_runs.size, device="cuda")
    num = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    dgc.dgc_encode(idx, val, counts, runs, vals, num)
    assert int(num.item()) == want_runs.size
    assert np.array_equal(runs.cpu().numpy().view(np.uint16), want_runs)
    assert np.array_equal(vals.cpu().numpy(), want_vals)
    dgc.close()


@pytest.mark.parametrize("flags", [0, DET])
@pytest.mark.parametrize("n,payloads", [(1 << 21, 6), ((1 << 22) + 77, 3)])   # by range in both orders
def test_decoding_leaves_unnamed_elements_to_others(n, payloads, flags):
    """Entries name elements of every other block of 64 only; those of the blocks between are counted up on
    another stream meanwhile.  All values are small whole numbers: no order of additions changes a sum."""
    import torch
    rng = np.random.default_rng(n)
    mine = (np.arange(n) // 64) % 2 == 0
    dgc = B.Dgc(B.make_config(flags=flags), [0, n])
    runs, vals, counts = [], [], []
    expect = np.zeros(n, np.float32)
    for w in range(payloads):
        idx = np.flatnonzero(mine & (rng.random(n) < 0.3))
        runs.append(torch.from_numpy((np.diff(idx, prepend=-1) - 1).astype(np.int16)).cuda())
        vals.append(torch.full((idx.size,), float(w + 1), device="cuda"))
        counts.append(idx.size)
        expect[idx] += w + 1
    dense = torch.zeros(n, device="cuda")
    others = dense[: n // 128 * 128].view(-1, 2, 64)[:, 1]
    rounds = 60
    dgc.dgc_decode_accumulate(torch.zeros(n, device="cuda"), runs, vals, counts)   # uploads the tables
    torch.cuda.synchronize()
    here, there = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(rounds):
        with torch.cuda.stream(here):
            dgc.dgc_decode_accumulate(dense, runs, vals, counts)
        with torch.cuda.stream(there):
            others.add_(1.0)
    torch.cuda.synchronize()
    expect *= rounds
    expect[: n // 128 * 128].reshape(-1, 2, 64)[:, 1] += rounds
    assert np.array_equal(dense.cpu().numpy(), expect)
    dgc.close()


def expected_entries(idx, val):
    """(runs, vals) of an ascending pair list."""
    gap = np.diff(idx, prepend=-1) - 1
    need = 1 + (gap >> 16)
    end = np.cumsum(need)
    runs = np.full(int(end[-1]) if idx.size else 0, 65535, np.int64)
    vals = np.zeros(runs.size, np.float32)
    runs[end - 1] = gap & 65535
    vals[end - 1] = val
    return runs.astype(np.uint16), vals


@pytest.mark.parametrize("large", [True, False])
@pytest.mark.parametrize("tensors", [1, 2, 63, 64, 65, 128, 129, 4095, 4096, 4097, 20000])
def test_encoding_many_tensors(tensors, large):
    """Regions of no pair, no room, one workgroup and, if a few are large, several: workgroups find their tensor
    by search then (numbers of tensors around the search's steps), and by their own number otherwise."""
    import torch
    rng = np.random.default_rng(tensors)
    sizes = rng.integers(1, 2000, tensors)
    if large:
        sizes[rng.integers(0, tensors, 1 + tensors // 400)] = rng.integers(8000, 40000)
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    dgc = B.Dgc(B.make_config(density=0.01, flags=B.DGC_FLAG_SORTED_OUTPUT), offsets)
    room = np.where(rng.random(tensors) < 0.2, 0, rng.integers(0, sizes + 1))
    layout = [int(x) for x in np.concatenate([[0], np.cumsum(room)])]
    dgc.set_layout(layout)
    counts = np.minimum(room, np.where(rng.random(tensors) < 0.3, 0, rng.integers(0, sizes + 1))).astype(np.int32)
    idx, val = np.zeros(max(1, layout[-1]), np.int32), np.zeros(max(1, layout[-1]), np.float32)
    for j in np.flatnonzero(counts):
        lo, c = layout[j], int(counts[j])
        idx[lo:lo + c] = offsets[j] + np.sort(rng.choice(int(sizes[j]), c, replace=False))
        val[lo:lo + c] = rng.standard_normal(c)
    used = np.concatenate([np.arange(layout[j], layout[j] + counts[j]) for j in range(tensors)]).astype(np.int64)
    runs, vals = expected_entries(idx[used].astype(np.int64), val[used])
    dev = [torch.from_numpy(t).cuda() for t in (idx, val, counts)]
    out_runs = torch.zeros(runs.size + 1, dtype=torch.int16, device="cuda")
    out_vals = torch.zeros(runs.size + 1, device="cuda")
    entries = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    dgc.dgc_encode(*dev, out_runs, out_vals, entries)
    assert int(entries) == runs.size
    assert np.array_equal(out_runs.cpu().numpy().view(np.uint16)[:-1], runs)
    assert np.array_equal(out_vals.cpu().numpy()[:-1].view(np.uint32), vals.view(np.uint32))
    dgc.close()


def test_encoding_many_tensors_takes_no_longer_than_compressing_them():
    """20000 tensors of 1500 elements: compress 500 us; the encoder 1260 when every workgroup walked all of them."""
    import torch
    offsets = np.arange(20001) * 1500
    n = int(offsets[-1])
    dgc = B.Dgc(B.make_config(density=0.001, flags=B.DGC_FLAG_SORTED_OUTPUT), offsets)
    layout = dgc.dgc_recommended_payload_layout(0.001)
    dgc.set_layout(layout)
    g = torch.randn(n, device="cuda")
    u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    out = dgc.alloc_payload("cuda")
    capacity = dgc.dgc_encode_max_entries(layout[-1])
    runs, vals = torch.zeros(capacity, dtype=torch.int16, device="cuda"), torch.zeros(capacity, device="cuda")
    entries = torch.zeros(1, dtype=torch.int32, device="cuda")
    times = []
    for call in (lambda: dgc.dgc_compress(g, u, v, *out, 0), lambda: dgc.dgc_encode(*out[:3], runs, vals, entries)):
        call()
        spans = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                call()
            b.record()
            b.synchronize()
            spans.append(a.elapsed_time(b) / 5)
        times.append(float(np.median(spans)))
    print("[many tensors] ms, compress and encode:", times, flush=True)
    assert times[1] < times[0]
    dgc.close()
