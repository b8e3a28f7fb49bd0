"""Encoding in one launch: numbers of workgroup slots on both sides of the line to two launches, lists around a slot's 4096
pairs, gaps that take fillers, empty regions, calls one after the other with decoding between them (which uses the same
scratch), captured calls, and workgroups that find no need of another and form them all themselves.  Entry by entry.
Run with `-m gpu` on an MI355X."""

import ctypes as C

import numpy as np
import pytest

from oracle import dgc_oracle as O
from paper_1712_01887_amd import binding as B
from tests.parity import capture

pytestmark = pytest.mark.gpu

CHUNK = 4096


class Encoder:
    def __init__(self, sizes, capacities, alone):
        self.offsets = np.concatenate([[0], np.cumsum(sizes)])
        self.layout = np.concatenate([[0], np.cumsum(capacities)]).tolist()
        self.dgc = B.Dgc(B.make_config(density=0.01, flags=B.DGC_FLAG_SORTED_OUTPUT), self.offsets)
        self.dgc.set_layout(self.layout)
        if alone:
            self.set_looks(0)

    def set_looks(self, looks):
        hook = B.load().dgc_test_set_looks
        hook.argtypes, hook.restype = [C.c_void_p, C.c_int32], None
        hook(self.dgc._h, looks)

    def payload(self, counts, rng):
        """Ascending indices of which a third lie in the first hundredth of every tensor: long gaps behind them."""
        import torch
        idx, val = np.zeros(self.layout[-1], np.int32), np.zeros(self.layout[-1], np.float32)
        flat_idx, flat_val = [], []
        for j, c in enumerate(counts):
            lo, size = int(self.offsets[j]), int(self.offsets[j + 1] - self.offsets[j])
            near = min(c // 3, size // 100)
            e = lo + np.sort(np.concatenate([rng.choice(max(1, size // 100), near, replace=False),
                                             size // 100 + rng.choice(size - size // 100, c - near, replace=False)]))
            x = rng.standard_normal(c).astype(np.float32)
            idx[self.layout[j]:self.layout[j] + c], val[self.layout[j]:self.layout[j] + c] = e, x
            flat_idx.append(e)
            flat_val.append(x)
        self.expect = O.encode(np.concatenate(flat_idx).astype(np.int64), np.concatenate(flat_val))
        return tuple(torch.from_numpy(t).cuda() for t in (idx, val, np.asarray(counts, np.int32)))

    def out(self):
        import torch
        cap = self.expect[0].size + 3
        return (torch.zeros(cap, dtype=torch.int16, device="cuda"), torch.zeros(cap, device="cuda"),
                torch.full((1,), -1, dtype=torch.int32, device="cuda"))

    def check(self, runs, vals, num):
        e = int(num.item())
        assert e == self.expect[0].size
        assert np.array_equal(runs[:e].cpu().numpy().view(np.uint16), self.expect[0])
        assert np.array_equal(vals[:e].cpu().numpy(), self.expect[1])


@pytest.mark.parametrize("alone", [False, True])
@pytest.mark.parametrize("sizes,capacities,counts", [
    ([300000], [CHUNK * 3], [0]),
    ([300000], [CHUNK * 3], [CHUNK * 2 + 1]),
    ([9000000, 50, 400000], [CHUNK + 1, 50, CHUNK], [40, 0, CHUNK]),                   # gaps of several fillers
    ([70000] * 40, [CHUNK] * 40, [CHUNK - 1, 0, 1, 4096] * 10),
    ([300] * 255, [300] * 255, [j % 4 for j in range(255)]),
    ([300] * 256, [300] * 256, [(7 * j) % 5 for j in range(256)]),
    ([300] * 257, [300] * 257, [(7 * j) % 5 for j in range(257)]),                     # two launches
    ([1200000] + [2000] * 100, [150 * CHUNK] + [2000] * 100, [100 * CHUNK + 77] + [300, 0] * 50),
])
def test_encode_once(sizes, capacities, counts, alone):
    import torch
    enc = Encoder(sizes, capacities, alone)
    rng = np.random.default_rng(len(sizes))
    for turn in range(3):
        payload = enc.payload(counts[turn % 2:] + counts[:turn % 2] if len(set(sizes)) == 1 else counts, rng)
        runs, vals, num = enc.out()
        enc.dgc.dgc_encode(*payload, runs, vals, num)
        enc.check(runs, vals, num)
        if int(num.item()):
            dense = torch.zeros(int(enc.offsets[-1]), device="cuda")
            e = int(num.item())
            enc.dgc.dgc_decode_accumulate(dense, [runs] * 5, [vals] * 5, [e] * 5)
    assert not (enc.dgc.dgc_get_diagnostics().flags & (B.DGC_DIAG_UNSORTED | B.DGC_DIAG_OVERFLOW))
    enc.dgc.close()


@pytest.mark.parametrize("tensors", [50, 200])
def test_unsorted_region_is_flagged(tensors):
    enc = Encoder([3000] * tensors, [200] * tensors, False)
    idx, val, counts = enc.payload([100] * tensors, np.random.default_rng(2))
    runs, vals, num = enc.out()
    enc.dgc.dgc_encode(idx, val, counts, runs, vals, num)
    assert not (enc.dgc.dgc_get_diagnostics().flags & B.DGC_DIAG_UNSORTED)
    at = enc.layout[tensors // 2]
    idx[at:at + 2] = idx[at:at + 2].flip(0)
    enc.dgc.dgc_encode(idx, val, counts, runs, vals, num)
    assert enc.dgc.dgc_get_diagnostics().flags & B.DGC_DIAG_UNSORTED
    enc.dgc.close()


def test_encode_once_in_a_graph():
    import torch
    tensors = 120
    enc = Encoder([70000] * tensors, [CHUNK] * tensors, False)
    rng = np.random.default_rng(4)
    payload = enc.payload([300] * tensors, rng)
    cap = enc.dgc.dgc_encode_max_entries(tensors * 400)
    runs, vals = torch.zeros(cap, dtype=torch.int16, device="cuda"), torch.zeros(cap, device="cuda")
    num = torch.zeros(1, dtype=torch.int32, device="cuda")
    enc.dgc.dgc_encode(*payload, runs, vals, num)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with capture(graph):
        enc.dgc.dgc_encode(*payload, runs, vals, num)
    for turn in range(4):
        fresh = enc.payload([(37 * j + 11 * turn) % 400 for j in range(tensors)], rng)
        for dst, src in zip(payload, fresh):
            dst.copy_(src)
        num.fill_(-1)
        graph.replay()
        enc.check(runs, vals, num)
        enc.dgc.dgc_encode(*payload, runs, vals, num)            # an eager call between the replays
        enc.check(runs, vals, num)
    enc.dgc.close()


@pytest.mark.parametrize("looks", [4096, -4096, 0])      # all needs of others found, every second one, none
@pytest.mark.parametrize("sizes,capacities,counts", [
    ([24575], [24575], [9000]), ([24576], [24576], [9000]),               # two launches, and one, for want of words for the needs
    ([700000] + [60] * 300, [150 * CHUNK] + [60, 0, 0] * 100, [100 * CHUNK + 77] + [60, 0, 0] * 100),      # slots searched for
    ([300] * 320, [300, 0, 300, 300, 0] * 64, [(5 * j) % 7 if j % 5 not in (1, 4) else 0 for j in range(320)]),
    ([90000] * 60, [4 * CHUNK] * 60, [(2777 * j) % (4 * CHUNK) for j in range(60)]),
])
def test_encode_with_needs_found_and_formed_again(sizes, capacities, counts, looks):
    """... and more tensors than a round of loads tells, some with no region at all."""
    enc = Encoder(sizes, capacities, False)
    enc.set_looks(looks)
    rng = np.random.default_rng(len(sizes))
    for _ in range(2):
        payload = enc.payload(counts, rng)
        out = enc.out()
        enc.dgc.dgc_encode(*payload, *out)
        enc.check(*out)
    enc.dgc.close()


@pytest.mark.parametrize("looks", [4096, -4096])
def test_encode_behind_exact_selection_in_its_scratch(looks):
    """In a workspace of the size that a set without exact selection needs the band lists of a compress call lie over the
    needs of the calls of the encoder before and behind it."""
    import torch
    sizes = [200001, 70000, 40000, 64]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    kw = dict(momentum=0.9, density=0.02, seed=3)
    sampled = B.Dgc(B.make_config(**kw), offsets)
    without = sampled.dgc_workspace_bytes()
    sampled.close()
    enc = Encoder(sizes, sizes, False)
    enc.dgc.close()
    enc.dgc = B.Dgc(B.make_config(flags=B.DGC_FLAG_EXACT_SELECT | B.DGC_FLAG_SORTED_OUTPUT, **kw), offsets)
    assert enc.dgc.dgc_workspace_bytes() > without
    enc.dgc.set_layout(enc.layout)
    enc.set_looks(looks)
    guard = torch.full((without + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    enc.dgc.workspace = guard
    enc.dgc._ws_ptr = (guard.data_ptr() + 255) // 256 * 256
    enc.dgc._ws_bytes = without
    u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    compressed = enc.dgc.alloc_payload("cuda")
    rng = np.random.default_rng(6)
    for it in range(4):
        payload = enc.payload([1000 * (it + 1), 3000, 0, 5], rng)
        out = enc.out()
        enc.dgc.dgc_encode(*payload, *out)
        enc.check(*out)
        g = torch.from_numpy((1e-2 * rng.standard_t(3, n)).astype(np.float32)).cuda()
        enc.dgc.dgc_compress(g, u, v, *compressed, it)
        idx, val, counts = (t.cpu().numpy() for t in compressed[:3])
        rows = [slice(enc.layout[j], enc.layout[j] + int(c)) for j, c in enumerate(counts)]
        enc.expect = O.encode(np.concatenate([idx[r] for r in rows]).astype(np.int64), np.concatenate([val[r] for r in rows]))
        out = enc.out()
        enc.dgc.dgc_encode(*compressed[:3], *out)
        enc.check(*out)
    enc.dgc.close()
