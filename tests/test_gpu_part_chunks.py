"""The part kernels of the receive side on payloads whose arrays start anywhere in a 128-byte line, with numbers of
pairs per part around the 64 and 256 slots that a wavefront takes at a time, in no order inside a part, and right up
to both ends of the arrays: the worker-ordered sum bit for bit.  Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from paper_1712_01887_amd import binding as B

pytestmark = pytest.mark.gpu

PART = 32768
SIZES = [3 * PART + 1000, 7, PART, 5000, 2 * PART - 1]
COUNTS = [0, 1, 3, 30, 33, 63, 65, 224, 225, 256, 257, 481, 4064, 4097]


def payload(layout, offsets, rng, shift_idx, shift_val, first):
    """Pairs per part taken from COUNTS in turn, shuffled inside the part; regions full where `first` says so."""
    import torch
    idx = np.zeros(layout[-1], np.int32)
    val = np.zeros(layout[-1], np.float32)
    counts = np.zeros(len(offsets) - 1, np.int32)
    pairs, turn = [], first
    for j in range(len(offsets) - 1):
        lo, hi = offsets[j], offsets[j + 1]
        at = layout[j]
        block = (lo // 1024) * 1024          # parts are counted from the 1024-element tile the tensor starts in
        while block < hi:
            a, b = max(lo, block), min(hi, block + PART)
            k = min(COUNTS[turn % len(COUNTS)], b - a, layout[j + 1] - at)
            if j == len(offsets) - 2:
                k = min(b - a, layout[j + 1] - at)   # the last region is full: the arrays end with the last pair
            e = a + rng.choice(b - a, k, replace=False)
            x = rng.standard_normal(k).astype(np.float32)
            idx[at:at + k], val[at:at + k] = e, x
            pairs.append((e, x))
            at += k
            turn += 1
            block += PART
        counts[j] = at - layout[j]
    held = []                                # the arrays lie at the very start, or end, of an allocation
    for host, shift in ((idx, shift_idx), (val, shift_val)):
        t = torch.empty(shift + host.size, dtype=torch.from_numpy(host).dtype, device="cuda")
        t[shift:] = torch.from_numpy(host).cuda()
        held.append(t[shift:])
    return pairs, held[0], held[1], torch.from_numpy(counts).cuda()


@pytest.mark.parametrize("workers", [1, 4, 16, 64])
@pytest.mark.parametrize("shift", [0, 1, 2, 31])
def test_parts_of_payloads_anywhere_in_a_line(workers, shift):
    import torch
    rng = np.random.default_rng([workers, shift])
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    n = int(offsets[-1])
    dgc = B.Dgc(B.make_config(density=0.25, num_workers=workers), offsets)
    layout = np.concatenate([[0], np.cumsum([min(s, 4 * 4100) for s in SIZES])]).tolist()
    dgc.set_layout(layout)
    made = [payload(layout, offsets, rng, shift, (shift * (w + 1)) % 33, w) for w in range(workers)]
    lists = tuple([m[i] for m in made] for i in (1, 2, 3))
    start = rng.standard_normal(n).astype(np.float32)
    lr = 0.25

    def ordered(dense, step):
        for pairs, *_ in made:
            for e, x in pairs:
                dense[e] = (dense[e] + np.float32(step) * x).astype(np.float32)
        return dense

    dense = torch.from_numpy(start).cuda()
    dgc.dgc_decompress_accumulate_regions(dense, *lists)
    assert np.array_equal(dense.cpu().numpy(), ordered(start.copy(), 1.0))
    dgc.dgc_dense_clear_regions(dense, lists[0], lists[2])
    cleared = ordered(start.copy(), 1.0)
    for pairs, *_ in made:
        for e, _ in pairs:
            cleared[e] = 0.0
    assert np.array_equal(dense.cpu().numpy(), cleared)
    dgc.dgc_decompress_replace_regions(dense, *lists, [lists[0][0]], [lists[2][0]])
    assert np.array_equal(dense.cpu().numpy(), ordered(np.zeros(n, np.float32), 1.0))
    theta = torch.from_numpy(start).cuda()
    dgc.dgc_sparse_sgd_apply_regions(theta, lr, *lists)
    assert np.array_equal(theta.cpu().numpy(), ordered(start.copy(), -lr))
    dgc.close()
