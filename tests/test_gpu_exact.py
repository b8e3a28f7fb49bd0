"""Exact selection (DGC_FLAG_EXACT_SELECT) from tensors of more than 32768 elements: a sampled band,
its keys listed by a pass over the tensor, the exact rank among those.  Bit for bit against the oracle,
at the edges of the range, where the band misses, where most elements are zero, and with NaNs.
Run with `-m gpu` on an MI355X."""

import numpy as np
import pytest

from oracle import dgc_oracle as O
from paper_1712_01887_amd import binding as B
from tests.parity import Pair, gather_payload

pytestmark = pytest.mark.gpu

EXACT = B.DGC_FLAG_EXACT_SELECT
# 32768 fits the registers of a workgroup, 32769 is the smallest that does not (a set that has a tensor above
# 65536 takes bands for all such); the others share tiles
SIZES = [5, 32769, 32768, 100003, 1, 70001, 262144, 29]


def band_sample(n, seed, iteration, tensor):
    """Positions of the band's sample: 1024 draws of 32 consecutive elements."""
    plan = O.SamplePlan(False, 32768, 0, 1024, n // 32, 0)
    return O.sample_positions(seed, iteration, tensor, plan, 32)


@pytest.mark.parametrize("density", [0.0005, 0.004, 0.02, 0.25, 0.68, 0.9])
@pytest.mark.parametrize("flags", [EXACT, EXACT | B.DGC_FLAG_SORTED_OUTPUT | B.DGC_FLAG_NESTEROV,
                                   EXACT | B.DGC_FLAG_NO_FACTOR_MASKING])
def test_exact_thresholds_of_large_tensors(density, flags):
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    # (no more than k pass an exact threshold: a region of k pairs cannot overflow)
    caps = None if flags == EXACT else [O.topk_count(density, s) for s in SIZES]
    clip = dict(clip_threshold=0.5, num_workers=4) if density == 0.004 else {}
    p = Pair(offsets, capacities=caps, momentum=0.9, density=density, seed=3, flags=flags, warmup_workspace=True, **clip)
    rng = np.random.default_rng(17)
    for it in range(2):
        g = (1e-2 * rng.standard_t(3, p.n)).astype(np.float32)
        res = p.step(g, it, label=f"exact d={density} flags={flags} it{it}")
        assert all(int(c) <= O.topk_count(density, s) for c, s in zip(res.counts, SIZES))
    assert p.dgc.dgc_query_plan(3)[:3] == (O.topk_count(density, SIZES[3]), SIZES[3], O.topk_count(density, SIZES[3]))
    p.close()


@pytest.mark.parametrize("sizes,listed", [
    ([65536, 40000, 7, 32769], False),             # no tensor above 65536 elements: a workgroup reads the tensor
    ([65537, 40000, 7, 32769], True),
    ([33000], False),
    ([57344] * 256 + [5], False),
    ([57345] + [32769] * 256, True),               # as many tensors as compute units, and more: above 57344
])
@pytest.mark.parametrize("density", [0.003, 0.3])
def test_exact_on_both_sides_of_the_rule_for_bands(sizes, listed, density):
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    p = Pair(offsets, momentum=0.9, density=density, seed=6, flags=EXACT)
    sampled = B.Dgc(B.make_config(momentum=0.9, density=density, seed=6), offsets)
    assert (p.dgc.dgc_workspace_bytes() > sampled.dgc_workspace_bytes()) == listed
    rng = np.random.default_rng(len(sizes))
    for it in range(2 if p.n < 1 << 20 else 1):
        g = (1e-2 * rng.standard_t(3, p.n)).astype(np.float32)
        p.step(g, it, label=f"exact, {len(sizes)} tensors up to {max(sizes)} d={density} it{it}")
    p.close()
    sampled.close()


@pytest.mark.parametrize("size", [81, 1000, 1500, 2048, 2049, 4096])
@pytest.mark.parametrize("rank", [78, 79, 80, 81, 127, 128])
def test_ranks_where_the_selection_of_small_tensors_changes_over(size, rank):
    """Up to 2048 elements the largest keys are listed for ranks below 80 only, above that up to rank 127."""
    offsets = np.arange(6) * size
    density = min(1.0, (rank - 0.5) / size)
    p = Pair(offsets, momentum=0.9, density=density, seed=8, flags=EXACT)
    rng = np.random.default_rng(size)
    for it in range(2):
        g = (1e-2 * rng.standard_t(3, p.n)).astype(np.float32)
        if it:
            g[: size // 2] = g[0]                      # ties across the rank
        p.step(g, it, label=f"rank {rank} of {size} it{it}")
    p.close()


@pytest.mark.parametrize("density", [0.001, 0.25])
@pytest.mark.parametrize("flags", [EXACT, EXACT | B.DGC_FLAG_SORTED_OUTPUT])
def test_exact_where_the_band_misses(density, flags):
    """The large values sit where the band's sample looks (fewer of them than are wanted)."""
    sizes = [777, 200001, 41]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    p = Pair(offsets, momentum=0.0, density=density, seed=9, flags=flags)
    rng = np.random.default_rng(5)
    for it in range(2):
        g = (1e-3 * rng.standard_normal(p.n)).astype(np.float32)
        pos = np.unique(band_sample(sizes[1], 9, it, 1))
        if density < 0.01:
            pos = pos[:180]                               # more than the rank the band starts at, fewer than k = 201
        g[offsets[1] + pos] = (5.0 + rng.random(pos.size)).astype(np.float32)
        assert pos.size < O.topk_count(density, sizes[1])
        p.step(g, it, label=f"exact, band misses d={density} it{it}")
    p.close()


@pytest.mark.parametrize("density", [0.001, 0.05])
@pytest.mark.parametrize("nonzero", [0, 40, 5000])
def test_exact_of_mostly_zero_tensors(density, nonzero):
    sizes = [100, 150000, 33000]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    p = Pair(offsets, momentum=0.9, density=density, seed=2, flags=EXACT)
    rng = np.random.default_rng(nonzero)
    for it in range(2):
        g = np.zeros(p.n, np.float32)
        g[rng.choice(p.n, nonzero, replace=False)] = rng.standard_normal(nonzero).astype(np.float32)
        p.step(g, it, label=f"exact, {nonzero} non-zeros d={density} it{it}")
    p.close()


@pytest.mark.parametrize("nans", [3, 500])
@pytest.mark.parametrize("density", [0.001, 0.02])
def test_exact_ranks_nans_above_everything_and_sends_none(nans, density):
    import torch
    sizes = [300, 100000, 40000]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    n = int(offsets[-1])
    dgc = B.Dgc(B.make_config(momentum=0.5, density=density, seed=4, flags=EXACT), offsets)
    layout = dgc.dgc_recommended_payload_layout(density)
    dgc.set_layout(layout)
    rng = np.random.default_rng(nans)
    g = rng.standard_t(3, n).astype(np.float32)
    g[rng.choice(n, nans, replace=False)] = np.nan
    g[777] = np.float32(np.inf)
    u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    out = dgc.alloc_payload("cuda")
    dgc.dgc_compress(torch.from_numpy(g).cuda(), u, v, *out, 0)
    ou, ov = np.zeros(n, np.float32), np.zeros(n, np.float32)
    with np.errstate(invalid="ignore"):
        res = O.compress(g, ou, ov, offsets, O.OracleConfig(momentum=0.5, density=density, seed=4, exact_select=True), 0)
    per_idx, per_val, counts = gather_payload(layout, *out[:3])
    assert np.array_equal(out[3].cpu().numpy(), res.thresholds, equal_nan=True)
    assert np.array_equal(counts, res.counts)
    for j in range(len(sizes)):
        assert np.array_equal(per_idx[j], res.indices[j]) and np.array_equal(per_val[j], res.values[j])
    assert np.array_equal(u.cpu().numpy(), ou, equal_nan=True) and np.array_equal(v.cpu().numpy(), ov, equal_nan=True)
    dgc.close()


@pytest.mark.parametrize("density", [0.02, 0.3])
def test_exact_where_the_band_is_crowded(density):
    """Three tenths of the tensor lie inside the band, where its sample did not look: the list does not fit."""
    sizes = [64, 200001]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    p = Pair(offsets, momentum=0.0, density=density, seed=12, flags=EXACT)
    rng = np.random.default_rng(8)
    g = rng.standard_normal(p.n).astype(np.float32)
    pos = np.unique(band_sample(sizes[1], 12, 0, 1))
    unseen = np.setdiff1d(np.arange(sizes[1]), pos)
    crowd = rng.choice(unseen, 60000, replace=False)
    mid = np.quantile(np.abs(g[offsets[1] + pos]), 1.0 - density)
    g[offsets[1] + crowd] = (mid * (1.0 + 1e-6 * rng.integers(-50, 50, crowd.size))).astype(np.float32)
    p.step(g, 0, label=f"exact, crowded band d={density}")
    p.close()


def test_exact_compress_leaves_the_scratch_of_the_receive_side_alone():
    """Which bytes of the workspace the part kernels, the encoder and the decoder use is seen from what they
    change; a compress call afterwards must not change them."""
    import torch
    offsets = np.concatenate([[0], np.cumsum([64, 200001, 40000, 70000])])
    n = int(offsets[-1])
    dgc = B.Dgc(B.make_config(momentum=0.9, density=0.02, seed=3, flags=EXACT | B.DGC_FLAG_SORTED_OUTPUT), offsets)
    layout = dgc.dgc_recommended_payload_layout(0.02)
    dgc.set_layout(layout)
    dgc.ensure_workspace("cuda").fill_(0x5A)
    u, v, dense = (torch.zeros(n, device="cuda") for _ in range(3))
    out = dgc.alloc_payload("cuda")
    grads = [torch.from_numpy((1e-2 * np.random.default_rng(it).standard_t(3, n)).astype(np.float32)).cuda() for it in range(2)]
    dgc.dgc_compress(grads[0], u, v, *out, 0)
    capacity = dgc.dgc_encode_max_entries(layout[-1])
    runs, vals = torch.zeros(capacity, dtype=torch.int16, device="cuda"), torch.zeros(capacity, device="cuda")
    entries = torch.zeros(1, dtype=torch.int32, device="cuda")

    def changes(call):
        before = dgc.workspace.clone()
        call()
        return before != dgc.workspace

    payload = ([out[0]] * 3, [out[1]] * 3, [out[2]] * 3)
    parts = changes(lambda: dgc.dgc_decompress_replace_regions(dense, *payload))
    wire = changes(lambda: dgc.dgc_encode(out[0], out[1], out[2], runs, vals, entries))
    wire |= changes(lambda: dgc.dgc_decode_accumulate(dense, [runs] * 3, [vals] * 3, [int(entries)] * 3))
    assert int(parts.sum()) > 0 and int(wire.sum()) > 0
    changed = changes(lambda: dgc.dgc_compress(grads[1], u, v, *out, 1))
    assert int(changed.sum()) > 0
    assert int((changed & parts).sum()) == 0 and int((changed & wire).sum()) == 0
    dgc.close()


def test_exact_selection_in_a_workspace_without_the_list():
    """A workspace of the size that a set without exact selection needs holds the band lists in the place of the
    receive side's scratch, and so does the static array where the whole does not fit it."""
    import torch
    offsets = np.concatenate([[0], np.cumsum(SIZES)])
    n = int(offsets[-1])
    kw = dict(momentum=0.9, density=0.02, seed=3)
    rng = np.random.default_rng(23)
    sampled = B.Dgc(B.make_config(**kw), offsets)
    without = sampled.dgc_workspace_bytes()
    sides = []
    for _ in range(3):
        dgc = B.Dgc(B.make_config(flags=EXACT, **kw), offsets)
        dgc.set_layout(dgc.dgc_recommended_payload_layout(0.02))
        sides.append((dgc, torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), dgc.alloc_payload("cuda")))
    # a slot per tensor above 32768 elements, three words per 64 elements
    extra = sides[0][0].dgc_workspace_bytes() - without
    assert 4 * 512 + 12 * (n // 64) <= extra <= 4 * 512 + 12 * (n // 64) + 512
    guard = torch.full((without + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    sides[1][0].workspace = guard
    sides[1][0]._ws_ptr = (guard.data_ptr() + 255) // 256 * 256
    sides[1][0]._ws_bytes = without
    for it in range(3):
        g = torch.from_numpy((1e-2 * rng.standard_t(3, n)).astype(np.float32)).cuda()
        for dgc, u, v, out in sides[:2]:
            dgc.dgc_compress(g, u, v, *out, it)
        sides[2][0].dgc_compress_static(g, *sides[2][1:3], *sides[2][3], it)
        for side in sides[1:]:
            for a, b in zip(sides[0][1:3] + sides[0][3][2:], side[1:3] + side[3][2:]):
                assert torch.equal(a, b), it
    behind = sides[1][0]._ws_ptr - guard.data_ptr() + without
    assert bool((guard[behind:] == 0xA5).all())
    sides[1][0]._ws_bytes = without - 256
    with pytest.raises(B.DgcError):
        sides[1][0].dgc_compress(g, *sides[1][1:3], *sides[1][3], 3)
    for dgc in [side[0] for side in sides] + [sampled]:
        dgc.close()


@pytest.mark.parametrize("numel", [25000000])
def test_exact_selection_of_a_large_set_in_the_static_array(numel):
    """With its lists the set does not fit the static array, without them it does."""
    import torch
    offsets = np.array([0, 40001, numel - 70003, numel])
    kw = dict(momentum=0.9, density=0.001, seed=5)
    dgc = [B.Dgc(B.make_config(flags=EXACT, **kw), offsets) for _ in range(2)]
    assert dgc[0].dgc_workspace_bytes() > 8 << 20 > B.Dgc(B.make_config(**kw), offsets).dgc_workspace_bytes()
    results = []
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    g = torch.randn(numel, device="cuda", generator=gen)
    for k, d in enumerate(dgc):
        d.set_layout(d.dgc_recommended_payload_layout(0.001))
        u, v, out = torch.zeros(numel, device="cuda"), torch.zeros(numel, device="cuda"), d.alloc_payload("cuda")
        for it in range(2):
            (d.dgc_compress_static if k else d.dgc_compress)(g, u, v, *out, it)
        results.append((u, v, out[2], out[3]))
        d.close()
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("whole_regions", [False, True])
@pytest.mark.parametrize("flags", [EXACT, EXACT | B.DGC_FLAG_SORTED_OUTPUT | B.DGC_FLAG_NO_FACTOR_MASKING])
@pytest.mark.parametrize("many", [9000, 12500, 30000])
def test_exact_at_low_densities_where_many_pass_the_floor(many, flags, whole_regions):
    """Large values where the band's sample did not look: up to 12288 that pass are listed on chip, more in the payload
    region if they fit there, and otherwise the tiles are walked over."""
    sizes = [500, 200001, 90000, 64]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    caps = list(sizes) if whole_regions else None
    p = Pair(offsets, capacities=caps, momentum=0.0, density=0.002, seed=14, flags=flags)
    rng = np.random.default_rng(many)
    for it in range(2):
        g = (1e-3 * rng.standard_normal(p.n)).astype(np.float32)
        unseen = np.setdiff1d(np.arange(sizes[1]), np.unique(band_sample(sizes[1], 14, it, 1)))
        pos = rng.choice(unseen, many, replace=False)
        g[offsets[1] + pos] = rng.standard_normal(many).astype(np.float32) + 3.0
        p.step(g, it, label=f"exact, {many} unseen flags={flags} it{it}")
    p.close()


@pytest.mark.parametrize("density", [0.001, 0.002, 0.0021])
@pytest.mark.parametrize("size", [40960, 40961, 65537, 3_000_000, 4_600_000])
def test_exact_on_both_sides_of_the_rule_for_bands_in_the_pass(density, size):
    """Up to 0.2 %, from 40961 elements on and as long as what exceeds the floor fits one workgroup's list; with the
    re-threshold beside it, and with a density that changes under one handle and workspace."""
    offsets = [0, 40000, 40000 + size]
    p = Pair(offsets, layout_density=0.02, momentum=0.9, density=density, seed=15, flags=EXACT, refine_alpha=2.0)
    rng = np.random.default_rng(size)
    for it, d in enumerate((density, 0.02, density)):
        p.set_density(d)
        g = (1e-2 * rng.standard_t(3, p.n)).astype(np.float32)
        p.step(g, it, label=f"exact, n={size} d={d}")
    p.close()


@pytest.mark.parametrize("kind", ["one magnitude", "four levels", "few of one magnitude", "ties at the end", "rows"])
@pytest.mark.parametrize("size", [50_000, 400_001])
def test_floor_in_the_pass_with_ties_and_rows(kind, size):
    """The floor is itself the threshold: found among the first elements, far into the tensor, or nowhere but at its end;
    and large values side by side, so that tiles lose many elements at once.  A NaN beside them."""
    rng = np.random.default_rng(size)
    offsets = [0, 333, 333 + size]
    p = Pair(offsets, layout_density=0.02, momentum=0.0, density=0.002, seed=16, flags=EXACT)
    g = rng.standard_normal(offsets[-1]).astype(np.float32)
    where = np.arange(offsets[-1])
    if kind == "one magnitude":
        g = np.sign(g)
    elif kind == "four levels":
        g = np.clip(np.round(g), -2, 2)
    elif kind == "few of one magnitude":
        g = np.sign(g) * (rng.random(g.size) < 0.01)
    elif kind == "ties at the end":
        g = np.where(where >= offsets[-1] - size // 100, np.sign(g), 0.0)
    else:
        g = g * np.where(where // 650 % 100 == 0, 100.0, 1.0)
    g = g.astype(np.float32)
    p.step(g, 0, label=f"exact, {kind}, n={size}")
    g[offsets[-1] // 2] = np.nan
    p.step(g, 1, label=f"exact, {kind} and a NaN, n={size}")
    p.close()


def in_rows(g, lo, hi, width, rows, rng):
    """Large values in rows of a matrix that fills [lo, hi)."""
    for r in rng.choice((hi - lo) // width, rows, replace=False):
        g[lo + r * width:lo + (r + 1) * width] *= 100


@pytest.mark.parametrize("kind", ["spread", "one in rows", "all in rows", "few magnitudes", "misses", "mostly zero", "unseen rows",
                                  "rows of NaNs", "many NaNs"])
@pytest.mark.parametrize("tensors", [3, 7])
def test_exact_of_sets_that_decide_on_the_device(kind, tensors):
    """Sets large enough for floors in the pass, with tensors so long that the sample has to bear the floor out: all
    floors in the pass, some, or (with fewer elements beside a tensor that cannot) none.  A NaN in every tensor in the second
    call, another density in the third."""
    sizes = [333] + [3_000_000] * tensors + [40_001, 20]
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    flags = EXACT | (B.DGC_FLAG_NO_FACTOR_MASKING if kind == "misses" else 0)
    p = Pair(offsets, layout_density=0.004, momentum=0.0, density=0.001, seed=21, flags=flags)
    rng = np.random.default_rng([tensors, len(kind)])
    for it, d in enumerate((0.001, 0.001, 0.004) if tensors == 3 else (0.0005, 0.001)):
        p.set_density(d)
        g = rng.standard_normal(p.n, dtype=np.float32)
        lo, hi = int(offsets[1]), int(offsets[2])
        if kind == "one in rows":
            in_rows(g, lo, hi, 1500, 3, rng)
        elif kind == "all in rows":
            for j in range(1, tensors + 1):
                in_rows(g, int(offsets[j]), int(offsets[j + 1]), 1500, 3, rng)
        elif kind == "few magnitudes":
            g[lo:hi] = np.clip(np.round(g[lo:hi]), -2, 2)
        elif kind == "mostly zero":
            g[lo:hi] *= np.arange(hi - lo) // 1500 % 50 == 0
        elif kind == "misses":                       # one large value to a sampled block: fewer than k, more than the floor's rank
            first = np.unique(band_sample(sizes[1], 21, it, 1) // 32 * 32)
            g[lo + first + rng.integers(0, 32, first.size)] = 50.0 + rng.random(first.size, dtype=np.float32)
        elif kind == "rows of NaNs" and it == 1:     # more than k: the threshold is one, and nothing is sent
            g[lo + 30_000:lo + 36_000] = np.nan
        elif kind == "many NaNs" and it == 1:
            g[lo + rng.choice(hi - lo, 6000, replace=False)] = np.nan
        elif kind == "unseen rows":                  # many more pass than the sample lets expect: the list in LDS does not hold them
            unseen = np.setdiff1d(np.arange(sizes[1] // 32), band_sample(sizes[1], 21, it, 1) // 32)
            g[lo + (rng.choice(unseen, 700, replace=False)[:, None] * 32 + np.arange(32)).ravel()] *= 100
        if it == 1:
            g[(offsets[:-1] + offsets[1:]) // 2] = np.nan
        p.step(g, it, label=f"exact, {kind}, {tensors} tensors, d={d} it{it}")
    p.close()


def test_floors_in_the_pass_and_collected_bands_in_the_static_array():
    """The static array has no areas for bands: those that are collected beside floors in the pass lie in other scratch."""
    import torch
    offsets = np.concatenate([[0], np.cumsum([777] + [3_000_000] * 7 + [50_001])])
    n = int(offsets[-1])
    rng = np.random.default_rng(11)
    sides = []
    for _ in range(2):
        dgc = B.Dgc(B.make_config(momentum=0.9, density=0.001, seed=31, flags=EXACT), offsets)
        dgc.set_layout(dgc.dgc_recommended_payload_layout(0.001))
        sides.append((dgc, torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), dgc.alloc_payload("cuda")))
    for it in range(3):
        g = rng.standard_normal(n, dtype=np.float32)
        in_rows(g, int(offsets[2]), int(offsets[3]), 1500, 3, rng)
        if it == 2:
            for j in range(1, 7):
                in_rows(g, int(offsets[j]), int(offsets[j + 1]), 1500, 5, rng)
        g = torch.from_numpy(g).cuda()
        sides[0][0].dgc_compress(g, *sides[0][1:3], *sides[0][3], it)
        sides[1][0].dgc_compress_static(g, *sides[1][1:3], *sides[1][3], it)
        for a, b in zip(sides[0][1:3] + sides[0][3][2:], sides[1][1:3] + sides[1][3][2:]):
            assert torch.equal(a, b), it
        (ia, va, _), (ib, vb, _) = (gather_payload(side[0]._layout, *side[3][:3]) for side in sides)
        assert all(np.array_equal(a, b) for a, b in zip(ia + va, ib + vb)), it
    for side in sides:
        side[0].close()
