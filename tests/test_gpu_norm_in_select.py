"""Clipping where the norm's sums are formed in the selection's launch: sizes around a workgroup's shares and with
elements behind the last four, on both sides of the line to the launch of its own, in a captured graph, and with a
selection that finds no share and sums them all itself.  Run with `-m gpu` on an MI355X."""

import ctypes as C

import numpy as np
import pytest

from oracle import dgc_oracle as O
from paper_1712_01887_amd import binding as B
from tests.parity import Pair, capture

pytestmark = pytest.mark.gpu

MOST = 4 << 20


def set_looks(dgc, looks):
    hook = B.load().dgc_test_set_looks
    hook.argtypes, hook.restype = [C.c_void_p, C.c_int32], None
    hook(dgc._h, looks)


def never_look(p):
    set_looks(p.dgc, 0)


@pytest.mark.parametrize("sizes", [[1], [3, 2], [4096 * 4], [4096 * 4 + 1], [50000, 5 * 4096 * 4 - 50000 + 2],
                                   [7001] * 64, [7001] * 65])
@pytest.mark.parametrize("alone", [False, True])
def test_norm_and_selection(sizes, alone):
    p = Pair(np.concatenate([[0], np.cumsum(sizes)]), momentum=0.9, density=0.004, seed=5, clip_threshold=0.3, num_workers=4)
    if alone:
        never_look(p)
    rng = np.random.default_rng(len(sizes))
    for it in range(3):
        p.step((10.0 ** (it - 1) * rng.standard_t(3, p.n)).astype(np.float32), it, label=f"{sizes[:2]} alone={alone}")
    p.step(np.zeros(p.n, np.float32), 3, label="zeros")      # a sum of nothing is there, too
    p.close()


@pytest.mark.parametrize("n", [MOST - 1, MOST, MOST + 1])
@pytest.mark.parametrize("density", [0.001, 0.05])
def test_norm_around_the_line(n, density):
    import torch
    g = (1e-2 * np.random.default_rng(n).standard_t(3, n)).astype(np.float32)
    dgc = B.Dgc(B.make_config(density=density, clip_threshold=0.5, num_workers=4), np.array([0, n // 3, n]))
    dgc.set_layout(dgc.dgc_recommended_payload_layout(density))
    u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    out = dgc.alloc_payload("cuda")
    want = float(np.sqrt((g.astype(np.float64) ** 2).sum()))
    for it in range(2):
        dgc.dgc_compress(torch.from_numpy(g).cuda(), u, v, *out, it)
        d = dgc.dgc_get_diagnostics()
        assert abs(d.norm - want) <= 1e-12 * want and d.scale == np.float32(min(1.0, 0.25 / d.norm))
    dgc.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1e30])
def test_norm_that_is_not_finite(value):
    import torch
    n = 100000
    g = torch.zeros(n, device="cuda")
    g[77777] = value
    dgc = B.Dgc(B.make_config(density=0.01, clip_threshold=0.5), np.array([0, n]))
    dgc.set_layout(dgc.dgc_recommended_payload_layout(0.01))
    u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    out = dgc.alloc_payload("cuda")
    for it in range(2):
        dgc.dgc_compress(g, u, v, *out, it)
        d = dgc.dgc_get_diagnostics()
        finite = np.isfinite(value)
        assert bool(d.flags & B.DGC_DIAG_NONFINITE) != finite
        assert not finite or d.scale == np.float32(0.5 / d.norm)
    dgc.close()


def test_norm_in_a_graph():
    """Every replay finds the places of the shares empty."""
    import torch
    n = 300001
    kw = dict(density=0.01, clip_threshold=0.5, num_workers=4, momentum=0.9, seed=2)
    dgc = B.Dgc(B.make_config(**kw), np.array([0, n]))
    layout = dgc.dgc_recommended_payload_layout(0.01)
    dgc.set_layout(layout)
    rng = np.random.default_rng(1)
    g, u, v = (torch.zeros(n, device="cuda") for _ in range(3))
    out = dgc.alloc_payload("cuda")
    dgc.dgc_compress(g, u, v, *out, 0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with capture(graph):
        dgc.dgc_compress(g, u, v, *out, 0)
    u.zero_()
    v.zero_()
    for it in range(4):
        x = ((it + 1) * 1e-2 * rng.standard_t(3, n)).astype(np.float32)
        g.copy_(torch.from_numpy(x))
        graph.replay()
        d = dgc.dgc_get_diagnostics()
        want = float(np.sqrt((x.astype(np.float64) ** 2).sum()))
        assert abs(d.norm - want) <= 1e-12 * want, it
    dgc.close()


@pytest.mark.parametrize("n", [4096 * 4 * 2 + 3, 70 * 4096 * 4, MOST - 1])            # 3 shares, 70 and 128
def test_norm_of_shares_found_and_formed_again(n):
    """Every second share is found, and the others are formed again beside it: the same bits as when all are found, and as
    when none is, in sets of a tensor and of several."""
    import torch
    rng = np.random.default_rng(n)
    grads = [torch.from_numpy((10.0 ** (it - 2) * rng.standard_t(3, n)).astype(np.float32)).cuda() for it in range(3)]
    for offsets in (np.array([0, n]), np.array([0, n // 3, n // 3 + 5, n])):
        seen = []
        for looks in (4096, -4096, 0):
            dgc = B.Dgc(B.make_config(density=0.004, clip_threshold=0.3, num_workers=4, momentum=0.9, seed=3), offsets)
            dgc.set_layout(dgc.dgc_recommended_payload_layout(0.004))
            set_looks(dgc, looks)
            u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
            out = dgc.alloc_payload("cuda")
            norms = []
            for it, g in enumerate(grads):
                dgc.dgc_compress(g, u, v, *out, it)
                d = dgc.dgc_get_diagnostics()
                want = float(np.sqrt((g.cpu().numpy().astype(np.float64) ** 2).sum()))
                assert abs(d.norm - want) <= 1e-12 * want, (looks, it)
                norms.append((d.norm, d.scale))
            seen.append((norms, u, v, out[2].clone(), out[3].clone()))
            dgc.close()
        for other in seen[1:]:
            assert seen[0][0] == other[0]
            assert all(torch.equal(a, b) for a, b in zip(seen[0][1:], other[1:]))
