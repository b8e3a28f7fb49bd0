"""Captures in the GPU tests (no GPU needed): nothing may be finalized while one is under way, because the
destructor of an earlier CUDAGraph waits for the device and takes the process down if it cannot."""

import contextlib
import gc
import glob
import os
import weakref

import pytest

from tests.parity import capture


class Finalized:
    """In the place of a CUDAGraph: notes whether a capture was under way when it went."""

    def __init__(self, log):
        self.log = log

    def __del__(self):
        self.log["seen"].append(self.log["capturing"])


def expect_an_error(log):
    """What a test with `pytest.raises(...) as err` leaves behind: its locals in a reference cycle."""
    graph = Finalized(log)
    with pytest.raises(ValueError) as err:
        raise ValueError("refused")
    assert err.value.args
    return weakref.ref(graph)


def test_nothing_is_finalized_inside_a_capture(monkeypatch):
    import torch
    log = {"capturing": False, "seen": []}

    @contextlib.contextmanager
    def graph_context(graph):
        log["capturing"] = True
        try:
            yield
        finally:
            log["capturing"] = False

    monkeypatch.setattr(torch.cuda, "graph", graph_context)
    thresholds = gc.get_threshold()
    gc.disable()
    before = expect_an_error(log)
    assert before() is not None                    # the function has returned and the object is still there
    try:
        gc.set_threshold(1, 1, 1)                  # every allocation may start the collector
        gc.enable()
        with capture(None):
            inside = expect_an_error(log)
            assert [[] for _ in range(1000)] and inside() is not None
        assert gc.isenabled()
    finally:
        gc.set_threshold(*thresholds)
        gc.enable()
    gc.collect()
    assert before() is None and inside() is None
    assert log["seen"] == [False, False]


def test_captures_of_the_gpu_tests_go_through_the_helper():
    here = os.path.dirname(os.path.abspath(__file__))
    for path in sorted(glob.glob(os.path.join(here, "test_gpu_*.py")) + glob.glob(os.path.join(here, "test_zz_*.py"))):
        with open(path) as f:
            assert "torch.cuda.graph(" not in f.read(), path
