"""Simulation.capture on the host alone (the torch graph calls replaced): no garbage collection
runs inside a capture, however much garbage there is, and the collector is left as it was found,
also after an error."""
import contextlib
import gc
import weakref

import pytest

torch = pytest.importorskip("torch")


class _Stream:
    def wait_stream(self, other):
        pass


@pytest.fixture
def sim(monkeypatch):
    from paper_2511_22951_amd import sim as S
    inside = []

    @contextlib.contextmanager
    def graph(g, stream=None):
        inside.append(True)
        try:
            yield
        finally:
            inside.pop()

    monkeypatch.setattr(torch.cuda, "Stream", _Stream)
    monkeypatch.setattr(torch.cuda, "current_stream", _Stream)
    monkeypatch.setattr(torch.cuda, "CUDAGraph", object)
    monkeypatch.setattr(torch.cuda, "graph", graph)
    x = S.Simulation.__new__(S.Simulation)
    x.rebuild_every, x.n_steps, x.fused, x.primed = 0, 0, False, False
    x.inside = inside
    return x


class _Node:
    pass


def _cycle():
    a, b = _Node(), _Node()
    a.other, b.other = b, a
    return weakref.ref(a)


@pytest.mark.parametrize("enabled", [True, False])
def test_no_collection_inside_a_capture(sim, enabled):
    runs = []

    def watch(phase, info):
        if phase == "start":
            runs.append(bool(sim.inside))

    dead = []

    def step(ev):
        assert sim.inside and all(d() is not None for d in dead)
        for _ in range(20):
            dead.append(_cycle())
        keep = [[k] for k in range(5000)]  # many allocations: a collection would be due
        del keep

    sim.step = step
    before, limits = gc.isenabled(), gc.get_threshold()
    (gc.enable if enabled else gc.disable)()
    gc.set_threshold(50)
    gc.callbacks.append(watch)
    try:
        sim.capture(4)
        assert gc.isenabled() == enabled
    finally:
        gc.callbacks.remove(watch)
        gc.set_threshold(*limits)
        (gc.enable if before else gc.disable)()
    assert not any(runs)
    gc.collect()
    assert len(dead) == 80 and all(d() is None for d in dead)


def test_collector_back_after_an_error(sim):
    def step(ev):
        raise RuntimeError("in the capture")

    sim.step = step
    before = gc.isenabled()
    gc.enable()
    try:
        with pytest.raises(RuntimeError):
            sim.capture(1)
        assert gc.isenabled() and not sim._capturing
    finally:
        (gc.enable if before else gc.disable)()
