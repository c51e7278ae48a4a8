"""Which entry point a batch's sweep calls, without a GPU: a stand-in for the library records
the calls."""
from __future__ import annotations

import pytest
import torch

from paper_1006_2566_amd import batch as hb


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            return 0
        return call


class Stream:
    cuda_stream = 0

    def synchronize(self):
        pass


@pytest.fixture
def rec(monkeypatch):
    r = Recorder()
    hb._bind()
    monkeypatch.setattr(hb, "lib", lambda: r)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream())
    return r


def chains(L, n, **kw):
    return [hb.ChainSpec(L=L, seed=i, J_group=1000 * L + i, J_seed=i, **kw) for i in range(n)]


def route(rec, batch, n_sweeps=1):
    rec.calls.clear()
    batch.sweep(n_sweeps)
    return [c.replace("hsg_batch_", "") for c in rec.calls]


def batch(specs, **kw):
    return hb.Batch(specs, device="cpu", init=False, **kw)


def test_a_workgroup_size_asked_for(rec):
    b = batch(chains(16, 4))
    assert route(rec, b) == ["group_sweep"]
    for threads in (64, 128, 512, 1024):
        b.threads = threads
        assert route(rec, b) == ["sweep"]
        assert route(rec, batch(chains(16, 4), threads=threads)) == ["sweep"]
    for threads in (0, hb.THREADS):
        b.threads = threads
        assert route(rec, b) == ["group_sweep"]
    assert route(rec, batch(chains(8, 4), threads=256)) == ["sweep"]


def test_budgets_that_may_end_before_the_call(rec):
    """At L = 32 and one phase a sweep, 600 * 2 * 27 <= 32^3 < 600 * 2 * 28."""
    b = batch(chains(32, 4), track_remaining=True)
    assert route(rec, b, 27) == ["group_sweep"]
    assert route(rec, b, 28) == route(rec, b, 10 ** 6) == ["sweep"]
    b = batch(chains(32, 4, n_or=2), track_remaining=True)
    assert route(rec, b, 9) == ["group_sweep"] and route(rec, b, 10) == ["sweep"]
    assert route(rec, batch(chains(32, 4)), 10 ** 6) == ["group_sweep"]


def test_budgets_of_a_batch_in_groups(rec, monkeypatch):
    monkeypatch.setattr(hb, "tiles_pay", lambda specs: False)
    monkeypatch.setattr(hb, "GROUP_SPIN_BYTES", 2 * 3 * 32 ** 3 * 4)
    b = batch(chains(32, 8) + chains(16, 3), track_remaining=True)
    assert b._tiles[4].size - 1 == 4
    assert route(rec, b, 6) == ["sweep", "group_sweep"]  # the small chains, then the others
    assert route(rec, b, 7) == ["sweep"]


def test_tuned_size_keeps_the_tiles(rec, monkeypatch, tmp_path):
    from paper_1006_2566_amd import autotune
    monkeypatch.setattr(autotune, "device_key", lambda: "cpu")
    monkeypatch.setattr(autotune, "_event_ms", lambda fn, reps: fn() or 1.0)
    path = str(tmp_path / "tune.json")
    tiled, alone = batch(chains(32, 4)), batch(chains(8, 4))
    assert autotune.batch_threads(tiled, path=path) == hb.THREADS
    assert route(rec, tiled) == ["group_sweep"]
    assert autotune.batch_threads(alone, path=path) == 64  # the first of equals
    assert route(rec, alone) == ["sweep"]
