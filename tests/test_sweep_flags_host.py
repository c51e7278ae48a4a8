"""The flags that Lattice.sweep hands to the library, without a GPU."""
from __future__ import annotations

import pytest
import torch

import paper_1006_2566_amd as hsg


@pytest.fixture
def sent(monkeypatch):
    got = []

    class Library:
        def __getattr__(self, name):
            return lambda lat, params, *rest: got.append((name, params._obj.flags)) or 0

    class Stream:
        cuda_stream = 0
    lat = hsg.Lattice(32, device="cpu", init=None)
    monkeypatch.setattr(hsg, "lib", lambda: Library())
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream())

    def flags(f, **kw):
        lat.sweep(T=0.5, flags=f, **kw)
        lat.sweep_timed(T=0.5, flags=f, **kw)
        (a, x), (b, y) = got[-2:]
        assert (a, b) == ("hsg_sweep", "hsg_sweep_timed") and x == y
        return x
    return flags


@pytest.mark.parametrize("name", ["STREAM_LOADS", "PLANE_LAUNCH", "PHASE_LAUNCH", "PHASE_MC", "FUSED"])
def test_default_flags_with_a_traversal_added(sent, name):
    extra = getattr(hsg, "HSG_" + name)
    assert sent(hsg.default_flags(32) | extra) == hsg.HSG_SNAKE | extra


def test_flags_that_go_together(sent):
    brick = hsg.HSG_SNAKE | hsg.HSG_BRICK
    assert sent(None) == sent(hsg.default_flags(32)) == brick
    assert sent(hsg.HSG_BRICK) == hsg.HSG_BRICK and sent(0) == 0
    assert sent(hsg.HSG_STREAM_LOADS) == hsg.HSG_STREAM_LOADS
    assert sent(hsg.default_flags(32), heat_bath=True) == brick | hsg.HSG_HEAT_BATH
    assert sent(1 << 20) == 1 << 20  # unknown ones are the library's to refuse
