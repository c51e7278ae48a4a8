"""The tile form of a batched sweep without a GPU: rejected arguments and the rule that
chooses it."""
from __future__ import annotations

import ctypes

import pytest

from paper_1006_2566_amd import batch as hb
from paper_1006_2566_amd import lib


def chains(L, n):
    return [hb.ChainSpec(L=L, seed=i, J_group=i, J_seed=i) for i in range(n)]


def test_rejected_arguments():
    hb._bind()
    d = hb._Batch(2, 0, 1, 1, 1, 1, 1, 1, None, 1, 256, 0)
    good = dict(tiles=1, first=1, n_tiles=2, tile_sites=256, partials=1, any_mc=1, max_n_or=0,
                renorm=0, n=1)

    def call(d=d, **kw):
        a = {**good, **kw}
        return lib().hsg_batch_tile_sweep(ctypes.byref(d) if d else None, a["tiles"], a["first"],
                                          a["n_tiles"], a["tile_sites"], a["partials"],
                                          a["any_mc"], a["max_n_or"], a["renorm"], a["n"], None)
    assert call(n=0) == 0
    for bad in (dict(d=None), dict(tiles=None), dict(first=None), dict(partials=None),
                dict(n_tiles=1), dict(n=-1), dict(max_n_or=-1), dict(max_n_or=0x8000),
                dict(tile_sites=32), dict(tile_sites=100), dict(tile_sites=2048),
                dict(d=hb._Batch(0, 0, 1, 1, 1, 1, 1, 1, None, 1, 256, 0))):
        assert call(**bad) == -1, bad


def test_rejected_table():
    hb._bind()
    f = lib().hsg_batch_tile_table
    for bad in ((None, 2, 256, 8, 8), (8, 0, 256, 8, 8), (8, 2, 100, 8, 8), (8, 2, 2048, 8, 8),
                (8, 2, 256, None, 8), (8, 2, 256, 12, 8), (8, 2, 256, 8, None)):
        assert f(*bad, None) == -1, bad


@pytest.mark.parametrize("L,n,pays", [
    (8, 1, False), (8, 5000, False), (12, 48, False), (16, 192, True), (16, 193, False),
    (20, 512, True), (20, 513, False), (24, 512, True), (24, 4096, False), (32, 1, True),
    (32, 2048, True), (32, 2049, False), (256, 1, True)])
def test_rule(L, n, pays):
    assert hb.tiles_pay(chains(L, n)) is pays


def test_rule_on_mixed_sizes():
    assert hb.tiles_pay(chains(48, 10) + chains(8, 100))
    assert not hb.tiles_pay(chains(32, 1) + chains(16, 20000))
