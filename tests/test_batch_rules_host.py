"""Which batches go over tiles, where their chains' hits and over-relaxation phases decide."""
from __future__ import annotations

import random

import numpy as np
import pytest

from paper_1006_2566_amd import batch as hb


def chains(L, n, **kw):
    return [hb.ChainSpec(L=L, seed=i, J_group=i, J_seed=i, **kw) for i in range(n)]


@pytest.mark.parametrize("L,n,k,n_or,pays", [
    (16, 112, 1, 2, True), (16, 113, 1, 1, False), (16, 192, 4, 1, True), (16, 152, 4, 2, True),
    (16, 153, 4, 2, False), (20, 480, 4, 2, True), (20, 481, 4, 2, False),
    (20, 416, 2, 1, True), (20, 417, 2, 1, False), (20, 512, 4, 1, True),
    (24, 512, 1, 4, True), (32, 2048, 1, 4, True), (32, 2049, 1, 4, False)])
def test_hits_and_phases(L, n, k, n_or, pays):
    assert hb.tiles_pay(chains(L, n, k=k, n_or=n_or)) is pays


@pytest.mark.parametrize("small,n_or,large,k,pays", [
    (8, 3, 32, 4, True), (8, 10, 32, 4, True), (8, 50, 32, 4, False), (8, 3, 20, 1, False),
    (12, 10, 20, 1, False), (16, 10, 20, 1, True), (16, 50, 32, 4, True), (24, 50, 32, 4, True)])
def test_phases_of_small_chains(small, n_or, large, k, pays):
    assert hb.tiles_pay(chains(small, 8, k=1, n_or=n_or) + chains(large, 8, k=k)) is pays


def test_groups_by_what_their_tiles_have_to_do():
    def some(f, n_or, k=4):
        n = int(3072 * f)
        return hb.groups_pay(chains(32, n, k=k, n_or=n_or) + chains(32, 3072 - n, k=k))
    assert some(1.0, 8) and some(0.2, 2) and some(0.5, 8) and some(0, 0)
    assert not some(0.01, 2) and not some(0.1, 8) and not some(0.33, 8)
    # phases of chains that have a workgroup each do not count, but the time they take does
    large = chains(48, 2400, k=4)
    assert hb.groups_pay(large + chains(16, 100, n_or=50))
    assert not hb.groups_pay(large + chains(24, 100, n_or=100))


def test_table_and_specs_are_the_same():
    g = random.Random(1)
    specs = [hb.ChainSpec(L=g.choice([4, 16, 32, 256]), seed=i, J_group=i, J_seed=i,
                          k=g.choice([0, 1, 4, 0xFFFF]), n_or=g.choice([1, 2, 0x7FFF]),
                          heat_bath=g.random() < 0.3) for i in range(400)]
    table = np.zeros(400, dtype=hb.CHAIN_DTYPE)
    for i, c in enumerate(specs):
        table[i] = (0, 0, 0, 0, c.L, c.k, c.n_or, 0, hb.HSG_HEAT_BATH if c.heat_bath else 0, 0)
    assert hb._kinds(table) == hb._kinds(specs) == hb._kinds(hb._kinds(specs))
