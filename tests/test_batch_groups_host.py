"""Which batches run in groups, and the groups the entry point refuses."""
from __future__ import annotations

import ctypes

import numpy as np

from paper_1006_2566_amd import batch as hb
from paper_1006_2566_amd import lib


def chains(L, n):
    return [hb.ChainSpec(L=L, seed=i, J_group=i, J_seed=i) for i in range(n)]


def test_rule():
    assert hb.groups_pay(chains(32, 2049)) and not hb.groups_pay(chains(30, 5000))
    assert hb.groups_pay(chains(48, 10) + chains(8, 100))
    assert not hb.groups_pay(chains(32, 1) + chains(16, 20000))


def test_rejected_groups():
    hb._bind()
    d = hb._Batch(2, 0, 1, 1, 1, 1, 1, 1, None, 1, 256, 0)

    def call(groups, n_groups=None, n=0):
        g = None if groups is None else np.asarray(groups, dtype=np.int32)
        return lib().hsg_batch_group_sweep(
            ctypes.byref(d), 1, 1, None if g is None else g.ctypes.data,
            len(groups) - 1 if n_groups is None else n_groups, 256, 1, 1, 0, 0, n, None)
    assert call([0, 2]) == 0 == call([0, 3, 4])
    for bad in ([0, 0], [0, 3, 3], [1, 4], [0, 1], [0, 5, 2]):
        assert call(bad) == -1, bad
    assert call([0, 4], n_groups=0) == -1 == call(None, n_groups=1)
    assert call([0, 4], n=-1) == -1
