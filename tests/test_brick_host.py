"""HSG_BRICK without a GPU: where it is the default, the work size it needs, the flags it
does not go with, and the reciprocal division its kernel indexes with."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import paper_1006_2566_amd as hsg


def test_default_and_work_size():
    brick = hsg.HSG_SNAKE | hsg.HSG_BRICK
    for L in (2, 14, 16, 40, 64):
        assert hsg.default_flags(L) == brick
    assert hsg.default_flags(66) == hsg.HSG_SNAKE
    assert hsg.default_flags(40, torch.float64) == brick
    assert hsg.default_flags(42, torch.float64) == hsg.HSG_SNAKE
    for L, dtype, es in ((16, torch.float32, 4), (62, torch.float32, 4), (12, torch.float64, 8),
                         (40, torch.float64, 8)):
        second = 3 * L ** 3 * es
        work = hsg.lattice_bytes(L, dtype)[2]
        assert work >= second + 8 * 1024 * 64
    # one workgroup holds these: no second array
    assert hsg.lattice_bytes(14)[2] < hsg.lattice_bytes(16)[2] - 2 * 14 ** 3 * 4


@pytest.mark.parametrize("flags", [4, 32, 64, 128, 256, 4 | 16])
def test_flags_it_does_not_go_with(flags):
    lib = hsg.lib()
    d = hsg._Lattice(16, 0, 1, 0, 0x1000, 0x2000, 0x3000, 0x4000, hsg.lattice_bytes(16)[2])
    p = hsg._SweepParams(1.0, 1, 1, 0, hsg.HSG_BRICK | flags)
    assert lib.hsg_sweep(ctypes.byref(d), ctypes.byref(p), 1, None) == -1
    p = hsg._SweepParams(1.0, 1, 1, 0, hsg.HSG_BRICK)
    assert lib.hsg_sweep_noalloc(ctypes.byref(d), ctypes.byref(p), 1, None) == -1
    assert d.sweep == 0


def test_reciprocal_division():
    """floor(2^20 / d) + 1 from a reciprocal up to an ulp off divides every n < 4096 exactly."""
    n = np.arange(4096, dtype=np.uint64)
    one = np.float32(1)
    for d in range(1, 64):
        r = one / np.float32(d)
        near = (r,) if d & (d - 1) == 0 else (np.nextafter(r, np.float32(0)), r, np.nextafter(r, one))
        for x in near:
            m = np.uint64(np.uint32(np.float32(1048576) * x) + 1)
            assert int((n * m).max()) < 2 ** 32
            assert np.array_equal((n * m) >> np.uint64(20), n // np.uint64(d))
