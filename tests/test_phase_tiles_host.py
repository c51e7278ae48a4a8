"""The tiles of the phase launches, without a GPU: for every lattice, precision and form, the
tiles that a plan cuts have the columns, rows and places that the kernel of the form deals
with, no two sites of a tile share a place, and the launch fits its arrays."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import paper_1006_2566_amd as hsg

LATTICES = [64, *range(98, 1025, 2)]


def plan(L, dtype, passes):
    n, T, wave = (ctypes.c_int32 * 3)(), ctypes.c_int32(), ctypes.c_int32()
    rc = hsg.lib().hsg_phase_tiles(L, dtype, passes, n, ctypes.byref(T), ctypes.byref(wave))
    return None if rc else (tuple(n), T.value, bool(wave.value))


def extents(E, n):
    """The different lengths of n tiles of an extent E; they cover it."""
    cut = [t * E // n for t in range(n + 1)]
    assert cut[0] == 0 and cut[-1] == E
    return set(np.diff(cut).tolist())


def places(items, n, w, h, wave):
    """LDS places of the items of a window of n rows of w columns, h of them halo on either
    side, as the kernels deal them to threads."""
    i = np.arange(items)
    if not wave:
        return i[i < n * w]
    e = i - 64 * n
    c = e & (2 * h - 1)
    row = np.where(e < 0, i >> 6, e >> h)
    col = np.where(e < 0, h + (i & 63), np.where(c < h, c, 64 + c))
    return (row * w + col)[e < 2 * h * n]


@pytest.mark.parametrize("dtype,passes", [(d, p) for d in (0, 1) for p in (2, 3, 4)])
def test_every_place_is_one_site(dtype, passes):
    most = 512 if dtype else 1024                                  # threads, colour-0 sites
    colour1 = {2: 1024 if dtype else 1536, 3: 672 if dtype else 1344, 4: most}[passes]
    halo = {2: 1, 3: 2, 4: 4}[passes]                              # rows around a tile
    for L in LATTICES:
        (px, py, pz), T, wave = plan(L, dtype, passes)
        assert T % 64 == 0 and 64 <= T <= most, L
        widths, heights, runs = extents(L // 2, px), extents(L, py), extents(L, pz)
        assert min(widths) > 0 and min(heights) > 0 and min(runs) > 0, L
        hx = int(px > 1)
        if passes == 3:  # a partial energy per workgroup, where the passes have one per tile
            assert px * py * pz <= -(-L * L // 2 // 256) * L, L
        assert not wave or (passes == 3 and hx), L
        for nx in widths:
            for ny in heights:
                if passes == 4:  # one window for all stages
                    windows = [(T, ny + 2 * halo, nx + 6 * hx, 3 * hx, most)]
                else:            # colour 0; colour 1, two sites a thread; colour 1 after B
                    r0 = ny + 2 * halo
                    windows = [(T, r0, nx + 2 * hx, hx, most),
                               (2 * T, r0 + 2, nx + 4 * hx, 2 * hx, colour1)]
                    if passes == 3:
                        windows.append((T, r0 - 2, nx + 2 * hx, hx, most))
                for items, n, w, h, size in windows:
                    p = places(items, n, w, h, wave)
                    assert n * w <= size, (L, nx, ny)
                    assert np.array_equal(np.sort(p), np.arange(n * w)), (L, nx, ny, n, w)


def test_where_there_are_none():
    for L, dtype, passes in ((96, 0, 2), (1026, 1, 3), (66, 0, 4), (128, 0, 1), (128, 0, 5),
                             (99, 0, 2), (128, 2, 2)):
        assert plan(L, dtype, passes) is None
    assert hsg.lib().hsg_phase_tiles(128, 0, 2, None, None, None) == -1
