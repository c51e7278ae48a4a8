"""Launches of an over-relaxation phase without a GPU: the lattices they apply to, the work
size, and the flags of a sweep that names none."""
from __future__ import annotations

import torch

import paper_1006_2566_amd as hsg


def test_lattices_and_work_size():
    assert hsg.phase_supported(98) and not hsg.phase_supported(99)
    assert not any(hsg.phase_supported(L) for L in (62, 66, 96, 1026))
    for L, dtype, es in ((98, torch.float32, 4), (1024, torch.float64, 8)):
        assert hsg.lattice_bytes(L, dtype)[2] >= 3 * L ** 3 * es
    assert hsg.lattice_bytes(1026)[2] < 3 * 1026 ** 3


def test_flags_of_a_call():
    one, carry = hsg.HSG_SNAKE | hsg.HSG_PHASE_LAUNCH, hsg.HSG_SNAKE | hsg.HSG_PHASE_MC
    f64 = torch.float64
    assert hsg.call_flags(64) == hsg.HSG_SNAKE | hsg.HSG_BRICK
    assert hsg.call_flags(96) == hsg.call_flags(1026) == hsg.HSG_SNAKE
    assert hsg.call_flags(98, k=2) == hsg.call_flags(126, k=3) == hsg.call_flags(204, k=4) == one
    assert hsg.call_flags(126, k=0, heat_bath=True) == hsg.call_flags(254, k=5) == one
    assert hsg.call_flags(98) == hsg.call_flags(114, k=2) == hsg.call_flags(218) == carry
    assert hsg.call_flags(128, k=3) == hsg.call_flags(128, k=9, heat_bath=True) == carry
    assert hsg.call_flags(226, k=4) == hsg.call_flags(226, heat_bath=True) == carry
    assert hsg.call_flags(256, k=8) == carry
    assert hsg.call_flags(206, k=2) == hsg.call_flags(224, k=4) == hsg.HSG_SNAKE
    assert hsg.call_flags(224, heat_bath=True) == hsg.HSG_SNAKE
    assert hsg.call_flags(124, f64) == hsg.call_flags(446, f64, k=5) == one
    assert hsg.call_flags(448, f64, heat_bath=True) == one
    assert hsg.call_flags(126, f64) == hsg.call_flags(180, f64, k=4) == carry
    assert hsg.call_flags(448, f64, k=5) == one
    assert hsg.call_flags(162, f64) == hsg.call_flags(178, f64, k=8) == hsg.HSG_SNAKE


def test_flags_of_a_call_with_more_phases():
    one, carry = hsg.HSG_SNAKE | hsg.HSG_PHASE_LAUNCH, hsg.HSG_SNAKE | hsg.HSG_PHASE_MC
    f64 = torch.float64
    assert hsg.call_flags(130, n_or=2) == hsg.call_flags(256, k=4, n_or=2) == one
    assert hsg.call_flags(210, k=4, n_or=2) == hsg.call_flags(448, k=8, n_or=4) == one
    assert hsg.call_flags(310, k=4, n_or=2) == hsg.call_flags(310, heat_bath=True, n_or=2) == carry
    assert hsg.call_flags(400, f64, n_or=2) == hsg.call_flags(170, f64, k=4, n_or=3) == one
    assert hsg.call_flags(210, n_or=3) == hsg.call_flags(190, f64, k=4, n_or=3) == carry
    assert hsg.call_flags(210, k=0) == one and hsg.call_flags(210, k=2) == hsg.HSG_SNAKE
