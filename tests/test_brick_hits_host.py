"""Small lattices with many hits run pass by pass; heat-bath draws, of which one counts, do not."""
from __future__ import annotations

import pytest
import torch

import paper_1006_2566_amd as hsg

F32, F64 = torch.float32, torch.float64


@pytest.mark.parametrize("L,dtype,n_or,most", [
    (10, F32, 0, 56), (12, F32, 1, 17), (14, F32, 0, 5), (14, F32, 2, 14), (34, F32, 1, 34),
    (44, F32, 0, 28), (46, F32, 1, 12), (48, F32, 2, 8), (64, F32, 3, 8), (10, F64, 1, 22),
    (14, F64, 0, 14), (34, F64, 0, 10), (40, F64, 1, 13)])
def test_most_hits(L, dtype, n_or, most):
    brick = hsg.HSG_SNAKE | hsg.HSG_BRICK
    assert hsg.call_flags(L, dtype, most, n_or=n_or) == brick
    assert hsg.call_flags(L, dtype, most + 1, n_or=n_or) == hsg.HSG_SNAKE
    assert hsg.call_flags(L, dtype, 0xFFFF, True, n_or) == brick


@pytest.mark.parametrize("L,dtype", [(2, F32), (8, F32), (16, F32), (32, F32), (8, F64), (12, F64), (16, F64), (32, F64)])
def test_any_number(L, dtype):
    assert hsg.call_flags(L, dtype, 0xFFFF, n_or=0) == hsg.HSG_SNAKE | hsg.HSG_BRICK
