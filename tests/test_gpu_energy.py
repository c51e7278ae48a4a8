"""The energy reduction against a plain binary64 sum, at the edges of its tile order: fewer
tiles than workgroups, one more, counts that eight XCDs do not divide, partial last tiles."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,dtype", [(2, torch.float32), (64, torch.float32), (80, torch.float64),
                                     (82, torch.float32), (84, torch.float32), (90, torch.float64),
                                     (102, torch.float32), (130, torch.float32)])
def test_energy_against_a_plain_sum(L, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as hsg
    lat = hsg.Lattice(L, dtype, seed=17 + L)
    s, J = (t.double().reshape(3, L, L, L) for t in lat.export())  # [component][z][y][x]
    ref = 0.0
    for d, axis in enumerate((3, 2, 1)):  # +x, +y, +z bonds
        ref -= (J[d] * (s * torch.roll(s, -1, dims=axis)).sum(0)).sum().item()
    scale = J.abs().sum().item()
    # 3 L^3 products of unit spins in binary64, whose rounding errors add like a random walk
    assert abs(lat.energy(recompute=True).item() - ref) <= 1e-14 * scale
