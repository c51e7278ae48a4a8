"""L = 1022 in binary32, whose 511 columns are cut into eight tiles of 63 and 64: the launch
with the Monte Carlo pass against the pass-by-pass schedule, bit for bit."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,heat_bath", [(4, False), (1, True)])
def test_tiles_of_two_widths(k, heat_bath):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as hsg
    L = 1022
    assert hsg.call_flags(L, torch.float32, k, heat_bath) & hsg.HSG_PHASE_MC
    a, b = [hsg.Lattice(L, torch.float32, seed=12) for _ in range(2)]
    kw = dict(T=0.4, k=k, n_or=1, renorm_every=2, n_sweeps=3, heat_bath=heat_bath)
    a.sweep(flags=hsg.HSG_SNAKE, **kw)
    b.sweep(**kw)
    assert torch.equal(a.spins, b.spins)
    # 4.2 million and 744 partial sums of the same binary64 energy changes
    assert abs(a.E.item() - b.E.item()) <= 1e-12 * abs(a.E.item())
