"""Long calls of lattices that one workgroup holds: how many launches they are cut into, the
same spins as pass by pass, and the sweep index at the end of its range."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as m
    m.lib()
    return m


# 8192 phases or groups of hits a launch, 4096 sweeps, at least one
@pytest.mark.parametrize("k,n_or,heat_bath,n,launches", [
    (1, 0, False, 4097, 2), (64, 0, False, 1025, 3), (61, 4, False, 410, 2), (0, 8, False, 1024, 1),
    (500, 1, True, 4096, 1), (1, 16383, False, 2, 2), (65535, 0, False, 2, 2)])
def test_launches_of_a_call(hsg, k, n_or, heat_bath, n, launches):
    a, b = [hsg.Lattice(4, torch.float32, seed=3) for _ in range(2)]
    kw = dict(T=0.5, k=k, n_or=n_or, n_sweeps=n, heat_bath=heat_bath)
    rec = b.sweep_timed(flags=hsg.HSG_BRICK, **kw)
    assert [kind for kind, _ in rec] == [hsg.LAUNCH_MARCH] * launches
    a.sweep(flags=0, **kw)
    assert torch.equal(a.spins, b.spins)
    # the energy changes of 64 sites and n sweeps, added in another order
    assert abs(a.E.item() - b.E.item()) <= 1e-12 * n * max(1, k)


@pytest.mark.parametrize("L,dtype", [(8, torch.float32), (14, torch.float32), (10, torch.float64)])
@pytest.mark.parametrize("every", [2, 3, 5])
def test_renormalisation_at_the_last_sweep_index(hsg, L, dtype, every):
    """Sweeps 2^32 - 3 to 2^32 - 1; 2^32 is a multiple of 2, not of 3 or 5."""
    a, b = [hsg.Lattice(L, dtype, seed=3) for _ in range(2)]
    for lat, flags in ((a, 0), (b, hsg.HSG_BRICK)):
        lat.sweep_index = 2 ** 32 - 3
        lat.sweep(T=0.5, k=1, n_or=1, renorm_every=every, n_sweeps=3, flags=flags)
    assert torch.equal(a.spins, b.spins) and b.sweep_index == 2 ** 32
