"""HSG_PHASE_LAUNCH and HSG_PHASE_MC over the lattices they apply to, against the
pass-by-pass schedule: the same spins bit for bit, the same energy (in another order of
binary64 additions when the launch carries a Monte Carlo pass), whatever the schedule."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
F32, F64 = torch.float32, torch.float64

# k, n_or, heat bath, renormalise every, sweeps: odd and even numbers of phases, groups of
# four hits complete and incomplete, no Monte Carlo phase
SCHEDULES = [(4, 1, False, 2, 3), (1, 2, False, 1, 2), (6, 1, False, 0, 2), (1, 1, True, 1, 4),
             (0, 3, False, 2, 2), (2, 4, False, 0, 1), (1, 5, True, 2, 3), (0, 1, False, 3, 7)]


@pytest.fixture(scope="module")
def hsg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as m
    m.lib()
    return m


def same(a, b):
    assert torch.equal(a.spins, b.spins) and a.sweep_index == b.sweep_index
    # the same energy changes added in another order: at most 2^15 partial sums a lattice
    assert abs(a.E.item() - b.E.item()) <= 1e-12 * max(1.0, abs(a.E.item()))


# The smallest lattice and its neighbour, rows a multiple of a wave and not, runs of unequal
# length, tiles of whole rows with rows left over, tiles cut in x (evenly and not) into two
# and more, more workgroups than compute units, and runs in z that fill their last round
@pytest.mark.parametrize("L,dtype", [(L, F32) for L in (64, 98, 100, 126, 128, 150, 178, 202, 226,
                                                        254, 300, 302, 354, 402, 544)]
                         + [(L, F64) for L in (64, 98, 110, 128, 150, 170, 222, 260, 404, 448)])
def test_phase_launches_equal_passes(hsg, L, dtype):
    lats = [hsg.Lattice(L, dtype, seed=5 + L) for _ in range(3)]
    for k, n_or, hb, R, n in SCHEDULES:
        for lat, flags in zip(lats, (hsg.HSG_SNAKE, hsg.HSG_SNAKE | hsg.HSG_PHASE_LAUNCH,
                                     hsg.HSG_SNAKE | hsg.HSG_PHASE_MC)):
            lat.sweep(T=0.45, k=k, n_or=n_or, renorm_every=R, n_sweeps=n, heat_bath=hb, flags=flags)
        assert torch.equal(lats[0].E, lats[1].E)  # the passes' own order
        same(lats[0], lats[1])
        same(lats[0], lats[2])


@pytest.mark.parametrize("L,dtype,k", [(100, F32, 4), (130, F32, 2), (210, F32, 2), (190, F64, 4)])
def test_default_of_a_call(hsg, L, dtype, k):
    kinds = {0: [1, 1, 2, 2, 1, 1, 2, 2, 0], hsg.HSG_PHASE_LAUNCH: [1, 1, 3, 1, 1, 3, 0],
             hsg.HSG_PHASE_MC: [1, 1, 4, 1, 3, 0]}
    a, b = [hsg.Lattice(L, dtype, seed=9) for _ in range(2)]
    a.sweep(T=0.5, k=k, n_or=1, n_sweeps=2, flags=0)
    rec = b.sweep_timed(T=0.5, k=k, n_or=1, n_sweeps=2)
    phase = hsg.call_flags(L, dtype, k) & (hsg.HSG_PHASE_LAUNCH | hsg.HSG_PHASE_MC)
    assert [kd for kd, _ in rec] == kinds[phase]
    same(a, b)


def test_a_wave_per_row(hsg):
    """L = 512, whose tiles are 64 columns: a wave takes a row, others the halo columns."""
    for k, hb in ((4, False), (1, False), (1, True)):
        a, b = [hsg.Lattice(512, F32, seed=8) for _ in range(2)]
        for lat, flags in ((a, 0), (b, hsg.HSG_PHASE_MC)):
            lat.sweep(T=0.45, k=k, n_or=1, renorm_every=2, n_sweeps=3, heat_bath=hb, flags=flags)
        assert torch.equal(a.spins, b.spins)
        assert abs(a.E.item() - b.E.item()) <= 1e-12 * abs(a.E.item())


# launches that a call's over-relaxation phases run in: two phases (5), one (3), with the next
# Monte Carlo pass (4), two passes (2, 2); an even number of the first three
@pytest.mark.parametrize("k,n_or,R,n,flags,kinds", [
    (0, 1, 0, 4, "PHASE_LAUNCH", [5, 5]), (0, 1, 0, 2, "PHASE_LAUNCH", [3, 3]),
    (0, 1, 0, 3, "PHASE_LAUNCH", [5, 3]), (0, 1, 2, 5, "PHASE_LAUNCH", [5, 0, 5, 0, 2, 2]),
    (0, 1, 1, 2, "PHASE_LAUNCH", [3, 0, 3, 0]), (0, 2, 1, 3, "PHASE_LAUNCH", [5, 0, 5, 0, 3, 3, 0]),
    (0, 3, 0, 2, "PHASE_LAUNCH", [5, 5, 3, 3]), (1, 2, 0, 2, "PHASE_LAUNCH", [1, 1, 5, 1, 1, 5, 0]),
    (1, 3, 0, 1, "PHASE_LAUNCH", [1, 1, 5, 3, 0]), (1, 4, 0, 1, "PHASE_LAUNCH", [1, 1, 5, 5, 0]),
    (1, 2, 0, 2, "PHASE_MC", [1, 1, 3, 4, 1, 3, 3, 0]),
    (1, 3, 0, 2, "PHASE_MC", [1, 1, 5, 4, 1, 5, 3, 0]), (1, 2, 0, 1, "PHASE_MC", [1, 1, 3, 3, 0])])
def test_launches_of_a_call(hsg, k, n_or, R, n, flags, kinds):
    a, b = [hsg.Lattice(100, F32, seed=9) for _ in range(2)]
    kw = dict(T=0.5, k=k, n_or=n_or, renorm_every=R, n_sweeps=n)
    a.sweep(flags=0, **kw)
    assert [kd for kd, _ in b.sweep_timed(flags=getattr(hsg, "HSG_" + flags), **kw)] == kinds
    same(a, b)


def test_captured_in_a_graph(hsg):
    """A captured call replays its own sweep indices; eager work lies between the replays."""
    a, b = [hsg.Lattice(130, F32, seed=6) for _ in range(2)]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            b.sweep(T=0.5, k=4, n_or=1, n_sweeps=3)
    torch.cuda.current_stream().wait_stream(s)
    for _ in range(3):
        a.sweep_index = 0
        a.sweep(T=0.5, k=4, n_or=1, n_sweeps=3, flags=0)
        g.replay()
        torch.cuda.synchronize()
        same(a, b)


def test_work_buffer_without_second_array(hsg):
    """The flags are ignored where the work buffer holds no second spin array."""
    a, b = [hsg.Lattice(100, F32, seed=4) for _ in range(2)]
    b._d.work_bytes -= 3 * 100 ** 3 * 4
    a.sweep(T=0.5, k=4, n_or=1, n_sweeps=2, flags=hsg.HSG_SNAKE)
    rec = b.sweep_timed(T=0.5, k=4, n_or=1, n_sweeps=2, flags=hsg.HSG_SNAKE | hsg.HSG_PHASE_MC)
    assert [kd for kd, _ in rec] == [1, 1, 2, 2, 1, 1, 2, 2, 0]
    same(a, b)
