"""HSG_BRICK, the small lattices' form with several colour passes per launch (the default
for them), against the pass-by-pass schedule: the same spins bit for bit, the same energy
in another order of binary64 additions, whatever the schedule, at the edges of every range
of sizes the rule tells apart."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
F32, F64 = torch.float32, torch.float64

# k, n_or, heat bath, renormalise every, sweeps: odd and even numbers of phases, groups of
# four hits complete, incomplete and more than one, no Monte Carlo phase, no other phase
SCHEDULES = [(4, 1, False, 2, 3), (1, 0, False, 1, 3), (3, 2, False, 0, 1), (6, 0, False, 2, 2),
             (8, 1, False, 0, 1), (5, 1, True, 1, 2), (0, 3, False, 2, 3), (0, 1, False, 1, 1)]


@pytest.fixture(scope="module")
def hsg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as m
    m.lib()
    return m


def pair(hsg, L, dtype):
    return [hsg.Lattice(L, dtype, seed=21 + L) for _ in range(2)]


def same(a, b):
    assert torch.equal(a.spins, b.spins) and a.sweep_index == b.sweep_index
    # the same energy changes added in another order: at most 2^13 partial sums a lattice
    assert abs(a.E.item() - b.E.item()) <= 1e-12 * max(1.0, abs(a.E.item()))


@pytest.mark.parametrize("L,dtype", [(L, F32) for L in (2, 4, 8, 10, 12, 14, 16, 18, 32, 34, 46,
                                                        48, 52, 54, 62, 64, 66)]
                         + [(L, F64) for L in (2, 8, 10, 12, 14, 22, 24, 32, 34, 38, 40, 42)])
def test_brick_equals_pass_by_pass(hsg, L, dtype):
    a, b = pair(hsg, L, dtype)
    for k, n_or, hb, R, n in SCHEDULES:
        for lat, flags in ((a, hsg.HSG_SNAKE), (b, hsg.HSG_SNAKE | hsg.HSG_BRICK)):
            lat.sweep(T=0.45, k=k, n_or=n_or, renorm_every=R, n_sweeps=n, heat_bath=hb, flags=flags)
        same(a, b)


def test_launches_of_many_sweeps(hsg):
    a, b = pair(hsg, 4, F32)  # a launch holds at most 4096 sweeps
    a.sweep(T=0.5, k=1, renorm_every=3, n_sweeps=4099, flags=0)
    b.sweep(T=0.5, k=1, renorm_every=3, n_sweeps=4099)
    same(a, b)


@pytest.mark.parametrize("L", [8, 24])
def test_captured_in_a_graph(hsg, L):
    """A captured call replays its own sweep indices; eager work lies between the replays."""
    a, b = pair(hsg, L, F32)
    b.sweep(T=0.5, k=4, n_or=1, n_sweeps=3)
    b.sweep_index = 0
    b.init_random()
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
    """The flag is ignored where the work buffer holds no second spin array."""
    a, b = pair(hsg, 20, F32)
    b._d.work_bytes -= 3 * 20 ** 3 * 4
    a.sweep(T=0.5, k=4, n_or=1, n_sweeps=2, flags=hsg.HSG_SNAKE)
    rec = b.sweep_timed(T=0.5, k=4, n_or=1, n_sweeps=2, flags=hsg.HSG_SNAKE | hsg.HSG_BRICK)
    assert [kd for kd, _ in rec] == [1, 1, 2, 2, 1, 1, 2, 2, 0]
    same(a, b)
