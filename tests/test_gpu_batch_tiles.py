"""Batches swept as launches over tiles of every chain: the same spins as the workgroup per
chain, bit for bit, the same energies (another order of binary64 additions), the same
counters and budgets, also captured in a graph; and the parallel exchange round against
the rule walked slot by slot."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1006_2566_amd import batch
    batch._bind()
    return batch


def specs(hb, Ls, **kw):
    """Chains of the given sizes, with every kind of schedule."""
    kinds = [dict(k=4), dict(k=1, n_or=2, renorm_every=2), dict(k=3, heat_bath=True),
             dict(k=0, n_or=1), dict(k=5, n_or=1, renorm_every=1)]
    return [hb.ChainSpec(L=L, seed=11 + i, J_group=i, J_seed=7 + i, T=0.3 + 0.1 * i,
                         **(kw or kinds[i % len(kinds)])) for i, L in enumerate(Ls)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("Ls", [
    (2, 4, 6, 8, 10, 22, 34),   # a tile larger than the chain, chains of several tiles
    (32, 30, 32, 18, 16, 40),   # colour sites a multiple of the tile and not
])
def test_tiles_equal_workgroup_per_chain(hb, Ls, dtype):
    a, b = hb.Batch(specs(hb, Ls), dtype), hb.Batch(specs(hb, Ls), dtype)
    a._tiles, b._tiles = None, b._tile_table()
    for n in (1, 3):
        a.sweep(n)
        b.sweep(n)
        assert torch.equal(a.spins, b.spins)
        assert torch.equal(a.sweep_ctr, b.sweep_ctr)
        # sums of the same binary64 terms: N additions of rounding 2^-53 of the sum of |terms|
        assert torch.allclose(a.E, b.E, rtol=1e-12, atol=1e-12)
    assert int(b._tiles[3].count_nonzero()) == 0  # the partials are left at zero


@pytest.mark.parametrize("chains", [None, [0, 3, 5], [1], [6]])
def test_table_equals_the_hosts(hb, chains):
    b = hb.Batch(specs(hb, (2, 8, 22, 34, 6, 64, 16)))
    active = np.arange(b.n, dtype=np.int32) if chains is None else np.array(chains, dtype=np.int32)
    tiles, first, n, partials, _ = b._tile_table(None if chains is None else active)
    out, m = np.zeros((n, 2), dtype=np.int32), ctypes.c_int32()
    hb.check(hb.lib().hsg_batch_tiles(b.table.ctypes.data, b.n, active.ctypes.data, active.size,
                                      hb.TILE_SITES, out.ctypes.data, n, ctypes.byref(m)))
    assert m.value == n == first[-1] and partials.count_nonzero() == 0
    np.testing.assert_array_equal(tiles.cpu().numpy(), out)
    for c, t in enumerate(first[:-1].tolist()):
        assert c not in active or tiles[t].tolist() == [c, 0]


def test_budgets_and_graph_replay(hb):
    budget = [0, 1, 5, 2, 7]
    Ls = (16, 24, 6, 32, 20)
    runs = []
    for tiled in (False, True):
        b = hb.Batch(specs(hb, Ls), track_remaining=True)
        b._tiles = b._tile_table() if tiled else None
        b.remaining.copy_(torch.tensor(budget, dtype=torch.int32))
        b.sweep(2)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                b.sweep(2)
        torch.cuda.current_stream().wait_stream(s)
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
        runs.append(b)
    a, b = runs
    assert b.sweep_ctr.tolist() == budget and b.remaining.tolist() == [0] * 5
    assert torch.equal(a.spins, b.spins) and torch.equal(a.sweep_ctr, b.sweep_ctr)
    assert torch.allclose(a.E, b.E, rtol=1e-12)


@pytest.mark.parametrize("n_ladders,n_temps", [(1, 1), (1, 2), (3, 5), (2, 24), (40, 24)])
def test_exchange_round_equals_the_rule(hb, n_ladders, n_temps):
    """One workgroup (up to 256 slots) and several; odd and even rounds and ladders."""
    import oracle
    n = n_ladders * n_temps
    b = hb.Batch([hb.ChainSpec(L=4, seed=i, J_group=0, J_seed=1) for i in range(n)])
    betas = np.linspace(3.0, 1.0, n_temps)
    pt = hb.Tempering(b, np.arange(n).reshape(n_ladders, n_temps), betas, seed=5)
    slots = np.arange(n).reshape(n_ladders, n_temps).copy()
    for rnd in range(5):
        E = b.E.cpu().numpy()
        for l in range(n_ladders):
            for t in range(rnd % 2, n_temps - 1, 2):
                ca, cb = slots[l, t], slots[l, t + 1]
                w = oracle.philox(np.array([[t, rnd, l, 3]], dtype=np.uint32), 5)[0]
                u = (2 * (int(w[0]) >> 9) + 1) * 2.0 ** -24
                d = (betas[t] - betas[t + 1]) * (E[ca] - E[cb])
                if d >= 0 or u < np.exp(d):
                    slots[l, t], slots[l, t + 1] = cb, ca
        pt.exchange()
        assert np.array_equal(pt.chain_at_slot.cpu().numpy(), slots)
        beta = np.empty(n)
        beta[slots.reshape(-1)] = np.tile(betas, n_ladders)
        assert np.array_equal(b.beta.cpu().numpy(), beta)
        assert int(pt.round.item()) == rnd + 1
        b.sweep(1)


@pytest.mark.parametrize("L", [2, 14, 16, 26, 40])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_pair_overlap_and_energy_at_remainders(hb, L, dtype):
    """Colours of fewer sites than the workgroup, whole rounds, and remainders."""
    b = hb.Batch([hb.ChainSpec(L=L, seed=3, J_group=0, J_seed=1),
                  hb.ChainSpec(L=L, seed=4, J_group=0, J_seed=1)], dtype)
    N = L ** 3
    (s0, J), (s1, _) = ([v.double().cpu() for v in b.export_chain(c)] for c in (0, 1))
    q = b.overlap([(0, 1)])[0].cpu()
    ref = torch.cat([(s0 @ s1.T).reshape(-1) / N, s0.sum(1) / N, s1.sum(1) / N])
    assert (q - ref).abs().max() <= 1e-13
    s, Jr = s0.reshape(3, L, L, L), J.reshape(3, L, L, L)
    H = -sum(float((Jr[d] * (s * torch.roll(s, -1, dim)).sum(0)).sum())
             for d, dim in enumerate((3, 2, 1)))
    assert abs(float(b.energies(recompute=True)[0]) - H) <= 1e-12 * N
