"""Large batches in groups of chains, the small chains of a mixed batch with a workgroup
each: the same chains as with a workgroup each for all."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1006_2566_amd import batch
    return batch


def specs(hb, Ls):
    kinds = [dict(k=4), dict(k=1, n_or=2, renorm_every=2), dict(k=0, n_or=1),
             dict(k=2, heat_bath=True, renorm_every=3)]
    return [hb.ChainSpec(L=L, seed=3 + i, J_group=i, J_seed=50 + i, T=0.4 + 0.01 * i,
                         **kinds[i % 4]) for i, L in enumerate(Ls)]


def same(a, b):
    assert torch.equal(a.spins, b.spins) and torch.equal(a.sweep_ctr, b.sweep_ctr)
    # at most 2^11 tiles of a chain added in another order
    assert torch.allclose(a.E, b.E, rtol=1e-12, atol=1e-12)


# one chain a group, several, groups that end between chains of other sizes, none left alone
@pytest.mark.parametrize("dtype,Ls,group_bytes", [
    (torch.float32, (32, 8, 34, 16, 40, 2, 32, 30, 36), 1),
    (torch.float32, (32, 8, 34, 16, 40, 2, 32, 30, 36), 900_000),
    (torch.float64, (34, 10, 32, 32, 12), 800_000), (torch.float32, (32,) * 5, 1_000_000)])
def test_groups_equal_a_workgroup_per_chain(hb, monkeypatch, dtype, Ls, group_bytes):
    monkeypatch.setattr(hb, "tiles_pay", lambda specs: False)
    monkeypatch.setattr(hb, "GROUP_SPIN_BYTES", group_bytes)
    s = specs(hb, Ls)
    a, b = hb.Batch(s, dtype=dtype, track_remaining=True), hb.Batch(s, dtype=dtype,
                                                                   track_remaining=True)
    a._tiles = None
    groups = b._tiles[4]
    assert 2 <= groups.size - 1 <= sum(L >= 32 for L in Ls)
    assert (b._alone is None) == (min(Ls) >= 32)
    budget = torch.arange(len(Ls), dtype=torch.int32, device="cuda") % 5
    for n in (1, 3):
        for x in (a, b):
            x.remaining.copy_(budget)
            x.sweep(n)
        same(a, b)
        assert torch.equal(a.remaining, b.remaining)
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        with torch.cuda.graph(g, stream=st):
            b.sweep(2)
    torch.cuda.current_stream().wait_stream(st)
    for _ in range(3):
        for x in (a, b):
            x.remaining.copy_(budget)
        a.sweep(2)
        g.replay()
        torch.cuda.synchronize()
        same(a, b)
    assert int(b._tiles[3].count_nonzero()) == 0
    np.testing.assert_array_equal(np.sort(groups), groups)
