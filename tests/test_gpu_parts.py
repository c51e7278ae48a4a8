"""Overlaps and energies of chains by several workgroups each: the same as by one, up to the
order of the binary64 sums."""
from __future__ import annotations

import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one part, the largest chain of one and the smallest of several, many parts, chains of other
# sizes than the largest
@pytest.mark.parametrize("dtype,Ls", [(torch.float32, (2, 48, 50, 96)), (torch.float64, (32, 20, 8)),
                                      (torch.float32, (16,)), (torch.float32, (128, 4))])
def test_parts_equal_one_workgroup(dtype, Ls):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as hsg
    from paper_1006_2566_amd import batch as hb
    specs = [hb.ChainSpec(L=L, seed=10 * L + r, J_group=g, J_seed=L, T=0.5)
             for g, L in enumerate(Ls) for r in range(2)]
    b = hb.Batch(specs, dtype=dtype)
    lib, st = hsg.lib(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    n, parts = len(specs), lib.hsg_batch_parts(max(Ls))
    assert parts == (1 if max(Ls) <= 48 else -(-max(Ls) ** 3 // 2 // 8192))
    E, spins = b.E.clone(), b.spins.clone()
    scratch = torch.full((15 * n * parts,), float("nan"), dtype=torch.float64, device="cuda")
    P = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    hsg.check(lib.hsg_batch_init_parts(ctypes.byref(b._d), max(Ls), P(scratch), st))
    assert torch.equal(b.spins, spins)
    # at most L^3 additions of terms below 10 in magnitude in either order, mean error far less
    assert torch.allclose(b.E, E, rtol=1e-12, atol=1e-9)
    pairs = [(2 * g, 2 * g + 1) for g in range(len(Ls))] + [(0, 0)]
    out = torch.empty((len(pairs), 15), dtype=torch.float64, device="cuda")
    pd = torch.tensor(pairs, dtype=torch.int32, device="cuda")
    hsg.check(lib.hsg_batch_overlap_parts(ctypes.byref(b._d), P(pd), len(pairs), max(Ls),
                                          P(scratch), P(out), st))
    assert torch.allclose(out, b.overlap(pairs), rtol=0, atol=1e-13)
