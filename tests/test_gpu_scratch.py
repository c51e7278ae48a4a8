"""The second spin array of a lattice's work buffer: whatever it holds before a call, the results
are the same."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# a phase per launch, one and two phases per launch with and without a Monte Carlo pass, fused
# passes
@pytest.mark.parametrize("L,dtype", [(64, "f32"), (64, "f64"), (98, "f32"), (128, "f64"),
                                     (150, "f32"), (256, "f32")])
def test_contents_of_the_second_array_do_not_matter(L, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as hsg
    dt = torch.float32 if dtype == "f32" else torch.float64
    lats = [hsg.Lattice(L, dt, seed=3) for _ in range(2)]
    n_bytes = lats[0].spins.numel() * lats[0].spins.element_size()
    assert lats[0].work.numel() > n_bytes  # there is one
    lats[0].work.zero_()
    sets = [None, 0, hsg.HSG_SNAKE | hsg.HSG_PHASE_LAUNCH, hsg.HSG_SNAKE | hsg.HSG_PHASE_MC]
    if hsg.fused_supported(L):
        sets.append(hsg.HSG_FUSED)
    for flags in sets:
        for k, n_or, hb in ((4, 1, False), (1, 2, True), (0, 3, False)):
            out = []
            for i, lat in enumerate(lats):
                def mess():
                    if i:
                        lat.work[-n_bytes:].fill_(255)  # NaN as binary32 and binary64
                mess()
                lat.sweep(T=0.5, k=k, n_or=n_or, renorm_every=2, n_sweeps=3, heat_bath=hb,
                          flags=flags)
                res = [lat.spins.clone(), lat.E.clone()]
                for f in (lat.energy, lambda: lat.energy(True), lambda: lat.overlap(lats[0]),
                          lambda: lat.overlap_fourier(lats[0])):
                    mess()
                    res.append(torch.as_tensor(f()).clone())
                out.append(res)
            for a, b in zip(*out):
                assert torch.equal(a, b), (flags, k, n_or, hb)
