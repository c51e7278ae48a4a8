"""Every binary32 Metropolis trial point has the oracle's bits.

Without couplings every trial is accepted, so a sweep of one hit leaves the trial points as the
spins.  Two sweeps at L = 512 draw 2.7e8 of them: all 2^22 arguments 1 - z^2 of the square root
(counted), and each of the 2^23 azimuths 32 times on average (one is missing with probability
2^23 e^-32 = 1e-7)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_points_of_every_argument():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1006_2566_amd as hsg
    L, seed = 512, 77
    N = L ** 3
    lat = hsg.Lattice(L, torch.float32, seed=seed, init=None)
    lat.load(torch.full((3, N), 0.5, device="cuda"), torch.zeros((3, N), device="cuda"))
    want, J = np.full((3, N), 0.5, dtype=np.float32), np.zeros((3, N), dtype=np.float32)
    seen = torch.zeros(2 ** 22, dtype=torch.bool, device="cuda")
    for sweep in range(2):
        lat.sweep(T=1.0, k=1, n_or=0, flags=0)
        got = lat.export()[0]
        z = (got[2].abs() * 2.0 ** 23).long()  # odd, below 2^23
        assert bool((z & 1).all())
        seen[z >> 1] = True
        del z
        r = oracle.sweep(L, seed, want, J, T=1.0, k=1, n_or=0, n_sweeps=1, sweep0=sweep)
        assert r["n_accepted"] == N
        for a in range(3):
            assert np.array_equal(got[a].cpu().numpy(), want[a]), (sweep, a)
        print(f"sweep {sweep}: {int(seen.sum())} of {2 ** 22} arguments", flush=True)
    assert bool(seen.all())
