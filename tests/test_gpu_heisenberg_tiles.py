"""The one-pass Heisenberg kernel on edges that are no multiple of its tiles,
against the half-sweep kernel (the same float32 arithmetic: bit for bit)."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W

pytestmark = pytest.mark.gpu


# partial tiles of one pair to 30 columns, segments longer and shorter than the
# edge and ones that do not divide it, a renormalisation, several replicas
@pytest.mark.parametrize("L,n_rep,n,planes", [(32, 2, 3, 2), (34, 8, 5, 0), (34, 7, 2, 24), (46, 3, 3, 3), (62, 2, 4, 8),
                                              (64, 1, 3, 3), (66, 1, 3, 32), (100, 1, 17, 0), (130, 1, 2, 16)])
def test_tiles_equal_half_sweeps(monkeypatch, L, n_rep, n, planes):
    import torch

    b = S.Batch(S.HEISENBERG, 3, L, n_rep, W.seed_for(600), renorm_every=16)
    assert S.sweep_plan(b)[1] == "k_heis3d_tiled" or n_rep * L ** 3 < 1 << 18
    out = []
    for way in ("1", "0"):
        monkeypatch.setenv("SPINMC_HEIS3D", way)
        if planes:
            monkeypatch.setenv("SPINMC_HEIS_PLANES", str(planes))
        spins = torch.zeros(3 * n_rep * L ** 3, dtype=torch.float32, device="cuda")
        S.spin_init(b, spins)
        acc = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
        S.metropolis_sweep(b, spins, np.linspace(0.4, 1.2, n_rep), 14, n, dE_accum=acc)
        out.append((spins.cpu().numpy(), acc.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
