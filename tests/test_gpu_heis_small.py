"""Small Heisenberg lattices on chip: the smallest and the largest edges, 2D and 3D, threads with one
to several pairs of sites, renormalisation inside a call; bit for bit the half-sweep launches."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,L,n_rep,n", [(2, 4, 3, 5), (2, 46, 2, 4), (2, 64, 2, 3), (2, 114, 2, 3), (3, 4, 65, 7),
                                           (3, 6, 3, 9), (3, 8, 2, 33), (3, 12, 3, 4), (3, 16, 2, 5), (3, 22, 3, 4)])
def test_small_equals_half_sweeps(monkeypatch, dim, L, n_rep, n):
    import torch

    outs = []
    for way in ("1", "0"):
        monkeypatch.setenv("SPINMC_HEIS_SMALL", way)
        b = S.Batch(S.HEISENBERG, dim, L, n_rep, W.seed_for(760 + L), renorm_every=4)
        spins = torch.zeros(b.spins_shape()[0], dtype=torch.float32, device="cuda")
        S.spin_init(b, spins)
        acc = torch.full((n_rep,), 5, dtype=torch.int64, device="cuda")
        S.metropolis_sweep(b, spins, np.linspace(0.0, 1.5, n_rep), 3, n, dE_accum=acc)
        outs.append((spins.cpu().numpy().view(np.uint32), acc.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
