"""The 2D bands (several sweeps per launch) at the shapes where they can go
wrong: halos that reach round the lattice, a short last band, row starts and
ends inside pieces, one piece per thread and several, an odd number of sweeps
over an even number of launches, whole lattices in LDS, edges below 16."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W
from tests import refrun

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).to("cuda")


# (edge, rows per band, sweeps per launch, sweeps); rows = edge: the whole lattice
SHAPES = [(4, 4, 5, 5), (6, 6, 4, 9), (14, 14, 3, 3), (18, 2, 1, 2), (18, 4, 4, 7), (20, 6, 2, 4), (24, 10, 2, 5),
          (30, 30, 4, 6), (32, 12, 3, 6), (46, 8, 2, 5), (48, 16, 2, 4), (100, 12, 3, 7), (130, 64, 6, 12),
          (200, 32, 4, 10), (208, 48, 2, 4), (390, 390, 2, 3), (1022, 24, 2, 3), (1008, 16, 4, 8)]


@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("L,rows,per,n", SHAPES)
def test_bands_against_oracle(monkeypatch, model, L, rows, per, n):
    import torch

    monkeypatch.setenv("SPINMC_SWEEP_LDS2D", "0")
    monkeypatch.setenv("SPINMC_BANDS2D", "1")
    monkeypatch.setenv("SPINMC_BANDS2D_ROWS", str(rows))
    monkeypatch.setenv("SPINMC_BANDS2D_SWEEPS", str(per))
    n_rep, seed = (3, W.seed_for(300 + L)) if L < 500 else (1, W.seed_for(300 + L))
    betas = [0.35, 0.0, 1.1][:n_rep]
    b = S.Batch(model, 2, L, n_rep, seed, rep_per_sample=2)
    ref_s, ref_c = refrun.init_uniform(model, 2, L, n_rep, seed, 2)
    spins = _dev(ref_s)
    coup = None if ref_c is None else _dev(ref_c)
    dE = torch.full((n_rep,), 7, dtype=torch.int64, device="cuda")
    S.metropolis_sweep(b, spins, betas, 5, n, couplings=coup, dE_accum=dE)
    ref_dE = refrun.sweep_uniform(model, 2, L, ref_s, ref_c, betas, seed, 5, n, 2) + 7
    assert np.array_equal(spins.cpu().numpy().reshape(ref_s.shape), ref_s)
    assert np.array_equal(dE.cpu().numpy(), ref_dE)


# (edge, rows and 16-site pieces per tile, sweeps per launch, sweeps): halo pieces that
# repeat own ones, rows that wrap under cut columns, short last tiles
TILES = [(16, 16, 1, 5, 5), (16, 4, 1, 2, 4), (32, 8, 1, 4, 8), (32, 32, 1, 8, 16), (48, 16, 2, 3, 6), (64, 20, 3, 8, 16),
         (96, 40, 4, 6, 12), (112, 112, 2, 4, 8), (128, 2, 1, 8, 16), (208, 48, 5, 2, 4), (512, 128, 8, 2, 4)]


@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("L,rows,words,per,n", TILES)
def test_tiles_against_oracle(monkeypatch, model, L, rows, words, per, n):
    monkeypatch.setenv("SPINMC_BANDS2D_WORDS", str(words))
    test_bands_against_oracle(monkeypatch, model, L, rows, per, n)


@pytest.mark.parametrize("L,n_rep,n", [(200, 16, 40), (512, 2, 41), (1000, 3, 9)])
def test_bands_chosen_shape_equals_half_sweeps(monkeypatch, L, n_rep, n):
    """The shape the library chooses against the half-sweep launches, over enough
    updates for exact (tail) decisions, at unaligned spins and couplings."""
    import torch

    outs = []
    for way in ("1", "0"):
        monkeypatch.setenv("SPINMC_BANDS2D", way)
        b = S.Batch(S.EA, 2, L, n_rep, W.seed_for(301))
        spins = torch.zeros(b.spins_shape()[0] + 3, dtype=torch.int8, device="cuda")[3:]
        coup = torch.zeros(b.coup_len() + 1, dtype=torch.int8, device="cuda")[1:]
        S.spin_init(b, spins, coup)
        dE = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
        S.metropolis_sweep(b, spins, [0.8] * n_rep, 3, n, couplings=coup, dE_accum=dE)
        outs.append((spins.cpu().numpy(), dE.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
