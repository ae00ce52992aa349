"""Calls as they come on large lattices, against the kernels that stand in for the
route they take: the packed 3D copy above edge 250 (8 planes per thread from 2^25
sites on, and ragged edges up to the largest), 2D tiles above edge 2048 and ragged 2D
rows above 1022, workgroups of whole 2D lattices too small for their words; tempering on
ragged packed lattices and half-sweeps by pieces of ragged 3D rows, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1101_1427_amd as S
import workloads as W
from tests import test_gpu_pairs3d, test_gpu_pieces

pytestmark = pytest.mark.gpu


def _state(b):
    spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
    coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda") if b.model == S.EA else None
    S.spin_init(b, spins, coup)
    return spins, coup


def _same(monkeypatch, b, n, env, beta):
    """n sweeps by default and with env set, from the same state."""
    spins, coup = _state(b)
    other = spins.clone()
    dE = [torch.full((b.n_rep,), 5, dtype=torch.int64, device="cuda") for _ in range(2)]
    S.metropolis_sweep(b, spins, beta, 3, n, couplings=coup, dE_accum=dE[0])
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    S.metropolis_sweep(b, other, beta, 3, n, couplings=coup, dE_accum=dE[1])
    assert torch.equal(spins, other) and torch.equal(dE[0], dE[1])


@pytest.mark.parametrize("model,L,n_rep,n", [(S.EA, 256, 2, 3), (S.EA, 512, 1, 3), (S.ISING, 512, 2, 6), (S.ISING, 768, 1, 6),
                                             (S.EA, 1024, 1, 3), (S.ISING, 502, 1, 2), (S.EA, 622, 1, 3),
                                             (S.ISING, 1022, 1, 2)])
def test_packed_copy_equals_kernels_on_bytes(monkeypatch, model, L, n_rep, n):
    _same(monkeypatch, S.Batch(model, 3, L, n_rep, W.seed_for(730)), n, {"SPINMC_PAIRS3D": "0"},
          np.linspace(0.25, 0.6, n_rep))


@pytest.mark.parametrize("model,L,n_rep,n", [(S.ISING, 4096, 2, 8), (S.EA, 4096, 1, 9), (S.ISING, 3840, 1, 10),
                                             (S.ISING, 2998, 1, 9), (S.EA, 3002, 2, 6), (S.EA, 1502, 3, 7),
                                             (S.ISING, 9000, 1, 4)])
def test_tiles_equal_other_kernels(monkeypatch, model, L, n_rep, n):
    _same(monkeypatch, S.Batch(model, 2, L, n_rep, W.seed_for(731)), n, {"SPINMC_BANDS2D": "0"},
          np.linspace(0.3, 0.7, n_rep))


@pytest.mark.parametrize("threads", ["64", "128", "256", "512"])
@pytest.mark.parametrize("L", [144, 160, 192, 208, 224, 240, 256])
def test_small_workgroups_of_whole_lattices(monkeypatch, L, threads):
    _same(monkeypatch, S.Batch(S.EA, 2, L, 300, W.seed_for(732)), 5, {"SPINMC_U2D_THREADS": threads},
          np.linspace(0.2, 1.0, 300))


# edges just above and between multiples of 16; from 42 on a replica has 16 and more workgroups, whose energy
# changes go through slots
@pytest.mark.parametrize("L,n_temps,m", [(18, 5, 1), (20, 3, 2), (26, 3, 1), (32, 4, 1), (34, 4, 2), (42, 2, 3), (50, 3, 1), (48, 3, 2)])
def test_tempering_on_packed_lattices(monkeypatch, L, n_temps, m):
    monkeypatch.setenv("SPINMC_SMALL3D", "0")
    monkeypatch.setenv("SPINMC_PAIRS3D", "1")  # (so few updates in all stay on the caller's bytes)
    b = S.Batch(S.EA, 3, L, 3 * n_temps, 1, rep_per_sample=n_temps)
    assert S.pt_plan(b, 3, n_temps, W.geometric_ladder(0.8, 2.0, n_temps), 4, sweeps_per_step=m)[0] > 4 * (2 * m + 1)
    test_gpu_pairs3d.test_pairs_tempering_against_oracle(L, n_temps, m)


@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("L", [16, 18, 20, 22, 24, 30, 32, 34, 46, 48, 50])
def test_pieces_of_3d_rows(monkeypatch, model, L):
    for name in ("SPINMC_SMALL3D", "SPINMC_PAIRS3D"):
        monkeypatch.setenv(name, "0")
    monkeypatch.setenv("SPINMC_PIECES", "1")
    test_gpu_pieces.test_pieces_against_oracle(monkeypatch, model, 3, L, "0")

