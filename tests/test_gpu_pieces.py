"""The general path's 16-site pieces where they can go wrong: edges just above,
at and between multiples of 16 (row borders inside a piece, a partial last
piece), every neighbour wrap, beta = 0, several replicas, odd byte offsets and
shared draws; spins and energy changes bit-exact against the oracle."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W
from tests import refrun

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).to("cuda")


@pytest.mark.parametrize("bands", ["0", "1"])
@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("dim,L", [(2, 16), (2, 18), (2, 20), (2, 24), (2, 30), (2, 34), (2, 46), (2, 48), (2, 100),
                                   (2, 130), (2, 200), (2, 262), (3, 16), (3, 18), (3, 20), (3, 22), (3, 24), (3, 30),
                                   (3, 32), (3, 34), (3, 50)])
def test_pieces_against_oracle(monkeypatch, model, dim, L, bands):
    for name in ("SPINMC_SWEEP3D", "SPINMC_SWEEP_LDS2D"):
        monkeypatch.setenv(name, "0")
    monkeypatch.setenv("SPINMC_BANDS2D", bands)
    import torch

    n_rep, seed, n = 3, W.seed_for(200 + L), 3
    betas = [0.0, 0.35, 1.1]
    b = S.Batch(model, dim, L, n_rep, seed, rep_per_sample=2)
    ref_s, ref_c = refrun.init_uniform(model, dim, L, n_rep, seed, 2)
    spins = _dev(ref_s)
    coup = None if ref_c is None else _dev(ref_c)
    dE = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
    S.metropolis_sweep(b, spins, betas, 5, n, couplings=coup, dE_accum=dE)
    ref_dE = refrun.sweep_uniform(model, dim, L, ref_s, ref_c, betas, seed, 5, n, 2)
    assert np.array_equal(spins.cpu().numpy().reshape(ref_s.shape), ref_s)
    assert np.array_equal(dE.cpu().numpy(), ref_dE)


@pytest.mark.parametrize("dim", [2, 3])
def test_pieces_uneven_odd_offsets(dim):
    """An uneven batch at odd byte offsets (no alignment at all), the last replica ending at the buffer's end."""
    import torch

    from oracle import oracle as O

    seed, rows, so, co = W.seed_for(260), [], 1, 3
    edges = (18, 16, 50, 22) if dim == 2 else (18, 16, 24, 22)
    for k, L in enumerate(edges):
        rows.append((L, k, so, co))
        so += L ** dim + (5 if k < 3 else 0)
        co += dim * L ** dim + (1 if k < 3 else 0)
    inst = np.array(rows, np.int64)
    spins, coup = refrun.init_uneven(S.EA, dim, inst, seed)
    dev, cdev = _dev(spins), _dev(coup)
    dE = torch.zeros(len(rows), dtype=torch.int64, device="cuda")
    S.metropolis_sweep(S.Batch(S.EA, dim, 0, len(rows), seed, inst=inst), dev, [0.7] * 4, 0, 3, couplings=cdev,
                       dE_accum=dE)
    for r, (L, _, s0, c0) in enumerate(rows):
        N = L ** dim
        s = spins[s0:s0 + N].copy()
        d = O.run(dim, L, coup[c0:c0 + dim * N].copy(), s, 0.7, seed, r, 0, 3)
        spins[s0:s0 + N] = s
        assert int(dE[r]) == d
    assert np.array_equal(dev.cpu().numpy(), spins)  # the bytes between replicas too


def test_pieces_ties_and_shared_draws(monkeypatch):
    """2^23 updates meet the exact (tail) decision; multi-spin groups share their draws."""
    outs = []
    for way in ("1", "0"):
        import torch

        monkeypatch.setenv("SPINMC_PIECES", way)
        b = S.Batch(S.EA, 2, 90, 64, W.seed_for(261))
        spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
        coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda")
        S.spin_init(b, spins, coup)
        dE = torch.zeros(64, dtype=torch.int64, device="cuda")
        S.msc_sweep(b, spins, [0.4] * 32 + [0.9] * 32, 3, 16, couplings=coup, dE_accum=dE)
        outs.append((spins.cpu().numpy(), dE.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
