"""3D half-sweeps on the packed copy at the edges where they can go wrong: row
borders inside a piece at every offset, a partial last piece, every wrap, 1 to 4
planes per thread, several replicas with shared samples, beta = 0, unaligned
arrays; and tempering on it."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W
from oracle import oracle as O
from tests import refrun

pytestmark = pytest.mark.gpu


def _dev(a, shift=0):
    import torch

    t = torch.zeros(a.size + shift, dtype=torch.int8, device="cuda")
    t[shift:] = torch.from_numpy(np.ascontiguousarray(a).reshape(-1))
    return t[shift:]


@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("L,planes", [(16, 1), (16, 4), (18, 1), (20, 1), (22, 1), (24, 1), (26, 1), (28, 1), (30, 1),
                                      (32, 2), (34, 1), (46, 1), (48, 1), (48, 2), (48, 4), (48, 8), (64, 1)])
def test_pairs_against_oracle(monkeypatch, model, L, planes):
    import torch

    monkeypatch.setenv("SPINMC_SMALL3D", "0")
    monkeypatch.setenv("SPINMC_PAIRS3D", "1")
    monkeypatch.setenv("SPINMC_PAIRS3D_PLANES", str(planes))
    n_rep, seed, n = 3, W.seed_for(700 + L), 3
    betas = [0.35, 0.0, 1.1]
    b = S.Batch(model, 3, L, n_rep, seed, rep_per_sample=2)
    ref_s, ref_c = refrun.init_uniform(model, 3, L, n_rep, seed, 2)
    spins = _dev(ref_s, 3)
    coup = None if ref_c is None else _dev(ref_c, 1)
    dE = torch.full((n_rep,), 11, dtype=torch.int64, device="cuda")
    S.metropolis_sweep(b, spins, betas, 5, n, couplings=coup, dE_accum=dE)
    ref_dE = refrun.sweep_uniform(model, 3, L, ref_s, ref_c, betas, seed, 5, n, 2) + 11
    assert np.array_equal(spins.cpu().numpy().reshape(ref_s.shape), ref_s)
    assert np.array_equal(dE.cpu().numpy(), ref_dE)


@pytest.mark.parametrize("model,L,n_rep,n", [(S.EA, 128, 2, 6), (S.ISING, 192, 1, 4), (S.EA, 102, 3, 8),
                                             (S.ISING, 250, 1, 3)])
def test_pairs_equal_kernels_on_bytes(monkeypatch, model, L, n_rep, n):
    """The chosen shapes on larger lattices (exact tail decisions among them)."""
    import torch

    outs = []
    for way in ("", "0"):
        if way:
            monkeypatch.setenv("SPINMC_PAIRS3D", way)
        b = S.Batch(model, 3, L, n_rep, W.seed_for(701))
        spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
        coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda") if model == S.EA else None
        S.spin_init(b, spins, coup)
        dE = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
        S.metropolis_sweep(b, spins, [0.6] * n_rep, 3, n, couplings=coup, dE_accum=dE)
        outs.append((spins.cpu().numpy(), dE.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("L,n_temps,m", [(18, 5, 1), (20, 3, 2), (32, 4, 1)])
def test_pairs_tempering_against_oracle(L, n_temps, m):
    import torch

    n_chains, steps, t0, seed = 3, 4, 3, W.seed_for(720 + L)
    beta = W.geometric_ladder(0.8, 2.0, n_temps)
    n_rep, N = n_chains * n_temps, L ** 3
    b = S.Batch(S.EA, 3, L, n_rep, seed, rep_per_sample=n_temps)
    ref_s, ref_c = refrun.init_uniform(S.EA, 3, L, n_rep, seed, n_temps)
    E0 = np.array([O.energy(3, L, ref_c[r // n_temps], ref_s[r]) for r in range(n_rep)], np.int64)
    perm = np.stack([np.roll(np.arange(n_temps, dtype=np.int32), q) for q in range(n_chains)])
    perm[1, 0] = perm[1, 1]  # not a permutation: the chain stays as it is
    spins, coup = _dev(ref_s), _dev(ref_c)
    E, sot = torch.from_numpy(E0.astype(np.float64)).to("cuda"), torch.from_numpy(perm.reshape(-1).copy()).to("cuda")
    acc = torch.zeros(n_chains * (n_temps - 1), dtype=torch.int64, device="cuda")
    S.pt_sweep_swap(b, n_chains, n_temps, beta, spins, sot, E, t0, steps, couplings=coup, swap_accepts=acc,
                    sweeps_per_step=m)
    for q in range(n_chains):
        rows = slice(q * n_temps, (q + 1) * n_temps)
        s, e, p, a = ref_s[rows].copy(), E0[rows].copy(), perm[q].copy(), np.zeros(n_temps - 1, np.uint64)
        if q != 1:
            O.pt_run(3, L, ref_c[q], s, beta, p, e, seed, q, q * n_temps, t0, steps, a, sweeps_per_step=m)
        assert np.array_equal(spins.cpu().numpy().reshape(n_rep, N)[rows], s), q
        assert np.array_equal(E.cpu().numpy()[rows], e.astype(np.float64))
        assert np.array_equal(sot.cpu().numpy().reshape(n_chains, n_temps)[q], p)
        assert np.array_equal(acc.cpu().numpy().reshape(n_chains, -1)[q].astype(np.uint64), a)
