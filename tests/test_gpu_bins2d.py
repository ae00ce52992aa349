"""Exchange rounds of 2D tempering bins at the start of the next launch: odd and even numbers of
steps and of temperatures, one step, per-chain ladders, a chain whose slots are no permutation."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W
from oracle import oracle as O
from tests import refrun

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).to("cuda")


@pytest.mark.parametrize("L,n_temps,per_chain,steps,m", [(16, 2, False, 1, 1), (16, 5, True, 2, 1), (32, 6, False, 7, 1),
                                                         (48, 3, True, 4, 2), (64, 16, False, 5, 1)])
def test_bins_exchange_against_oracle(monkeypatch, L, n_temps, per_chain, steps, m):
    import torch

    monkeypatch.setenv("SPINMC_BANDS2D", "0")
    n_chains, t0, seed = 3, 3, W.seed_for(740 + L)
    beta = W.geometric_ladder(0.6, 2.0, n_temps)
    betas = np.stack([beta * (1 + 0.05 * q) for q in range(n_chains)]) if per_chain else np.stack([beta] * n_chains)
    n_rep, N = n_chains * n_temps, L * L
    b = S.Batch(S.EA, 2, L, n_rep, seed, rep_per_sample=n_temps)
    ref_s, ref_c = refrun.init_uniform(S.EA, 2, L, n_rep, seed, n_temps)
    spins, coup = _dev(ref_s), _dev(ref_c)
    E0 = np.array([O.energy(2, L, ref_c[r // n_temps], ref_s[r]) for r in range(n_rep)], np.int64)
    E = torch.from_numpy(E0.astype(np.float64)).to("cuda")
    perm = np.stack([np.roll(np.arange(n_temps, dtype=np.int32), q) for q in range(n_chains)])
    perm[1, 0] = perm[1, 1]  # not a permutation: the chain stays as it is
    sot = _dev(perm)
    acc = torch.full((n_chains * (n_temps - 1),), 2, dtype=torch.int64, device="cuda")
    S.pt_sweep_swap(b, n_chains, n_temps, betas if per_chain else beta, spins, sot, E, t0, steps, couplings=coup,
                    swap_accepts=acc, beta_per_chain=per_chain, sweeps_per_step=m)
    for q in range(n_chains):
        rows = slice(q * n_temps, (q + 1) * n_temps)
        s, e, p = ref_s[rows].copy(), E0[rows].copy(), perm[q].copy()
        a = np.zeros(n_temps - 1, np.uint64)
        if q != 1:
            O.pt_run(2, L, ref_c[q], s, betas[q], p, e, seed, q, q * n_temps, t0, steps, a, sweeps_per_step=m)
        assert np.array_equal(spins.cpu().numpy().reshape(n_rep, N)[rows], s), q
        assert np.array_equal(E.cpu().numpy()[rows], e.astype(np.float64))
        assert np.array_equal(sot.cpu().numpy().reshape(n_chains, n_temps)[q], p)
        assert np.array_equal(acc.cpu().numpy().reshape(n_chains, -1)[q].astype(np.uint64), a + 2)
