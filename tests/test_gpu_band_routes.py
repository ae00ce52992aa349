"""Calls that the 2D bands took over from other kernels: the one-pass kernel on
the edges that both serve, small lattices against the half-sweeps, and
tempering of edges outside the bins, against the oracle."""
import numpy as np
import pytest

import paper_1101_1427_amd as S
import workloads as W
from oracle import oracle as O
from tests import refrun

pytestmark = pytest.mark.gpu


def _sweep(b, betas, t0, n):
    import torch

    spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
    coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda") if b.model == S.EA else None
    S.spin_init(b, spins, coup)
    dE = torch.zeros(b.n_rep, dtype=torch.int64, device="cuda")
    S.metropolis_sweep(b, spins, betas, t0, n, couplings=coup, dE_accum=dE)
    return spins.cpu().numpy(), dE.cpu().numpy()


@pytest.mark.parametrize("L,n_rep,n", [(1024, 1, 7), (1024, 5, 4), (2048, 2, 5), (1024, 2, 1)])
def test_bands_equal_one_pass_kernel(monkeypatch, L, n_rep, n):
    b = S.Batch(S.ISING, 2, L, n_rep, W.seed_for(500))
    betas = np.linspace(0.3, 0.5, n_rep)
    got = _sweep(b, betas, 3, n)
    monkeypatch.setenv("SPINMC_L2D_FUSE", "1")  # the one-pass kernel
    ref = _sweep(b, betas, 3, n)
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("model,L,n_rep,n", [(S.ISING, 16, 40, 300), (S.EA, 48, 9, 257), (S.EA, 112, 5, 20),
                                             (S.ISING, 128, 3, 1), (S.EA, 256, 9, 2)])
@pytest.mark.parametrize("threads", ["64", "512", ""])
def test_small_lattices_equal_half_sweeps(monkeypatch, model, L, n_rep, n, threads):
    b = S.Batch(model, 2, L, n_rep, W.seed_for(501))
    betas = np.linspace(0.2, 1.0, n_rep)
    if threads:
        monkeypatch.setenv("SPINMC_U2D_THREADS", threads)
    got = _sweep(b, betas, 250, n)
    monkeypatch.setenv("SPINMC_SWEEP_LDS2D", "0")
    ref = _sweep(b, betas, 250, n)
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


def test_sweeps_after_tempering_use_their_own_tables():
    """The same sweep before and after a tempering call of another batch on the
    same stream: both against the oracle (tables kept for a stream are not
    taken for ones that tempering has overwritten)."""
    import torch

    L, n_rep, seed = 16, 24, W.seed_for(512)
    betas = np.linspace(0.4, 1.4, n_rep)
    b = S.Batch(S.EA, 2, L, n_rep, seed, rep_per_sample=4)
    ref_s, ref_c = refrun.init_uniform(S.EA, 2, L, n_rep, seed, 4)
    spins, coup = (torch.from_numpy(a.reshape(-1).copy()).to("cuda") for a in (ref_s, ref_c))
    t = S.Batch(S.ISING, 2, 32, n_rep, seed)
    ts = torch.ones(t.spins_shape()[0], dtype=torch.int8, device="cuda")
    E = torch.full((n_rep,), -2.0 * 32 * 32, dtype=torch.float64, device="cuda")
    sot = torch.from_numpy(np.roll(np.arange(n_rep, dtype=np.int32), 5)).to("cuda")
    for k in range(2):
        dE = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
        S.metropolis_sweep(b, spins, betas, 9 * k, 9, couplings=coup, dE_accum=dE)
        ref_dE = refrun.sweep_uniform(S.EA, 2, L, ref_s, ref_c, betas, seed, 9 * k, 9, 4)
        assert np.array_equal(spins.cpu().numpy().reshape(ref_s.shape), ref_s), k
        assert np.array_equal(dE.cpu().numpy(), ref_dE), k
        S.pt_sweep_swap(t, 1, n_rep, W.geometric_ladder(1.8, 3.2, n_rep), ts, sot, E, k, 1)


@pytest.mark.parametrize("m,steps", [(1, 3), (3, 2)])
def test_large_tempering_equal_one_pass_kernel(monkeypatch, m, steps):
    import torch

    L, n_temps, n_chains, seed = 1024, 4, 2, W.seed_for(511)
    beta = W.geometric_ladder(2.0, 2.5, n_temps)
    b = S.Batch(S.ISING, 2, L, n_chains * n_temps, seed)
    perm = np.array([2, 0, 1, 3, 0, 0, 1, 2], np.int32)  # the second chain is left as it is
    outs = []
    for way in ("", "1"):
        if way:
            monkeypatch.setenv("SPINMC_L2D_FUSE", way)  # the one-pass kernel
        spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
        S.spin_init(b, spins)
        E = torch.zeros(b.n_rep, dtype=torch.float64, device="cuda")
        S.measure_energy_magnetisation(b, spins, E)
        sot = torch.from_numpy(perm.copy()).to("cuda")
        acc = torch.zeros(n_chains * (n_temps - 1), dtype=torch.int64, device="cuda")
        S.pt_sweep_swap(b, n_chains, n_temps, beta, spins, sot, E, 7, steps, swap_accepts=acc, sweeps_per_step=m)
        outs.append([t.cpu().numpy() for t in (spins, E, sot, acc)])
    for x, y in zip(*outs):
        assert np.array_equal(x, y)


# edges: below 16 and ragged (whole lattices), several sweeps per step in one and
# more launches, an odd number of launches in the call
@pytest.mark.parametrize("bands", ["1", "0"])
@pytest.mark.parametrize("model,L,n_temps,m,steps", [(S.EA, 10, 6, 1, 5), (S.EA, 50, 4, 3, 4), (S.ISING, 130, 3, 7, 3),
                                                     (S.ISING, 272, 3, 1, 3), (S.EA, 304, 2, 5, 3)])
def test_tempering_on_bands_against_oracle(monkeypatch, model, L, n_temps, m, steps, bands):
    import torch

    monkeypatch.setenv("SPINMC_BANDS2D", bands)
    n_chains, t0, seed = 3, 3, W.seed_for(510)
    beta = W.geometric_ladder(0.8, 2.0, n_temps) if model == S.EA else W.geometric_ladder(2.0, 3.0, n_temps)
    n_rep, N = n_chains * n_temps, L * L
    b = S.Batch(model, 2, L, n_rep, seed, rep_per_sample=n_temps)
    ref_s, ref_c = refrun.init_uniform(model, 2, L, n_rep, seed, n_temps)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).to("cuda")  # noqa: E731
    J = [None if ref_c is None else ref_c[q] for q in range(n_chains)]
    E0 = np.array([O.energy(2, L, J[r // n_temps], ref_s[r]) for r in range(n_rep)], np.int64)
    perm = np.stack([np.roll(np.arange(n_temps, dtype=np.int32), q) for q in range(n_chains)])
    perm[1, 0] = perm[1, 1]  # not a permutation: the chain stays as it is
    spins, E, sot = dev(ref_s), dev(E0.astype(np.float64)), dev(perm)
    acc = torch.zeros(n_chains * (n_temps - 1), dtype=torch.int64, device="cuda")
    S.pt_sweep_swap(b, n_chains, n_temps, beta, spins, sot, E, t0, steps,
                    couplings=None if ref_c is None else dev(ref_c), swap_accepts=acc, sweeps_per_step=m)
    for q in range(n_chains):
        rows = slice(q * n_temps, (q + 1) * n_temps)
        s, e, p, a = ref_s[rows].copy(), E0[rows].copy(), perm[q].copy(), np.zeros(n_temps - 1, np.uint64)
        if q != 1:
            O.pt_run(2, L, J[q], s, beta, p, e, seed, q, q * n_temps, t0, steps, a, sweeps_per_step=m)
        assert np.array_equal(spins.cpu().numpy().reshape(n_rep, N)[rows], s), q
        assert np.array_equal(E.cpu().numpy()[rows], e.astype(np.float64))
        assert np.array_equal(sot.cpu().numpy().reshape(n_chains, n_temps)[q], p)
        assert np.array_equal(acc.cpu().numpy().reshape(n_chains, -1)[q].astype(np.uint64), a)
