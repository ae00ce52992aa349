"""Energy changes at the line between adding to the caller's totals directly (fewer than
16 workgroups per replica, or at most 32 in all, or 256 over the launches) and slots: equal to the measured energies."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1101_1427_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,dim,L,n_rep", [
    (S.EA, 3, 40, 2), (S.EA, 3, 40, 3),        # 16 workgroups per replica: 32 and 48 in all
    (S.ISING, 3, 48, 1), (S.ISING, 3, 48, 2),  # 27: 27 and 54
    (S.ISING, 3, 64, 1), (S.ISING, 3, 64, 2),   # 64 and, over the two launches of a sweep, 256
    (S.EA, 2, 512, 1), (S.EA, 2, 1000, 1)])
@pytest.mark.parametrize("n", [1, 4])
def test_sums_equal_measured_energies(monkeypatch, model, dim, L, n_rep, n):
    for name in ("SPINMC_PAIRS3D", "SPINMC_BANDS2D"):
        monkeypatch.setenv(name, "0")
    b = S.Batch(model, dim, L, n_rep, 6)
    spins = torch.zeros(b.spins_shape()[0], dtype=torch.int8, device="cuda")
    coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda") if model == S.EA else None
    S.spin_init(b, spins, coup)
    E = [torch.zeros(n_rep, dtype=torch.float64, device="cuda") for _ in range(2)]
    dE = torch.full((n_rep,), 7, dtype=torch.int64, device="cuda")
    S.measure_energy_magnetisation(b, spins, E[0], couplings=coup)
    S.metropolis_sweep(b, spins, np.full(n_rep, 0.4), 2, n, couplings=coup, dE_accum=dE)
    S.measure_energy_magnetisation(b, spins, E[1], couplings=coup)
    assert torch.equal((E[1] - E[0]).to(torch.int64) + 7, dE) and bool((dE != 7).all())
