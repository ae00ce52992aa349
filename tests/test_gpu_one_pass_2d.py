"""The one-pass 2D Ising sweep and tempering on it, on the edges that calls leave to
the tiles by themselves: the oracle comparisons of the tests that name k_ising2d_split,
with the tiles switched off, and a check that the kernel is the one that runs."""
import pytest

torch = pytest.importorskip("torch")

import paper_1101_1427_amd as S
import workloads as W
from tests.test_gpu_gates import test_ising_1024_crop_2000_sweeps  # noqa: F401
from tests.test_gpu_parity import test_split_kernel_bit_exact  # noqa: F401
from tests.test_gpu_pt_split2d import (test_invalid_chain_is_left_unchanged,  # noqa: F401
                                       test_split_and_generic_paths_agree,
                                       test_split_tempering_one_sweep_per_step_two_chains,
                                       test_split_tempering_two_sweeps_per_step)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_tiles(monkeypatch):
    monkeypatch.setenv("SPINMC_BANDS2D", "0")


def _launches(call):
    S.kernel_timing_enable(True)
    call()
    torch.cuda.synchronize()
    n = S.kernel_timing_read()[1]
    S.kernel_timing_enable(False)
    return n


def test_every_sweep_is_a_launch(monkeypatch):
    """A launch per sweep is the one-pass kernel's; tiles make several sweeps in one, half-sweeps take two."""
    L, n_temps, m, steps = 1024, 4, 2, 3
    b = S.Batch(S.ISING, 2, L, n_temps, W.seed_for(96))
    spins = torch.zeros(n_temps * L * L, dtype=torch.int8, device="cuda")
    S.spin_init(b, spins)
    E = torch.zeros(n_temps, dtype=torch.float64, device="cuda")
    S.measure_energy_magnetisation(b, spins, E)
    sot = torch.arange(n_temps, dtype=torch.int32, device="cuda")
    sweeps = lambda: S.metropolis_sweep(b, spins, [0.4] * n_temps, 0, 8)  # noqa: E731
    temper = lambda: S.pt_sweep_swap(b, 1, n_temps, [0.3, 0.4, 0.45, 0.5], spins, sot, E, 0, steps,  # noqa: E731
                                     sweeps_per_step=m)
    assert _launches(sweeps) == 8 and _launches(temper) == steps * m
    monkeypatch.delenv("SPINMC_BANDS2D")
    assert _launches(sweeps) < 8 and _launches(temper) != steps * m
