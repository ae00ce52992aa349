"""smc_autotune of 2D sweeps that hold a whole lattice: the workgroup that a call
takes untuned is one of the candidates, what is kept is kept for the replica
count it was measured with, and batches that hold no whole lattice are left alone."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S
from tests import refrun
from tests.test_launch_limits import BandShape, _shape

DEV = "cuda"


def _whole(L, n_rep, ea, limit):
    f = S.lib()["_ZN3smc13bands2d_wholeEiibiiPNS_9BandShapeE"]
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_int, C.c_bool, C.c_int, C.c_int, C.c_void_p]
    sh = BandShape()
    assert f(L, n_rep, ea, 16, limit, C.byref(sh))
    return sh


@pytest.mark.parametrize("L", range(16, 257, 16))
@pytest.mark.parametrize("ea", [False, True])
def test_the_untuned_workgroup_is_a_candidate(L, ea):
    n_rep = 1024  # whole lattices whatever the edge
    own = _shape(L, n_rep, ea, 16)
    assert own.whole
    threads = [_whole(L, n_rep, ea, limit).threads for limit in (64, 128, 256, 512, 1024)]
    assert threads[-1] == own.threads and threads == sorted(threads)
    assert all(t <= limit for t, limit in zip(threads, (64, 128, 256, 512, 1024)))


def _lines(path):
    return [l.split() for l in path.read_text().splitlines() if not l.startswith("#")]


@pytest.mark.gpu
def test_kept_by_replica_count_and_measured_again(tmp_path):
    path = tmp_path / "tune.txt"
    for n_rep in (300, 700):
        S.autotune(S.Batch(S.EA, 2, 256, n_rep, 3), str(path))
    mine = [l for l in _lines(path) if l[1:4] == ["u2d", "256", "1"]]
    assert sorted(int(l[4]) for l in mine) == [300, 700]
    assert all(int(l[5]) in (64, 128, 256, 512, 1024) for l in mine)
    # a line of any replica count holds a size that was not compared with the default
    path.write_text(f"{mine[0][0]} u2d 240 0 0 64 0 0\n")
    S.autotune(S.Batch(S.ISING, 2, 240, 400, 3), str(path))
    assert [l[4] for l in _lines(path) if l[1:4] == ["u2d", "240", "0"]] == ["400"]


@pytest.mark.gpu
def test_uneven_batches_have_nothing_to_tune(tmp_path):
    path = tmp_path / "tune.txt"
    inst = refrun.uneven_table(2, [208, 224], 4)
    S.autotune(S.Batch(S.EA, 2, 0, len(inst), 3, inst=inst), str(path))
    assert not path.exists()


@pytest.mark.gpu
@pytest.mark.parametrize("L,n_rep", [(128, 300), (192, 260), (256, 257)])
def test_tuned_results(L, n_rep, tmp_path):
    b = S.Batch(S.EA, 2, L, n_rep, 5)

    def run():
        spins = torch.zeros(n_rep * L * L, dtype=torch.int8, device=DEV)
        coup = torch.zeros(b.coup_len(), dtype=torch.int8, device=DEV)
        S.spin_init(b, spins, coup)
        dE = torch.zeros(n_rep, dtype=torch.int64, device=DEV)
        S.metropolis_sweep(b, spins, np.linspace(0.2, 0.9, n_rep), 1, 18, couplings=coup, dE_accum=dE)
        return spins.cpu(), dE.cpu()

    before = run()
    S.autotune(b, str(tmp_path / "tune.txt"))
    after = run()
    assert torch.equal(before[0], after[0]) and torch.equal(before[1], after[1])
