"""Which calls on the edges that both serve run on 2D tiles and which on the one-pass
kernel (a launch per sweep, against several sweeps in an even number of launches)."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S


def _tiles(L, n_rep, n, tempering=False):
    f = S.lib()["_ZN3smc22bands_before_lattice2dEPK8smc_descib"]
    f.restype, f.argtypes = C.c_bool, [C.POINTER(S.Desc), C.c_int32, C.c_bool]
    return f(C.byref(S.Batch(S.ISING, 2, L, n_rep, 1).desc(1 << 62, 0)), n, tempering)


@pytest.mark.parametrize("L,n_rep,least", [(1024, 1, 1), (1024, 8, 1), (2048, 2, 1), (1024, 9, 2), (2048, 3, 3),
                                           (1024, 16, 2), (2048, 4, 3), (1024, 17, 3), (2048, 5, 4), (1024, 24, 3),
                                           (1024, 25, 6), (1024, 32, 6), (2048, 8, 4), (4096, 1, 8), (4096, 2, 12)])
def test_the_fewest_sweeps(L, n_rep, least):
    assert _tiles(L, n_rep, least) and (least == 1 or not _tiles(L, n_rep, least - 1))
    assert _tiles(L, n_rep, 8 if L > 2048 else 1, True)


@pytest.mark.parametrize("L,n_rep", [(1024, 33), (2048, 9), (4096, 3), (8192, 1)])
def test_too_many_sites(L, n_rep):
    assert not _tiles(L, n_rep, 100) and not _tiles(L, n_rep, 100, True)


@pytest.mark.gpu
@pytest.mark.parametrize("L,n_rep,n,launches", [(1024, 32, 2, 2), (1024, 32, 5, 5), (2048, 4, 2, 2), (4096, 2, 10, 10),
                                                (1024, 32, 6, None), (2048, 4, 3, None), (4096, 2, 12, None)])
def test_launches_and_results(monkeypatch, L, n_rep, n, launches):
    """One launch per sweep on the one-pass kernel, fewer on the tiles; the same result."""
    b = S.Batch(S.ISING, 2, L, n_rep, 4)
    spins = torch.zeros(n_rep * L * L, dtype=torch.int8, device="cuda")
    S.spin_init(b, spins)
    other, beta = spins.clone(), np.linspace(0.3, 0.5, n_rep)
    S.kernel_timing_enable(True)
    S.metropolis_sweep(b, spins, beta, 0, n)
    torch.cuda.synchronize()
    got = S.kernel_timing_read()[1]
    S.kernel_timing_enable(False)
    assert got == launches if launches else got < n
    monkeypatch.setenv("SPINMC_BANDS2D", "1" if launches else "0")  # (the other one)
    S.metropolis_sweep(b, other, beta, 0, n)
    assert torch.equal(spins, other)
