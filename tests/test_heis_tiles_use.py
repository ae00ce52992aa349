"""Which calls of uniform 3D Heisenberg batches sweep in one pass over tiles."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S
from tests import refrun  # noqa: F401


def _tiled(L, n_rep, n):
    f = S.lib()["_ZN3smc16use_heis3d_tiledEPK8smc_descl"]
    f.restype, f.argtypes = C.c_bool, [C.POINTER(S.Desc), C.c_int64]
    return f(C.byref(S.Batch(S.HEISENBERG, 3, L, n_rep, 1).desc(1 << 62, 0)), n)


@pytest.mark.parametrize("L,n_rep,n,want", [
    (34, 64, 1, False), (36, 64, 1, False), (38, 64, 1, False), (34, 64, 2, True), (38, 64, 3, False), (38, 64, 5, True),
    (34, 8, 3, True), (40, 64, 1, True),
    (66, 8, 1, True), (100, 1, 1, True), (32, 1, 1, True), (64, 1, 1, True), (34, 2, 5, False), (30, 64, 5, False)])
def test_which_calls(L, n_rep, n, want):
    assert _tiled(L, n_rep, n) == want


@pytest.mark.gpu
def test_one_sweep_equals_the_tiles(monkeypatch):
    """Two calls of one sweep (half-sweeps) and one of two (tiles) give the same spins and counts."""
    b = S.Batch(S.HEISENBERG, 3, 34, 7, 3, renorm_every=2)
    start = torch.zeros(b.spins_shape()[0], dtype=torch.float32, device="cuda")
    S.spin_init(b, start)
    beta, out = np.linspace(0.4, 0.9, 7), []
    for n in (1, 2):
        spins, acc = start.clone(), torch.zeros(7, dtype=torch.int64, device="cuda")
        for k in range(0, 2, n):
            S.metropolis_sweep(b, spins, beta, k, n, dE_accum=acc)
        out.append((spins.cpu(), acc.cpu()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
