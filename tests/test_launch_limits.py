"""Batches of a great many replicas: the launches of every path that a batch is
sent to stay below 2^32 work-items (launch_check.hpp), so that no batch is
refused that a path with fewer threads per replica would take."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S
from oracle import oracle as O


class BandShape(C.Structure):
    _fields_ = [("rows", C.c_int), ("words", C.c_int), ("sweeps", C.c_int), ("threads", C.c_int), ("whole", C.c_bool),
                ("ns_per_sweep", C.c_double)]


def _shape(L, n_rep, ea, n_sweeps, even=True):
    f = S.lib()["_ZN3smc13bands2d_shapeEiibibPNS_9BandShapeE"]
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_int, C.c_bool, C.c_int, C.c_bool, C.c_void_p]
    sh = BandShape()
    return sh if f(L, n_rep, ea, n_sweeps, even, C.byref(sh)) else None


@pytest.mark.parametrize("L", [16, 48, 96, 112, 128, 192, 256, 100, 514])
@pytest.mark.parametrize("n_sweeps", [1, 20])
def test_tiles_of_many_lattices(L, n_sweeps):
    """A shape is offered only where its launch is one; a lattice of up to 128^2 that is held as a
    whole always gets one, with fewer threads (64 of them serve 2^26 - 1 lattices)."""
    for n_rep in (1, 1 << 20, (1 << 22) - 1, 1 << 22, 7456541, (1 << 24) + 1, (1 << 26) - 1):
        sh = _shape(L, n_rep, False, n_sweeps)
        if sh is None:
            assert L > 128 or n_rep > (1 << 26) - 1, (L, n_rep)
            continue
        tiles = 1 if sh.whole else -(-L // sh.rows) * (-(-(L // 16) // sh.words) if L % 16 == 0 else 1)
        assert sh.threads >= 64 and sh.threads % 64 == 0 and n_rep * tiles * sh.threads < 1 << 32, (L, n_rep, sh.threads)


def test_many_lattices_do_not_divide_by_zero():
    """The parts of all rows, 16 of each of 2^28 lattices, are a multiple of 2^32; no shape serves the call
    (64 threads of each lattice are more than a launch has)."""
    assert _shape(256, 1 << 28, False, 10) is None


@pytest.mark.gpu
def test_sweep_of_2_22_lattices():
    """2^22 Ising lattices of 128^2 (69 GB), a thread per word of each: as many work-items as no launch has."""
    L, n, seed, beta = 128, 1 << 22, 7, 0.44
    b = S.Batch(S.ISING, 2, L, n, seed)
    spins = torch.ones(n * L * L, dtype=torch.int8, device="cuda")
    S.metropolis_sweep(b, spins, np.full(n, beta), 0, 1)
    for r in (0, 1, n // 2 + 3, n - 1):
        ref = np.ones(L * L, np.int8)
        O.run(2, L, None, ref, beta, seed, r, 0, 1)
        assert np.array_equal(spins[r * L * L:(r + 1) * L * L].cpu().numpy(), ref), r


@pytest.mark.gpu
def test_packed_copy_of_2_36_sites():
    """3D Ising of 2^36 and more sites in all, for which packing takes as many work-items as no launch has."""
    L, seed, beta = 64, 8, 0.22
    n = (1 << 36) // L ** 3 + 1
    assert L ** 3 // 16 % 256 == 0 and L ** 3 // 16 * n >= 1 << 32
    b = S.Batch(S.ISING, 3, L, n, seed)
    spins = torch.ones(n * L ** 3, dtype=torch.int8, device="cuda")
    S.metropolis_sweep(b, spins, np.full(n, beta), 0, 3)
    for r in (0, n - 1):
        ref = np.ones(L ** 3, np.int8)
        O.run(3, L, None, ref, beta, seed, r, 0, 3)
        assert np.array_equal(spins[r * L ** 3:(r + 1) * L ** 3].cpu().numpy(), ref), r


@pytest.mark.gpu
def test_tempering_of_2_23_bins(monkeypatch):
    """2^23 lattices of 112^2 (105 GB), each a bin of its own, in chains of two."""
    monkeypatch.setenv("SPINMC_BANDS2D", "0")  # (tiles otherwise)
    L, n, seed, betas = 112, 1 << 23, 9, [0.42, 0.44]
    b = S.Batch(S.ISING, 2, L, n, seed)
    spins = torch.ones(n * L * L, dtype=torch.int8, device="cuda")
    slots = torch.arange(n, dtype=torch.int32, device="cuda") % 2
    E = torch.full((n,), -2.0 * L * L, dtype=torch.float64, device="cuda")
    S.pt_sweep_swap(b, n // 2, 2, betas, spins, slots, E, 0, 1)
    s, e = slots.cpu().numpy().reshape(-1, 2), E.cpu().numpy()
    assert np.array_equal(np.sort(s, axis=1), np.broadcast_to([0, 1], s.shape))
    for r in (0, 1, n // 2, n - 2, n - 1):
        ref = np.ones(L * L, np.int8)
        O.run(2, L, None, ref, betas[r % 2], seed, r, 0, 1)
        assert np.array_equal(spins[r * L * L:(r + 1) * L * L].cpu().numpy(), ref), r
        assert e[r] == O.energy(2, L, None, ref)
