"""Half-sweeps by pieces of 16 sites: which batches take them, and the comparisons of
test_gpu_pieces.py with them wherever they can be taken (small batches with ragged rows
have a thread per pair of sites by themselves)."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S
from tests import test_gpu_pieces as P

NONE, FEW, ALL = 0, 1, 2


@pytest.mark.parametrize("dim,min_L,ragged,sites,want", [
    (2, 14, True, 1 << 30, NONE), (3, 4, False, 64, NONE),
    (2, 16, False, 256, ALL), (3, 16, False, 4096, ALL), (3, 64, False, 1 << 18, ALL),
    (2, 18, True, 324, FEW), (2, 200, True, (1 << 18) - 1, FEW), (2, 200, True, 1 << 18, ALL),
    (3, 26, True, 26 ** 3, FEW), (3, 50, True, (1 << 19) - 1, FEW), (3, 50, True, 1 << 19, ALL)])
def test_which_batches(dim, min_L, ragged, sites, want):
    f = S.lib()["_ZN3smc9piece_useEiibl"]
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_int, C.c_bool, C.c_int64]
    assert f(dim, min_L, ragged, sites) == want


@pytest.mark.gpu
@pytest.mark.parametrize("pieces", ["1", None])
@pytest.mark.parametrize("model", [S.ISING, S.EA])
@pytest.mark.parametrize("L", [16, 18, 20, 24, 30, 34, 46, 48, 100, 130, 200, 262])
def test_2d_rows(monkeypatch, model, L, pieces):
    if pieces:
        monkeypatch.setenv("SPINMC_PIECES", pieces)
    P.test_pieces_against_oracle(monkeypatch, model, 2, L, "0")


@pytest.mark.gpu
@pytest.mark.parametrize("pieces", ["1", None])
@pytest.mark.parametrize("dim", [2, 3])
def test_uneven_batches(monkeypatch, dim, pieces):
    if pieces:
        monkeypatch.setenv("SPINMC_PIECES", pieces)
    P.test_pieces_uneven_odd_offsets(dim)
