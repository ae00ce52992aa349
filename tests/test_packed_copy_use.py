"""Which calls run on the packed copy of 3D lattices: not the short ones on small
lattices, which are bound by their launches."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S


def _packed(model, L, n_rep, n):
    f = S.lib()["_ZN3smc11use_pairs3dEPK8smc_descl"]
    f.restype, f.argtypes = C.c_bool, [C.POINTER(S.Desc), C.c_int64]
    return f(C.byref(S.Batch(model, 3, L, n_rep, 1).desc(1 << 62, 1 << 62)), n)


@pytest.mark.parametrize("model,L,n_rep,n,packed", [
    (S.ISING, 48, 1, 3, False), (S.ISING, 48, 1, 7, False), (S.ISING, 48, 1, 8, True),
    (S.EA, 64, 5, 3, False), (S.EA, 64, 6, 3, True),   # 3.9e6 and 4.7e6 updates
    (S.EA, 50, 4, 2, False), (S.EA, 50, 5, 2, True), (S.EA, 64, 64, 2, False),
    (S.EA, 256, 1, 3, True), (S.ISING, 512, 1, 5, False), (S.ISING, 512, 1, 6, True), (S.ISING, 1024, 1, 100, False),
    (S.EA, 1024, 1, 3, True), (S.ISING, 14, 1000, 100, False)])
def test_which_calls(monkeypatch, model, L, n_rep, n, packed):
    assert _packed(model, L, n_rep, n) == packed
    monkeypatch.setenv("SPINMC_PAIRS3D", "0")
    assert not _packed(model, L, n_rep, n)
    monkeypatch.setenv("SPINMC_PAIRS3D", "1")
    assert _packed(model, L, n_rep, n) == (L >= 16)
