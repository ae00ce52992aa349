"""The entry points that take inverse temperatures accept a pointer to doubles
and nothing else of that place in the argument list."""
import ctypes as C

import pytest

import paper_1101_1427_amd as S

N = 2


def _calls():
    """name -> call with beta as its only open argument, on a batch of which nothing is launched."""
    d = S.Batch(S.ISING, 2, 64, N, 1).desc(N * 64 * 64, 0)
    dm = S.Batch(S.ISING, 2, 64, 32, 1).desc(32 * 64 * 64, 0)
    dh = S.Batch(S.HEISENBERG, 2, 64, N, 1).desc(N * 64 * 64 * 3, 0)
    p, L, D = C.c_void_p(4096), S.lib(), C.byref(d)
    name = C.c_char_p()
    return {
        "metropolis": lambda b: L.smc_metropolis_sweep(D, p, None, b, 0, 0, None, None),
        "msc": lambda b: L.smc_msc_sweep(C.byref(dm), p, None, b, 0, 0, 32, None, None),
        "dcb": lambda b: L.smc_dcb_sweep(D, p, None, b, 0, 0, 32, 1, 0, None, None, None),
        "heis_dcb": lambda b: L.smc_heis_dcb_sweep(C.byref(dh), p, b, 0, 0, 32, 1, S.HEIS_FAST, 0, 0.0, None, None),
        "dcb_plan": lambda b: L.smc_dcb_plan(D, b, 32, C.byref(name)),
    }


@pytest.mark.parametrize("call", sorted(_calls()))
def test_only_doubles(call):
    run = _calls()[call]
    assert run((C.c_double * 32)(*([0.5] * 32))) == S.OK
    assert run(None) == S.EINVAL
    for other in ((C.c_float * 32)(*([0.5] * 32)), C.byref(C.c_float(0.5)), 4096, C.c_void_p(4096), b"0.5"):
        with pytest.raises(C.ArgumentError):
            run(other)


def test_forms_of_beta():
    """A number, a list, and arrays of any kind reach the library as the same doubles."""
    import numpy as np

    b = S.Batch(S.ISING, 2, 128, 3, 1)
    fixed = np.array([0.4, 0.5, 0.0])
    fixed.setflags(write=False)
    for beta in ([0.4, 0.5, 0.0], (0.4, 0.5, 0.0), fixed, np.array([0.4, 0.5, 0.0]), np.array([[0.4, 9], [0.5, 9], [0, 9]])[:, 0]):
        assert S.dcb_plan(b, beta, 64) == "k_dcb2d"  # (a replica at beta = 0)
        assert S.dcb_plan(b, np.asarray(beta) + 0.1, 64) == "k_dcb2d_packed"
    assert S.dcb_plan(b, 0.4, 64) == S.dcb_plan(S.Batch(S.ISING, 2, 128, 1, 1), [0.4], 64) == "k_dcb2d_packed"
    with pytest.raises(S.SpinMCError):
        S.dcb_plan(S.Batch(S.ISING, 2, 128, 0, 1), [], 64)
