"""The instance table of an uneven batch as the binding hands it over: a row
per replica, in any of the forms a caller may hold it in."""
import numpy as np
import pytest

import paper_1101_1427_amd as S

N = 4
ROWS = [(16, 0, 0, 0), (32, 1, 256, 512), (16, 2, 1280, 2560), (4, 3, 1536, 3072)]


def _table(inst, n_rep=N):
    d = S.Batch(S.EA, 2, 0, n_rep, 1, inst=inst).desc(1 << 20, 1 << 20)
    return [(d.inst[r].L, d.inst[r].sample, d.inst[r].spin_off, d.inst[r].coup_off) for r in range(n_rep)]


@pytest.mark.parametrize("rows", [0, 1, N - 1, N + 1])
def test_a_table_of_another_length_is_refused(rows):
    inst = (ROWS + ROWS)[:rows]
    for form in (inst, np.array(inst, np.int64).reshape(rows, 4)):
        with pytest.raises(ValueError):
            _table(form)


@pytest.mark.parametrize("inst", [[16, 0, 0, 0], [r[:3] for r in ROWS]], ids=["one dimension", "three columns"])
def test_a_table_of_another_form_is_refused(inst):
    with pytest.raises((ValueError, IndexError)):
        _table(inst)


def test_no_table_is_refused():
    with pytest.raises(TypeError):
        _table(None)


@pytest.mark.parametrize("form", [
    ROWS, tuple(ROWS), np.array(ROWS, np.int64), np.array(ROWS, np.int32), np.array(ROWS, np.float64),
    np.asfortranarray(np.array(ROWS)), np.array([r + (7,) for r in ROWS]), [r + (7,) * k for k, r in enumerate(ROWS)]],
    ids=["list", "tuple", "int64", "int32", "float64", "columns", "five columns", "rows of several lengths"])
def test_forms_of_a_table(form):
    assert _table(form) == ROWS


def test_one_replica():
    assert _table(ROWS[:1], 1) == ROWS[:1]
