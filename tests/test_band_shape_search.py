"""The search for the shape of 2D tiles: it chooses what weighing every shape would
choose, in a fraction of the time that a short call takes on the chip."""
import os
import time

import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

from tests.test_launch_limits import BandShape, _shape  # noqa: F401

NAMES = ("SPINMC_BANDS2D_ROWS", "SPINMC_BANDS2D_SWEEPS", "SPINMC_BANDS2D_WORDS")


def _forced(L, n_rep, ea, n, even, rows, words, sweeps):
    """The estimate of one shape, or None if it does not serve the call."""
    for name, v in zip(NAMES, (rows, sweeps, words)):
        os.environ[name] = str(v)
    try:
        return _shape(L, n_rep, ea, n, even)
    finally:
        for name in NAMES:
            del os.environ[name]


def _weigh_all(L, n_rep, ea, n, even):
    """Every shape that the search may choose, in its order of preference."""
    all_words = L // 16 if L % 16 == 0 else 0
    best = None

    def offer(rows, words, sweeps):
        nonlocal best
        sh = _forced(L, n_rep, ea, n, even, min(rows, L), words, sweeps)
        if sh is not None and (best is None or sh.ns_per_sweep < best.ns_per_sweep):
            best = sh

    offer(L, all_words, min(n, 256))
    for sweeps in (1, 2, 3, 4, 5, 6, 8):
        if sweeps > ((n + 1) // 2 if even else n):
            continue
        for parts in range(1, max(all_words, 1) + 1):
            if all_words and all_words % parts:
                continue
            words = all_words // parts
            for per_cu in (1, 2, 4, 8):
                strips = 256 * per_cu // min(256 * 8, n_rep * parts)
                if strips > 0:
                    offer(max(2, -(-L // strips)), words, sweeps)
            for rows in (8, 16, 32, 64, 128):
                if rows < L and (not all_words or rows in (32, 128)):
                    offer(rows, words, sweeps)
    return best


@pytest.mark.parametrize("L", [16, 64, 96, 100, 128, 200, 256, 384, 500, 512, 720, 960, 1024, 1502, 2048, 3000, 3840, 4096])
def test_the_choice_is_that_of_weighing_every_shape(L):
    for n_rep in (1, 3, 64, 700):
        for n, even in ((1, True), (2, True), (3, False), (10, True), (100, True), (7, False)):
            ea = (n + n_rep) % 2 == 0
            got, want = _shape(L, n_rep, ea, n, even), _weigh_all(L, n_rep, ea, n, even)
            fields = [f for f, _ in BandShape._fields_]
            as_list = lambda sh: sh and [getattr(sh, f) for f in fields]
            assert as_list(got) == as_list(want), (L, n_rep, ea, n, even)


def _time(f, reps=400):
    best = float("inf")
    for _ in range(reps):
        t0 = time.perf_counter()
        f()
        best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("L", [384, 960, 1024, 2048])
def test_the_search_is_short(L):
    """Against a call that has one shape to weigh (weighing all takes three to four times as long, the binding's time included)."""
    _shape(L, 1, False, 10)
    assert _time(lambda: _shape(L, 1, False, 10)) < 2.0 * _time(lambda: _shape(L, 1, False, 1))
