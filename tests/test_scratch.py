"""The device memory that the library holds: one buffer per stream for the second
lattices and packed copies of all paths, and no copy that a path can do without
where it would take most of the free memory."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")  # (before the library: both then share one HIP runtime)

import paper_1101_1427_amd as S
from oracle import oracle as O

MiB = 1 << 20


def test_half_of_the_free_memory():
    f = S.lib()["_ZN3smc10spare_fitsEmmm"]
    f.restype, f.argtypes = C.c_bool, [C.c_size_t] * 3
    assert f(100, 0, 200) and not f(101, 0, 200)
    assert f(150, 100, 200) and not f(151, 100, 200)  # (what is held is given back first)
    assert f(100, 100, 0) and not f(101, 100, 0)


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.gpu
def test_one_buffer_for_the_copies_of_all_paths():
    stream = torch.cuda.Stream()  # (a stream has scratch of its own)
    calls = []
    for model, dim, L, n, sweeps, copy in ((S.ISING, 2, 8192, 2, 3, 2.0), (S.EA, 2, 1502, 60, 4, 1.0),
                                           (S.ISING, 3, 512, 1, 3, 1.0), (S.EA, 3, 200, 32, 4, 0.5),
                                           (S.HEISENBERG, 3, 96, 20, 2, 12.0)):
        b = S.Batch(model, dim, L, n, 3)
        spins = torch.zeros(b.spins_shape()[0], dtype=torch.float32 if model == S.HEISENBERG else torch.int8, device="cuda")
        coup = torch.zeros(b.coup_len(), dtype=torch.int8, device="cuda") if model == S.EA else None
        S.spin_init(b, spins, coup, stream=stream)
        calls.append((b, spins, coup, sweeps, int(n * L ** dim * copy)))
    for s in (torch.cuda.Stream(), stream):  # (the first time round loads the kernels)
        before = _free()
        for b, spins, coup, sweeps, _ in calls:
            S.metropolis_sweep(b, spins, np.full(b.n_rep, 0.4), 0, sweeps, couplings=coup, stream=s)
        held = before - _free()
    most = max(c[-1] for c in calls)
    assert most <= held <= most + 32 * MiB, (held / MiB, [c[-1] / MiB for c in calls])


@pytest.mark.gpu
def test_a_copy_of_most_of_the_free_memory_is_not_taken():
    L, n, seed, beta = 3000, 400, 4, 0.44  # 3.6 GB, whose sweeps take tiles and a second lattice
    stream = torch.cuda.Stream()
    b = S.Batch(S.ISING, 2, L, n, seed)
    spins = torch.ones(n * L * L, dtype=torch.int8, device="cuda")
    torch.cuda.empty_cache()
    filler = torch.empty(_free() - 6 * 1024 * MiB, dtype=torch.int8, device="cuda")
    before = _free()
    S.metropolis_sweep(b, spins, np.full(n, beta), 0, 2, stream=stream)
    assert before - _free() < 64 * MiB
    got = spins[(n - 1) * L * L:].cpu().numpy()
    del filler
    torch.cuda.empty_cache()
    before = _free()
    S.metropolis_sweep(b, spins, np.full(n, beta), 2, 2, stream=stream)
    assert before - _free() > n * L * L // 2  # (taken or not: 3.6 GB or next to nothing)
    ref = np.ones(L * L, np.int8)
    O.run(2, L, None, ref, beta, seed, n - 1, 0, 2)
    assert np.array_equal(got, ref)
    O.run(2, L, None, ref, beta, seed, n - 1, 2, 2)
    assert np.array_equal(spins[(n - 1) * L * L:].cpu().numpy(), ref)
