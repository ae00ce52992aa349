"""Calls on two streams that add to the same sums (energy changes, accepted moves):
nothing is lost, whichever path the calls take."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1101_1427_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,dim,L,n_rep,sweeps", [
    (S.ISING, 2, 128, 128, 4),      # tiles, sums collected from slots
    (S.EA, 2, 64, 512, 8),          # whole lattices
    (S.EA, 3, 48, 32, 3),           # packed copy
    (S.EA, 3, 10, 512, 8),          # whole replicas on chip
    (S.HEISENBERG, 3, 8, 512, 8),
    (S.HEISENBERG, 3, 64, 8, 1)])   # one pass per sweep
def test_two_streams_one_sum(model, dim, L, n_rep, sweeps):
    calls, b = 300, [S.Batch(model, dim, L, n_rep, seed) for seed in (1, 2)]
    heis = model == S.HEISENBERG
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    beta = np.full(n_rep, 0.3)
    spins, coup = [], []
    for q in b:
        spins.append(torch.zeros(q.spins_shape()[0], dtype=torch.float32 if heis else torch.int8, device="cuda"))
        coup.append(torch.zeros(q.coup_len(), dtype=torch.int8, device="cuda") if model == S.EA else None)
        S.spin_init(q, spins[-1], coup[-1])
    start = [s.clone() for s in spins]

    def run(sums):
        torch.cuda.synchronize()
        for k in range(calls):
            for q, s, c, st, d in zip(b, spins, coup, streams, sums):
                S.metropolis_sweep(q, s, beta, k * sweeps, sweeps, couplings=c, dE_accum=d, stream=st)
        torch.cuda.synchronize()

    apart = [torch.zeros(n_rep, dtype=torch.int64, device="cuda") for _ in b]
    run(apart)
    for s, s0 in zip(spins, start):
        s.copy_(s0)
    one = torch.zeros(n_rep, dtype=torch.int64, device="cuda")
    run([one, one])
    assert torch.equal(one, apart[0] + apart[1])
