"""smc_pt_plan bounds the launches of a tempering call.  Each case names the
launches that the call's route issues: prepare and finish, per step the sweeps,
the collection of the energy sums (16 and more workgroups per replica) and the
exchange round, and what a copy of the lattices takes."""
import numpy as np
import pytest

import paper_1101_1427_amd as S

UNEVEN3D = [(48, 0, k * 48 ** 3, 0) for k in range(3)]
UNEVEN2D = [(32, 0, k * 1024, 0) for k in range(3)] + [(64, 1, 3072 + k * 4096, 2048) for k in range(3)]


@pytest.mark.parametrize("model,dim,L,n_chains,n,m,issued", [
    (S.EA, 3, 64, 2, 5, 1, 2 + 2 + 5 * (2 + 1 + 1)),       # packed copy: pack and unpack as well
    (S.EA, 3, 64, 2, 5, 3, 2 + 2 + 5 * (6 + 1 + 1)),
    (S.ISING, 3, 34, 2, 5, 2, 2 + 2 + 5 * (4 + 1)),        # (ten workgroups per replica: no collection)
    (S.EA, 3, 0, 1, 5, 2, 2 + 5 * (4 + 1 + 1)),            # uneven: half-sweeps on the caller's bytes
    (S.EA, 2, 514, 2, 5, 2, 2 + 5 * (1 + 1 + 1)),          # tiles, both sweeps of a step in one launch, a copy at the end
    (S.ISING, 2, 1024, 1, 5, 4, 2 + 5 * (1 + 1 + 1)),
    (S.EA, 2, 64, 2, 5, 2, 2 + 5 + 1),                     # bins, exchange rounds in the launches that follow
    (S.EA, 2, 0, 2, 5, 2, 2 + 5 + 1),
    (S.EA, 3, 10, 2, 5, 2, 1),                             # a chain on chip for the call
    (S.EA, 3, 16, 2, 5, 2, 1),
    (S.EA, 3, 64, 2, 0, 1, 0),
])
def test_plan_bounds_the_launches(model, dim, L, n_chains, n, m, issued):
    inst = None if L else np.array(UNEVEN3D if dim == 3 else UNEVEN2D)
    b = S.Batch(model, dim, L, 3 * n_chains, 3, rep_per_sample=3, inst=inst)
    launches = S.pt_plan(b, n_chains, 3, [0.3, 0.6, 0.9], n, sweeps_per_step=m)[0]
    assert issued <= launches <= (1 if issued == 1 else 6 + n * (2 * m + 4))
