"""The names that bench.py gives to kernels are of kernels that exist and, for the 3D
sweeps, of the ones that run (the rule of smc_metropolis_sweep, spelled out in spinmc.h)."""
import os
import re

import pytest

import bench
import paper_1101_1427_amd as S

CSRC = os.path.join(os.path.dirname(os.path.abspath(S.__file__)), "csrc")


def test_the_utilisation_summary_looks_for_kernels_of_the_sources():
    src = "".join(open(os.path.join(CSRC, f)).read() for f in sorted(os.listdir(CSRC)) if f.endswith(".hip"))
    kernels = set(re.findall(r"__global__[^;{]*?\b(k_\w+)\(", src))
    text = open(bench.__file__).read()
    names = re.search(r"    names = \((.*?)\)\n", text, re.S).group(1)
    for name in re.findall(r'"(k_\w+)"', names):
        assert any(k.startswith(name) for k in kernels), name


@pytest.mark.parametrize("model,L,n,env,want", [
    (S.EA, 256, 10, {}, "k_pairs3d_half"), (S.EA, 1024, 8, {}, "k_pairs3d_half"), (S.ISING, 256, 10, {}, "k_pairs3d_half"),
    (S.ISING, 512, 10, {}, "k_pairs3d_half"), (S.ISING, 512, 4, {}, "k_ising3d_pass"),
    (S.ISING, 1024, 8, {}, "k_ising3d_pass"), (S.EA, 256, 2, {}, "k_ising3d_half"),
    (S.EA, 256, 10, {"SPINMC_SWEEP3D_PASS": "1"}, "k_ising3d_pass"),
    (S.EA, 512, 10, {"SPINMC_SWEEP3D_PASS": "0"}, "k_ising3d_half"),
    (S.EA, 512, 10, {"SPINMC_SWEEP3D": "0"}, "k_half_sweep_pieces")])
def test_3d_rows(model, L, n, env, want, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    assert bench.sweep3d_kernel(S, S.Batch(model, 3, L, 1, 1), n, env) == want
