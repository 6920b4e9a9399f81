"""Host checks of the streamed register-owner schedule with solo slots (reg_schedule.cpp
compiled with g++, tests/cpp/solo_check.cpp): every edge exactly once, and no edge in the
pair slot whose words the solo edges take, up to as many edges between LDS rows as the
other pair slots hold."""
import os
import subprocess
from types import SimpleNamespace

import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("bin") / "solo_check")
    csrc = os.path.join(ROOT, "paper_2605_30355_amd", "csrc")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", csrc, "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "cpp", "solo_check.cpp"),
                           os.path.join(csrc, "reg_schedule.cpp"), "-o", out])
    return out


def run(checker, inst, colour, C, W, nth):
    txt = f"{inst.n} {len(inst.eu)} {C}\n" + "\n".join(
        f"{u} {v} {J} {c}" for u, v, J, c in zip(inst.eu, inst.ev, inst.J, colour))
    r = subprocess.run([checker, str(W), str(nth)], input=txt, capture_output=True, text=True,
                       timeout=120)
    if r.returncode == 2:
        return None
    assert r.returncode == 0, r.stderr
    return {k: int(v) for k, v in (kv.split("=") for kv in r.stdout.split())}


def two_sides(side, inner, cross, seed):
    """Four matchings between two sides of `side` vertices, and a fifth class of `inner`
    edges within one side and `cross` edges between them."""
    rng = np.random.default_rng(seed)
    edges = {}
    for c in range(4):
        for u, v in enumerate(rng.permutation(side)):
            edges.setdefault((u, side + int(v)), c)  # (a repeated pair keeps its first class)
    b = side + rng.permutation(side)
    for k in range(inner):
        edges[(int(b[2 * k]), int(b[2 * k + 1]))] = 4
    a = rng.permutation(side)
    for k in range(cross):
        edges.setdefault((int(a[k]), int(b[2 * inner + k])), 4)
    keys = list(edges)
    J = rng.choice([-2, -1, 1, 2], size=len(keys))
    return SimpleNamespace(n=2 * side, eu=[e[0] for e in keys], ev=[e[1] for e in keys], J=J), [
        edges[e] for e in keys]


@pytest.mark.parametrize("W", [2, 4])
@pytest.mark.parametrize("inner", [10, 900, 1228, 1382, 1530])
def test_edges_outside_the_registers(checker, inner, W):
    inst, colour = two_sides(4000, inner, 60, seed=inner)
    f = run(checker, inst, colour, 5, W, 512)
    if f is None:  # (more edges than the three slots left hold)
        assert inner == 1530
        return
    assert f["equal"] == 1 and f["bad"] == 0 and f["masks"] == 0, f
    assert f["solo"] > 0 and f["free"] >= inner, f


@pytest.mark.parametrize("side", [101, 139, 141])
def test_odd_tori(checker, side):
    inst = ci.torus(side, seed=4, weights="pm12")
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_TORUS, [side, side])
    f = run(checker, inst, colour, C, 4, 1024)
    assert f["equal"] == 1 and f["bad"] == 0 and f["masks"] == 0 and f["solo"] > 0, f
