"""Host checks of when FP32 phases may be left unwrapped between twists: a form that
takes an edge's difference from the edge's v end needs it exact, which it is below two
turns (host only: tests/cpp/wrap_check.cpp compiled with g++, the rounding by numpy)."""
import os
import subprocess

import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TURN = 1 << 23


def round_down(d):
    """The FP32 number at or below d units of 2^-23 turn (|d| below four turns)."""
    ulp = np.where(np.abs(d) < 2 * TURN, 1, 2)
    return np.floor_divide(d, ulp) * ulp


def test_difference_from_either_end():
    """floor(2d) from d rounded down at the u end, and from -d rounded down and taken
    times -2 at the v end: both exact below two turns, the v end's not above."""
    d = np.concatenate([np.arange(-3 * TURN, 3 * TURN + 1, TURN // 64),
                        *(k * TURN // 2 + np.arange(-3, 4) for k in range(-6, 7))])
    exact = np.floor_divide(2 * d, TURN)
    u_end = np.floor_divide(2 * round_down(d), TURN)
    v_end = np.floor_divide(-2 * round_down(-d), TURN)
    assert np.array_equal(u_end, exact)
    near = np.abs(d) <= 2 * TURN
    assert np.array_equal(v_end[near], exact[near])
    assert v_end[d == -2 * TURN - 1] == exact[d == -2 * TURN - 1] + 1


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("bin") / "wrap_check")
    csrc = os.path.join(ROOT, "paper_2605_30355_amd", "csrc")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", csrc, "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "cpp", "wrap_check.cpp"),
                           os.path.join(csrc, "wrap_bound.cpp"), "-o", out])
    return out


def bounds(checker, inst, method, sides, alpha0, ratio, period):
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, method, sides)
    txt = f"{inst.n} {inst.m} {C}\n" + "\n".join(
        f"{u} {v} {J} {c}" for u, v, J, c in zip(inst.eu, inst.ev, inst.J, colour))
    r = subprocess.run([checker, str(alpha0), str(ratio), str(period)], input=txt,
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    return {k: int(v) for k, v in (kv.split("=") for kv in r.stdout.split())}


CASES = [
    (ci.torus(16, seed=7, weights="pm1"), cosm.COLOR_TORUS, [16, 16]),
    (ci.torus(12, seed=1, weights="pm12"), cosm.COLOR_TORUS, [12, 12]),
    (ci.torus(13, seed=2), cosm.COLOR_TORUS, [13, 13]),
    (ci.random_regular(200, 3, seed=4), cosm.COLOR_BALANCED, None),
    (ci.random_regular(130, 5, seed=5, weights="pm1"), cosm.COLOR_MISRA_GRIES, None),
    (ci.erdos_renyi_capped(401, 4, 8, seed=6), cosm.COLOR_MISRA_GRIES, None),
    (ci.cycle(7), cosm.COLOR_GREEDY, None),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0].name)
def test_no_difference_reaches_two_turns(checker, case):
    left = 0
    for alpha0 in (3.0, 7.0, 14.0, 17.0, 25.0, 27.1, 28.6, 40.0, 80.0):
        for ratio in (0.0, 0.5, 1.5):
            for period in (1, 2, 3, 6):
                f = bounds(checker, *case, alpha0, ratio, period)
                assert not f["dual"] or (f["twists"] and f["reach_dual"] < 2 * TURN), f
                assert not f["owner"] or (f["twists"] and f["reach_owner"] < 2 * TURN), f
                assert not f["sweeps"] or f["reach_sweep"] < 2 * TURN, f
                left += f["dual"] + f["owner"] + f["sweeps"]
    assert left > 0


def test_which_workloads_leave_the_wrap(checker):
    """The tori at 14 degrees and period 3 are wrapped at the twists in either form, a
    3-regular graph at period 6 in neither; at 28.6 degrees the differences of a torus
    may pass two turns."""
    for side in (20, 21):
        f = bounds(checker, ci.torus(side, seed=1), cosm.COLOR_TORUS, [side, side], 14.0, 0.5, 3)
        assert (f["twists"], f["dual"], f["owner"], f["sweeps"]) == (1, 1, 1, 1)
    f = bounds(checker, *CASES[1], 25.0, 1.0, 3)
    assert (f["twists"], f["sweeps"]) == (0, 1)
    f = bounds(checker, *CASES[3], 14.0, 1.0, 6)
    assert (f["twists"], f["dual"], f["owner"]) == (1, 0, 0)
    f = bounds(checker, *CASES[0], 28.6, 0.5, 3)
    assert (f["twists"], f["dual"], f["owner"], f["sweeps"]) == (1, 0, 0, 1)
