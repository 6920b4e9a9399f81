"""Small graphs on the GPU: the two-class sweep form (two colour classes per
barrier interval), which the library takes when every workgroup has a CU to
itself, bit-exact against the oracle's grid schedules."""
import numpy as np
import pytest

import cosm_inputs as ci
import oracle
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial, make, oparams, say

pytestmark = pytest.mark.gpu


def _eight_regular():
    return ci.random_regular(60, 8, seed=12, weights="pm12")


# class counts 3 to 10 (odd counts leave the last round half empty), odd vertex
# counts, isolated vertices, the largest graph, one wave and several
GRAPHS = {
    "torus8": (lambda: ci.torus(8, seed=1), cosm.COLOR_TORUS, [8, 8]),              # one wave
    "torus13": (lambda: ci.torus(13, seed=2), cosm.COLOR_TORUS, [13, 13]),          # seams, 169
    "torus32": (lambda: ci.torus(32, seed=3), cosm.COLOR_TORUS, [32, 32]),          # 1024
    "cycle7": (lambda: ci.cycle(7), cosm.COLOR_GREEDY, None),                       # 3 classes
    "rr3": (lambda: ci.random_regular(200, 3, seed=4), cosm.COLOR_BALANCED, None),
    "rr5": (lambda: ci.random_regular(130, 5, seed=5, weights="pm1"), cosm.COLOR_MISRA_GRIES, None),
    "er": (lambda: ci.erdos_renyi_capped(401, 4, 8, seed=6), cosm.COLOR_MISRA_GRIES, None),
    "rr8": (_eight_regular, cosm.COLOR_MISRA_GRIES, None),
}


@pytest.mark.parametrize("rw", [1, 2])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_two_class_form_fp32(name, rw):
    """Whole trials over several calls (an odd number of rounds leaves the rows
    in either copy), R not a multiple of the row width."""
    make_inst, method, sides = GRAPHS[name]
    inst = make_inst()
    colour, C, prob = make(inst, method, sides)
    assert 3 <= C <= 10
    p = cosm.Params(sweeps_per_trial=205, dwt_ratio=0.5, dwt_period=3, residency=cosm.RES_LDS,
                    replicas_per_wg=rw)
    info = check_trial(inst, colour, C, prob, p, seed=21, R=7, sweeps=205, chunks=4)
    assert info["twist_fused"] == 1 and info["threads_per_wg"] <= 512


@pytest.mark.parametrize("storage", [cosm.STORE_FIX32, cosm.STORE_FIX16])
@pytest.mark.parametrize("name", ["torus13", "rr3", "er"])
def test_two_class_form_fixed_point(name, storage):
    make_inst, method, sides = GRAPHS[name]
    inst = make_inst()
    colour, C, prob = make(inst, method, sides)
    R, S, sched = 5, 150, (oracle.SCHED_GRID16 if storage == cosm.STORE_FIX16
                           else oracle.SCHED_GRID)
    p = cosm.Params(sweeps_per_trial=S, dwt_ratio=0.5, dwt_period=2, residency=cosm.RES_LDS,
                    storage=storage, replicas_per_wg=2)
    say(f"[gpu] two-class {name} storage={storage}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=8, replicas=R) as st:
        st.sweep(75)
        st.sweep(S - 75)
        x = st.get_phases(cosm.UNIT_DEGREES)
        assert st.info()["twist_fused"] == 1
    op = oracle.Params(dwt_ratio=0.5, dwt_period=2, sweeps=S, schedule=sched)
    ref = oracle.init_phases(inst.n, 8, 0, R, sched)
    oracle.sweeps(prob, op, 8, 0, ref, 0, S, n_threads=2)
    assert np.array_equal(x, ref)


@pytest.mark.parametrize("alpha0,ratio,period,weights", [
    (27.1, 0.5, 3, "pm1"),    # drift 0.941 turn: wrapped at the twists
    (28.6, 0.5, 3, "pm1"),    # 0.993
    (28.9, 0.5, 3, "pm1"),    # 1.003: wrapped at the end of every sweep
    (25.0, 1.0, 3, "pm12"),   # 1.74 over three sweeps, 0.63 over one
    (80.0, 0.5, 1, "pm1"),    # 1.0 within one sweep: wrapped after every update
    (14.0, 0.5, 0, "pm1"),    # no twist
    (3.0, 0.5, 70, "pm1"),    # a twist less than once per 64-sweep table
])
def test_wrap_bounds_two_class(alpha0, ratio, period, weights):
    """The bounds under which FP32 phases are wrapped at the twists, at the ends
    of sweeps or after every update: the same trajectory."""
    inst = ci.torus(16, seed=7, weights=weights)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [16, 16])
    p = cosm.Params(alpha0_deg=alpha0, sweeps_per_trial=200, dwt_ratio=ratio, dwt_period=period,
                    residency=cosm.RES_LDS, replicas_per_wg=1)
    info = check_trial(inst, colour, C, prob, p, seed=31, R=9, sweeps=200, chunks=2)
    assert info["threads_per_wg"] == 128


def test_phases_set_off_the_grid():
    """Phases that are no multiples of 2^-23 turn: every layout wraps after each
    update and stays within 1e-5 turn of the oracle over one sweep."""
    inst = ci.torus(12, seed=3)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [12, 12])
    p = cosm.Params(sweeps_per_trial=50, residency=cosm.RES_LDS, replicas_per_wg=1)
    rng = np.random.default_rng(4)
    x0 = rng.random((3, inst.n)) * 360.0
    say("[gpu] phases off the grid")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=2, replicas=3) as st:
        st.set_phases(x0, cosm.UNIT_DEGREES, 0)
        st.sweep(1)
        x = st.get_phases(cosm.UNIT_DEGREES)
        st.reset(2)
        st.sweep(50)
        after = st.get_phases(cosm.UNIT_DEGREES)
    ref = x0.copy()
    oracle.sweeps(prob, oparams(p), 2, 0, ref, 0, 1, n_threads=1)
    d = np.abs((x - ref + 180.0) % 360.0 - 180.0) / 360.0
    assert np.median(d) < 1e-6 and np.mean(d < 1e-5) > 0.99
    ref = oracle.init_phases(inst.n, 2, 0, 3, oracle.SCHED_GRID)
    oracle.sweeps(prob, oparams(p), 2, 0, ref, 0, 50, n_threads=1)
    assert np.array_equal(after, ref)
