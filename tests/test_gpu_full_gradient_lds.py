"""The full-gradient update with the phases in LDS against the device-memory form
(residency HBM), which takes the same operations in the same order: equal bit
for bit in every storage format and schedule."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def run(inst, p, R, x0=None, h=None):
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_GREEDY)
    say(f"[gpu] full gradient {inst.name} R={R} store={p.storage} res={p.residency}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=6, replicas=R, h=h) as st:
        if x0 is not None:
            st.set_phases(x0, cosm.UNIT_TURNS, 0)
        st.sweep(p.sweeps_per_trial // 3)
        st.sweep(p.sweeps_per_trial - p.sweeps_per_trial // 3)
        return st.get_phases(cosm.UNIT_TURNS), *st.energy(), st.info()["residency"]


def both(inst, R, x0=None, h=None, **kw):
    p = cosm.Params(update=cosm.UPDATE_FULL_GRADIENT, **kw)
    a = run(inst, p, R, x0, h)
    p.residency = cosm.RES_HBM
    b = run(inst, p, R, x0, h)
    assert a[4] == cosm.RES_LDS and b[4] == cosm.RES_HBM
    for u, v in zip(a[:4], b[:4]):
        assert np.array_equal(u, v)


STORAGES = [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16, cosm.STORE_FIX16,
            cosm.STORE_FIX32, cosm.STORE_FP16_PK]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("inst", [
    ci.cycle(5), ci.torus(8, seed=2), ci.random_regular(130, 8, seed=3, weights="pm12"),
    ci.erdos_renyi_capped(901, 4, 8, seed=4), ci.erdos_renyi_capped(9000, 3, 8, seed=5)],
    ids=lambda i: i.name)
def test_formats_and_degrees(inst, storage):
    both(inst, 7, storage=storage, sweeps_per_trial=61, dwt_ratio=0.5, dwt_period=3)


@pytest.mark.parametrize("R", [1, 600, 1030])
def test_row_widths(R):
    """One, two and four words per row (the widest that gives each CU a workgroup),
    ragged at the end, a twist every sweep."""
    both(ci.random_regular(300, 3, seed=8), R, sweeps_per_trial=40, dwt_ratio=1.0, dwt_period=1)


@pytest.mark.parametrize("kw", [dict(schedule=cosm.SCHED_CONTINUOUS), dict(dwt_period=0),
                                dict(alpha0_deg=100.0)],
                         ids=["continuous", "no-twist", "drift-past-a-turn"])
def test_schedules(kw):
    both(ci.random_regular(130, 5, seed=9, weights="pm1"), 9, sweeps_per_trial=50, **kw)


def test_fields_and_phases_off_the_grid():
    inst = ci.random_regular(200, 3, seed=10, weights="pm1")
    rng = np.random.default_rng(1)
    both(inst, 5, h=rng.integers(-3, 4, size=inst.n).astype(np.int32), sweeps_per_trial=50,
         dwt_ratio=1.0, dwt_period=2)
    both(inst, 5, x0=rng.random((5, inst.n)), sweeps_per_trial=50)
