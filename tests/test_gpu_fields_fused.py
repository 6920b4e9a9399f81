"""Bias fields and the twist inside the last class's sub-sweep (lane schedules in
registers): one, two and up to four slots in the last class, rows outside it, and
schedules that keep passes of their own; against the device-memory form, bit for
bit, in every storage format."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial, make, say

pytestmark = pytest.mark.gpu

STORAGES = [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16, cosm.STORE_FIX16,
            cosm.STORE_FIX32, cosm.STORE_FP16_PK]


def with_fields(inst, seed):
    rng = np.random.default_rng(seed)
    inst.h = rng.integers(-2, 3, size=inst.n).astype(np.int32)  # zeros among them
    return inst


def phases(inst, colour, C, p, R):
    say(f"[gpu] fields {inst.name} store={p.storage} res={p.residency} th={p.threads_per_wg}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=3, replicas=R,
                    h=inst.h) as st:
        st.sweep(20)
        st.sweep(p.sweeps_per_trial - 20)
        return st.get_phases(cosm.UNIT_TURNS), st.info()["twist_fused"]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("threads,fused", [(256, 1), (128, 1), (64, 1)],
                         ids=["one-slot", "two-slots", "three-slots"])
def test_slots_of_the_last_class(threads, fused, storage):
    inst = with_fields(ci.random_regular(300, 3, seed=4, weights="pm1"), 1)
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_BALANCED)
    p = cosm.Params(sweeps_per_trial=61, dwt_ratio=1.0, dwt_period=3, storage=storage,
                    replicas_per_wg=2, threads_per_wg=threads, residency=cosm.RES_LDS)
    a, was = phases(inst, colour, C, p, 5)
    assert was == fused
    q = cosm.Params(sweeps_per_trial=61, dwt_ratio=1.0, dwt_period=3, storage=storage,
                    residency=cosm.RES_HBM)
    assert np.array_equal(a, phases(inst, colour, C, q, 5)[0])


@pytest.mark.parametrize("alpha0,period", [(14.0, 3), (60.0, 2), (14.0, 0)],
                         ids=["wrapped-at-sweep-ends", "wrapped-at-updates", "no-twist"])
@pytest.mark.parametrize("name", ["torus13", "er", "sparse"])
def test_against_the_oracle(name, alpha0, period):
    """Seam classes (few rows in the last class: passes), an irregular graph, and one
    where most rows lie outside the last class."""
    inst = {"torus13": lambda: ci.torus(13, seed=2),
            "er": lambda: ci.erdos_renyi_capped(401, 4, 8, seed=6),
            "sparse": lambda: ci.erdos_renyi_capped(300, 1.2, 4, seed=7)}[name]()
    inst = with_fields(inst, 2)
    colour, C, prob = make(inst, cosm.COLOR_MISRA_GRIES if name != "torus13" else cosm.COLOR_TORUS,
                           [13, 13] if name == "torus13" else None)
    p = cosm.Params(alpha0_deg=alpha0, sweeps_per_trial=90, dwt_ratio=0.5, dwt_period=period,
                    residency=cosm.RES_LDS, replicas_per_wg=4)
    check_trial(inst, colour, C, prob, p, seed=13, R=6, sweeps=90, chunks=2)
