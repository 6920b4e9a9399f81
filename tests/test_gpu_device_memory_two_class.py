"""Graphs past the LDS: the device-memory sweeps that take two colour classes per
pass and the replicas in groups, against the plain form (one replica and one class
per launch) bit for bit in every storage format, and against the oracle."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial, make, say

pytestmark = pytest.mark.gpu

STORAGES = [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16, cosm.STORE_FIX16,
            cosm.STORE_FIX32, cosm.STORE_FP16_PK]
TORUS = ci.torus(201, seed=3, weights="pm12")  # 40401 spins, 6 classes, odd n
# 5 classes at most (an odd last class alone), vertices without edges
SPARSE = ci.erdos_renyi_capped(40500, 1.6, 4, seed=4)


def phases(inst, colour, C, p, R, h=None):
    say(f"[gpu] {inst.name} R={R} store={p.storage} res={p.residency}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=3, replicas=R, h=h) as st:
        st.sweep(5)
        st.sweep(p.sweeps_per_trial - 5)
        return st.get_phases(cosm.UNIT_TURNS), st.info()["residency"]


def against_plain(inst, method, sides, R, h=None, **kw):
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, method, sides)
    p = cosm.Params(sweeps_per_trial=12, **kw)
    a, res = phases(inst, colour, C, p, R, h)
    assert res == cosm.RES_HBM
    p.residency = cosm.RES_PLAIN
    b, _ = phases(inst, colour, C, p, R, h)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("storage", STORAGES)
def test_torus(storage):
    against_plain(TORUS, cosm.COLOR_TORUS, [201, 201], 4, storage=storage, dwt_ratio=0.5,
                  dwt_period=3)


@pytest.mark.parametrize("storage", [cosm.STORE_FP32, cosm.STORE_BF16, cosm.STORE_FIX16])
@pytest.mark.parametrize("R", [1, 2, 5])
def test_sparse_ragged(storage, R):
    against_plain(SPARSE, cosm.COLOR_MISRA_GRIES, None, R, storage=storage, dwt_ratio=1.0,
                  dwt_period=1)


@pytest.mark.parametrize("kw", [dict(schedule=cosm.SCHED_CONTINUOUS), dict(dwt_period=0)],
                         ids=["continuous", "no-twist"])
def test_schedules(kw):
    against_plain(TORUS, cosm.COLOR_TORUS, [201, 201], 2, **kw)


def test_fields():
    rng = np.random.default_rng(1)
    against_plain(SPARSE, cosm.COLOR_MISRA_GRIES, None, 3, dwt_ratio=1.0, dwt_period=2,
                  h=rng.integers(-2, 3, size=SPARSE.n).astype(np.int32))


def test_replica_groups():
    """More replicas than one group: replicas of every group against the oracle."""
    inst = ci.torus(202, seed=5)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [202, 202])
    p = cosm.Params(sweeps_per_trial=9, dwt_ratio=0.5, dwt_period=3)
    check_trial(inst, colour, C, prob, p, seed=7, R=1300, sweeps=9, chunks=2,
                sample=[0, 511, 512, 767, 768, 1023, 1024, 1299])
