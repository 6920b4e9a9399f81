"""The grouped bisector readout (several replicas per workgroup, one-byte codes)
against the oracle's brute force: numbers of bisectors either side of 64 and of the
127 that a byte holds, replica counts either side of one workgroup of four, two and
one replicas per CU, phases on bisectors and a step beside them, large couplings,
every storage format, and graphs past one byte per vertex and replica in LDS."""
import numpy as np
import pytest

import cosm_inputs as ci
import oracle
import paper_2605_30355_amd as cosm
from test_gpu_parity import make, say

pytestmark = pytest.mark.gpu


def check(inst, method, sides, p, R, rows, x0=None):
    colour, C, prob = make(inst, method, sides)
    say(f"[gpu] readout {inst.name} B={p.n_bisectors} R={R} store={p.storage}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=4, replicas=R) as st:
        if x0 is not None:
            st.set_phases(x0, cosm.UNIT_TURNS, 0)
        x = st.get_phases(cosm.UNIT_DEGREES)
        H, cut, spins = st.energy()
    op = oracle.Params(sweeps=p.sweeps_per_trial, n_bisectors=p.n_bisectors, schedule=p.schedule)
    so, Ho, co, _ = oracle.readout(prob, op, np.ascontiguousarray(x[rows]))
    assert np.array_equal(H[rows], Ho) and np.array_equal(cut[rows], co)
    assert np.array_equal(spins[rows], so)


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 100, 127, 128, 500])
def test_bisectors(B):
    """On every bisector (rounded to the grid), a grid step below and above it, and
    the same half a turn on, among random phases."""
    inst = ci.erdos_renyi_capped(301, 4, 8, seed=3)
    p = cosm.Params(sweeps_per_trial=5, n_bisectors=B)
    rng = np.random.default_rng(B)
    k = rng.integers(0, 1 << 23, size=(6, inst.n))
    units = ((np.arange(B, dtype=np.int64) << 23) + B) // (2 * B)
    pick = rng.random((6, inst.n)) < 0.7
    on = (rng.choice(units, size=(6, inst.n)) + rng.integers(-1, 2, size=(6, inst.n))
          + (rng.integers(0, 2, size=(6, inst.n)) << 22)) % (1 << 23)
    x0 = np.where(pick, on, k) / float(1 << 23)
    check(inst, cosm.COLOR_GREEDY, None, p, 6, np.arange(6), x0)


@pytest.mark.parametrize("R", [1, 3, 511, 513, 1021, 1024, 1027])
def test_replicas(R):
    inst = ci.torus(9, seed=2)
    p = cosm.Params(sweeps_per_trial=5)
    check(inst, cosm.COLOR_TORUS, [9, 9], p, R, np.unique(np.r_[0, R // 2, R - 3:R]) % R)


@pytest.mark.parametrize("storage", [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16,
                                     cosm.STORE_FIX16, cosm.STORE_FIX32, cosm.STORE_FP16_PK])
def test_storages(storage):
    inst = ci.random_regular(250, 3, seed=5)
    p = cosm.Params(sweeps_per_trial=5, storage=storage)
    for R in (5, 1024, 1026):
        check(inst, cosm.COLOR_BALANCED, None, p, R, np.arange(0, R, max(1, R // 7)))


def test_large_couplings():
    """Energies past 32 bits."""
    inst = ci.random_regular(200, 4, seed=6)
    inst.J = np.random.default_rng(2).integers(-2**29, 2**29, size=inst.m).astype(np.int32)
    p = cosm.Params(sweeps_per_trial=5, alpha0_deg=1e-8)
    for R in (7, 1030):
        check(inst, cosm.COLOR_GREEDY, None, p, R, np.arange(0, R, max(1, R // 5)))


@pytest.mark.parametrize("side,R", [(203, 1025), (290, 515), (410, 3)])
def test_large_graphs(side, R):
    """Two and one byte codes per vertex in LDS, and codes in device memory."""
    inst = ci.torus(side, seed=7)
    p = cosm.Params(sweeps_per_trial=5)
    check(inst, cosm.COLOR_TORUS, [side, side], p, R, np.array([0, R // 2, R - 1]))
