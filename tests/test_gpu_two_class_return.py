"""The two-class form after phases off the grid: the pair layout in the workgroup's
requested shape while they are, the two-class form again from the next reset or the next
phases on the grid."""
import numpy as np
import pytest

import cosm_inputs as ci
import oracle
import paper_2605_30355_amd as cosm
from test_gpu_parity import make, oparams, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [0, 128])
def test_off_the_grid_and_back(threads):
    inst = ci.torus(12, seed=3)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [12, 12])
    p = cosm.Params(sweeps_per_trial=50, residency=cosm.RES_LDS, replicas_per_wg=1,
                    threads_per_wg=threads)
    off = np.random.default_rng(4).random((3, inst.n))
    on = np.floor(off * 2.0 ** 23) * 2.0 ** -23

    def trial(st, x0):
        ref = x0.copy()
        oracle.sweeps(prob, oparams(p), 2, 0, ref, 0, 50, n_threads=1)
        st.sweep(50)
        assert np.array_equal(st.get_phases(cosm.UNIT_DEGREES), ref)

    say(f"[gpu] off the grid and back, threads={threads}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=2, replicas=3) as st:
        def shape():
            return {k: st.info()[k] for k in ("twist_fused", "threads_per_wg", "lds_bytes")}

        two_class = shape()
        first = []
        for k in range(3):
            st.set_phases(off, cosm.UNIT_TURNS, 0)
            assert shape() != two_class
            assert not threads or st.info()["threads_per_wg"] == threads
            st.sweep(50)
            first.append(st.get_phases(cosm.UNIT_TURNS))
            if k == 0:
                st.reset(2)
                assert shape() == two_class
                trial(st, oracle.init_phases(inst.n, 2, 0, 3, oracle.SCHED_GRID))
            elif k == 1:
                st.set_phases(on, cosm.UNIT_TURNS, 0)
                assert shape() == two_class
                trial(st, on * 360.0)
        assert np.array_equal(first[0], first[1]) and np.array_equal(first[0], first[2])
