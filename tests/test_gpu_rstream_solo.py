"""Streamed register owners with solo slots beside many edges between LDS rows in the
same class: bit-exact against the oracle."""
import numpy as np
import pytest

import cosm_inputs as ci
import oracle
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial
from test_solo_schedule_cpu import two_sides

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rw", [2, 4])
@pytest.mark.parametrize("inner", [900, 1382])
def test_edges_outside_the_registers(inner, rw):
    g, colour = two_sides(4000, inner, 60, seed=inner)
    inst = ci.Instance(f"two_sides{inner}", g.n, *(np.array(a, np.int32) for a in (g.eu, g.ev, g.J)))
    colour = np.array(colour, np.int32)
    prob = oracle.Problem(inst.n, inst.eu, inst.ev, inst.J, colour=colour, C=5)
    p = cosm.Params(sweeps_per_trial=60, dwt_ratio=0.5, dwt_period=1, replicas_per_wg=rw,
                    threads_per_wg=512, lds_form=cosm.LDS_FORM_REGISTER_STREAM)
    info = check_trial(inst, colour, 5, prob, p, seed=6, R=9, sweeps=60, chunks=2)
    assert info["lds_form"] == cosm.LDS_FORM_REGISTER_STREAM
