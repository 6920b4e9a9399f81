"""Differences of more than two turns: phases on the grid whose unwrapped difference at
an edge is -2 turns and one grid step by its update in the third sweep.  Whichever end
of the edge decides its sign, the trajectory is the oracle's."""
import numpy as np
import pytest

import cosm_inputs as ci
import oracle
import paper_2605_30355_amd as cosm
from test_gpu_parity import make, oparams, say

pytestmark = pytest.mark.gpu

TURN = 1 << 23


def phases():
    """Random phases of a 16 x 16 torus, vertex 107 at 0 and its neighbour 123 chosen so
    that at 28.6 degrees they have parted that far before class 2 of the third sweep."""
    x = np.random.default_rng(950820146).integers(0, TURN, size=(256, 2048))[:, 1982]
    x[107], x[123] = 0, 7493873
    return x


@pytest.mark.parametrize("mirrored", [False, True], ids=["v", "u"])
@pytest.mark.parametrize("form,rw", [(cosm.LDS_FORM_PAIR, 1), (cosm.LDS_FORM_PAIR, 2),
                                     (cosm.LDS_FORM_PAIR, 4),
                                     (cosm.LDS_FORM_REGISTER_STREAM, 2)])
def test_two_turns_apart(form, rw, mirrored):
    """mirrored: the edges' ends swapped and the phases reflected, the same differences
    with the other vertex as each edge's v (the register owners hold one side)."""
    inst = ci.torus(16, seed=7, weights="pm1")
    x = phases()
    if mirrored:
        inst.eu, inst.ev = inst.ev, inst.eu
        x = TURN - 1 - x
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [16, 16])
    p = cosm.Params(alpha0_deg=28.6, sweeps_per_trial=200, dwt_ratio=0.5, dwt_period=3,
                    residency=cosm.RES_LDS, lds_form=form, replicas_per_wg=rw)
    deg = (x / TURN * 360.0)[None, :].repeat(4, 0)
    say(f"[gpu] two turns apart form={form} rw={rw} mirrored={mirrored}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=5, replicas=4) as st:
        st.set_phases(deg, cosm.UNIT_DEGREES, 0)
        st.sweep(3)
        got = st.get_phases(cosm.UNIT_DEGREES)
    ref = deg.copy()
    oracle.sweeps(prob, oparams(p), 5, 0, ref, 0, 3, n_threads=1)
    assert np.array_equal(got, ref)
