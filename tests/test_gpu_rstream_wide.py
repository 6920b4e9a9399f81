"""The streamed register-owner form at four replicas per row on graphs too large
for the pair layout at that width: seam vertices of an odd torus in the last
register row, with solo slots in the seam classes; bit-exact against the oracle
and against the pair layout."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial, make, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("period", [3, 9], ids=["wrap-at-twists", "wrap-each-update"])
def test_torus141_solo_slots(period):
    inst = ci.torus(141, seed=4)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [141, 141])
    p = cosm.Params(sweeps_per_trial=200, dwt_ratio=0.5, dwt_period=period,
                    lds_form=cosm.LDS_FORM_REGISTER_STREAM, threads_per_wg=1024)
    info = check_trial(inst, colour, C, prob, p, seed=5, R=1027, sweeps=200, chunks=2,
                       sample=[0, 3, 511, 1023, 1026])
    assert info["replicas_per_wg"] == 4 and info["register_rows"] == 10
    assert info["register_vertices"] == 9870  # half the torus, seams included


@pytest.mark.parametrize("inst,method,sides", [
    (ci.torus(139, seed=5, weights="pm12"), cosm.COLOR_TORUS, [139, 139]),  # |J| varies
    (ci.random_regular(16000, 3, seed=6), cosm.COLOR_BALANCED, None)],      # no minor class
    ids=lambda x: getattr(x, "name", None))
def test_against_the_pair_layout(inst, method, sides):
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, method, sides)
    out = []
    for form, rw in ((cosm.LDS_FORM_REGISTER_STREAM, 0), (cosm.LDS_FORM_PAIR, 2)):
        p = cosm.Params(sweeps_per_trial=100, dwt_ratio=1.0, dwt_period=2, lds_form=form,
                        replicas_per_wg=rw, threads_per_wg=1024)
        say(f"[gpu] {inst.name} form={form}")
        with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=2,
                        replicas=1024) as st:
            st.sweep(100)
            out.append((*st.energy(), st.info()["replicas_per_wg"]))
    assert out[0][3] == 4
    for a, b in zip(out[0][:3], out[1][:3]):
        assert np.array_equal(a, b)
