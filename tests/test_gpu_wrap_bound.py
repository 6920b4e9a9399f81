"""FP32 phases on the grid schedule wrapped at the twists only, up to a drift of
one turn between two twists (the parity step needs no exact difference): bit
for bit the oracle's trajectory, on either side of the bound."""
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import check_trial, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha0,ratio,period,weights", [
    (27.1, 0.5, 3, "pm1"),    # drift 0.941 turn: wrapped at the twists
    (28.6, 0.5, 3, "pm1"),    # 0.993
    (28.9, 0.5, 3, "pm1"),    # 1.003: wrapped after every update
    (80.0, 0.5, 1, "pm1"),    # 1.0
    (14.0, 0.5, 0, "pm1"),    # no twist
])
def test_wrap_bounds(alpha0, ratio, period, weights):
    """Either side of the bound under which FP32 phases are wrapped at the twists
    only: the same trajectory."""
    inst = ci.torus(16, seed=7, weights=weights)
    colour, C, prob = make(inst, cosm.COLOR_TORUS, [16, 16])
    p = cosm.Params(alpha0_deg=alpha0, sweeps_per_trial=200, dwt_ratio=ratio, dwt_period=period,
                    residency=cosm.RES_LDS, replicas_per_wg=4)
    check_trial(inst, colour, C, prob, p, seed=31, R=9, sweeps=200, chunks=2)


@pytest.mark.parametrize("large", [False, True], ids=["registers", "streamed"])
def test_wrap_at_twists_up_to_a_turn(large):
    """5-regular graphs at ratio 3/2, period 3 (drift 0.64 turn), schedules held
    in registers and streamed."""
    inst = ci.random_regular(8000 if large else 1500, 5, seed=9, weights="pm1")
    colour, C, prob = make(inst, cosm.COLOR_BALANCED)
    p = cosm.Params(sweeps_per_trial=120, dwt_ratio=1.5, dwt_period=3, residency=cosm.RES_LDS,
                    replicas_per_wg=2, threads_per_wg=1024 if large else 512)
    info = check_trial(inst, colour, C, prob, p, seed=5, R=6, sweeps=120, chunks=3)
    assert info["streamed"] == (1 if large else 0)
