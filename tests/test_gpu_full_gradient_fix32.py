"""The full-gradient update in LDS on 32-bit fixed-point phases that were set off the
2^-23 turn grid: bit for bit the device-memory form, twists included."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_full_gradient_lds import both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [False, True], ids=["plain", "fields"])
@pytest.mark.parametrize("R", [5, 600])
def test_phases_off_the_grid(R, h):
    inst = ci.random_regular(500, 5, seed=7, weights="pm1")
    rng = np.random.default_rng(2)
    both(inst, R, x0=rng.random((R, inst.n)), storage=cosm.STORE_FIX32, alpha0_deg=3.0,
         dwt_ratio=1.0, dwt_period=3, sweeps_per_trial=140,
         h=rng.integers(-2, 3, size=inst.n).astype(np.int32) if h else None)
