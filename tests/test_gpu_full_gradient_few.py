"""The full-gradient update of a few replicas of a large graph runs from device memory,
where all CUs share them, and many replicas or a small graph in LDS; the results are those
of the device-memory form."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_full_gradient_lds import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,storage,want", [
    (18000, 1, cosm.STORE_FP32, cosm.RES_HBM), (18000, 130, cosm.STORE_FP32, cosm.RES_LDS),
    (18000, 16, cosm.STORE_FIX16, cosm.RES_HBM), (300, 1, cosm.STORE_FP32, cosm.RES_LDS)])
def test_residency(n, R, storage, want):
    inst = ci.random_regular(n, 3, seed=3)
    p = cosm.Params(update=cosm.UPDATE_FULL_GRADIENT, storage=storage, sweeps_per_trial=31,
                    dwt_ratio=1.0, dwt_period=6)
    a = run(inst, p, R)
    p.residency = cosm.RES_HBM
    b = run(inst, p, R)
    assert a[4] == want
    for u, v in zip(a[:4], b[:4]):
        assert np.array_equal(u, v)
