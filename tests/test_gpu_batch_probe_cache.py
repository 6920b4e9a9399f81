"""The batch's probe cache: an instance of the same edges whose couplings or schedule
select another sweep path is probed for itself."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def test_probed_once_per_path():
    inst = ci.random_regular(1502, 3, seed=77)
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_BALANCED)
    mixed = np.where(np.arange(inst.m) % 2 == 0, 1, 2).astype(np.int32)
    ones = np.ones(inst.m, np.int32)
    say("[gpu] probe cache")
    with cosm.Batch(max_graphs=8, max_n=2000) as b:
        def tuned(J, **kw):
            p = cosm.Params(sweeps_per_trial=40, **kw)
            return b.shape(b.add(inst.n, inst.eu, inst.ev, J, colour, C, p, replicas=64))["tuned"]

        assert tuned(ones, dwt_period=3) == 1   # probed
        assert tuned(-ones, dwt_period=3) == 2  # the same path: from the cache
        assert tuned(mixed, dwt_period=3) == 1  # no word schedule
        assert tuned(ones, dwt_period=0) == 1   # wrapped after every update
        assert tuned(ones, dwt_period=3, schedule=cosm.SCHED_CONTINUOUS) == 1
        assert tuned(mixed, dwt_period=3) == 2
