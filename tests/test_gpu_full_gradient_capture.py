"""The full-gradient update in device memory: a captured reset and sweeps replayed between
eager calls of the same state, an odd number of sweeps each."""
import numpy as np
import pytest
import torch

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("residency", [cosm.RES_HBM, cosm.RES_AUTO], ids=["hbm", "auto"])
def test_replays_between_eager_calls(residency):
    inst = ci.random_regular(14000, 3, seed=2)
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_BALANCED)
    p = cosm.Params(sweeps_per_trial=7, dwt_ratio=1.0, dwt_period=6, residency=residency,
                    update=cosm.UPDATE_FULL_GRADIENT)

    def trial(st, seed):
        st.reset(seed)
        st.sweep(7)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=1, replicas=1) as st:
            want = {}
            for seed in (1, 2, 3):
                trial(st, seed)
                want[seed] = st.energy()
            say(f"[gpu] full gradient capture residency={residency}")
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                trial(st, 1)
            for seed in (2, 3, 2):
                graph.replay()
                for a, b in zip(st.energy(), want[1]):
                    assert np.array_equal(a, b)
                trial(st, seed)
                for a, b in zip(st.energy(), want[seed]):
                    assert np.array_equal(a, b)
