"""Graphs past the LDS: a captured reset and sweeps replayed between eager calls of the
same state.  The passes alternate between two phase buffers; every call leaves the phases
where the next one, and the readout, look for them."""
import numpy as np
import pytest
import torch

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


# an odd number of passes: one a sweep; two, and three on twist sweeps.  An even one.
@pytest.mark.parametrize("inst,method,sides,S", [
    (ci.cycle(40502), cosm.COLOR_GREEDY, None, 5),
    (ci.torus(201, seed=2), cosm.COLOR_TORUS, [201, 201], 7),
    (ci.torus(202, seed=2), cosm.COLOR_TORUS, [202, 202], 3)], ids=lambda x: getattr(x, "name", None))
def test_replays_between_eager_calls(inst, method, sides, S):
    colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, method, sides)
    p = cosm.Params(sweeps_per_trial=S, dwt_ratio=0.5, dwt_period=2)

    def trial(st, seed):
        st.reset(seed)
        st.sweep(S)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=1, replicas=6) as st:
            want = {}
            for seed in (1, 2, 3):
                trial(st, seed)
                want[seed] = st.energy()
            say(f"[gpu] capture {inst.name}")
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
            graph.replay()
            for a, b in zip(st.energy(), want[1]):
                assert np.array_equal(a, b)
