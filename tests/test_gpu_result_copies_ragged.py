"""Large results of an odd number of bytes on their way to the host: the last chunk
does not divide evenly among the threads that empty it, and the caller's array holds
every spin, in a state and in a batch."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def graph(n):
    inst = ci.erdos_renyi_capped(n, 4, 8, seed=n)
    return inst, *cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_MISRA_GRIES)


@pytest.mark.parametrize("n,R", [
    (753, 3601),    # 2.6 MB, 1 byte past a page per thread (two threads)
    (1003, 3267),   # 3.1 MB, the same
    (1025, 16369),  # 16 MiB + 1009 bytes
])
def test_every_spin_arrives(n, R):
    inst, colour, C = graph(n)
    p = cosm.Params(sweeps_per_trial=4, replicas_per_wg=4, threads_per_wg=512)
    say(f"[gpu] ragged results n={n} R={R}")
    with cosm.State(inst.n, inst.eu, inst.ev, inst.J, colour, C, p, seed=2, replicas=R) as st:
        st.sweep(4)
        spins = st.energy()[2]
        assert set(np.unique(spins)) <= {-1, 1}
        assert np.array_equal(st.energy(spins)[2], spins)  # every byte back through the device
    with cosm.Batch(max_graphs=1, max_n=n) as b:
        g = b.add(inst.n, inst.eu, inst.ev, inst.J, colour, C,
                  cosm.Params(sweeps_per_trial=4, replicas_per_wg=4), seed=2, replicas=R)
        b.run([g])
        b.wait()
        assert np.array_equal(b.results(g, return_spins=True)[2], spins)
