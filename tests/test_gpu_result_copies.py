"""Energies, cuts and spins on their way to the host: sizes either side of the
limits between one pinned copy, the runtime's own staging and chunks through pinned
memory, in one state, in a batch, and from two threads with a state each."""
import threading

import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

INST = ci.torus(32, seed=3)  # 1024 spins: R kilobytes of spins
# around 192 KiB, 2.5 MiB, 8 MiB and a ragged number of 2 MiB chunks; H and cut of
# 24000 replicas lie either side of the short limit too
SIZES = [1, 191, 192, 193, 2559, 2560, 2561, 8191, 8192, 9000, 24577]


def graph():
    return cosm.build_partitions(INST.n, INST.eu, INST.ev, cosm.COLOR_TORUS, [32, 32])


def reference(spins):
    s = spins.astype(np.int64)
    e = s[:, INST.eu] * s[:, INST.ev]
    return -(e * INST.J).sum(1), -(INST.J * (e < 0)).sum(1)


def check(R, seed, rounds=2):
    colour, C = graph()
    p = cosm.Params(sweeps_per_trial=4, replicas_per_wg=4, threads_per_wg=512)
    with cosm.State(INST.n, INST.eu, INST.ev, INST.J, colour, C, p, seed=seed, replicas=R) as st:
        for k in range(rounds):
            st.reset(seed + k)
            st.sweep(4)
            H, cut, spins = st.energy()
            assert set(np.unique(spins)) <= {-1, 1}
            rows = np.unique(np.r_[0, R // 3, R // 2, R - 1, np.arange(0, R, max(1, R // 50))])
            Hr, cr = reference(spins[rows])
            assert np.array_equal(H[rows], Hr) and np.array_equal(cut[rows], cr)
            Hn, cn, _ = st.energy(return_spins=False)
            assert np.array_equal(H, Hn) and np.array_equal(cut, cn)
            Hs, cs, back = st.energy(spins)  # every byte back through the device
            assert np.array_equal(Hs, H) and np.array_equal(back, spins)


@pytest.mark.parametrize("R", SIZES)
def test_sizes(R):
    say(f"[gpu] results of {R} replicas")
    check(R, 5)


def test_two_threads():
    say("[gpu] results from two threads")
    bad = []

    def run(seed):
        try:
            check(9000, seed, rounds=4)
        except BaseException as e:  # noqa: BLE001 (reported below)
            bad.append(e)

    t = [threading.Thread(target=run, args=(s,)) for s in (11, 12)]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not bad, bad


def test_batch():
    colour, C = graph()
    with cosm.Batch(max_graphs=3, max_n=1024) as b:
        ids = [b.add(INST.n, INST.eu, INST.ev, INST.J, colour, C,
                     cosm.Params(sweeps_per_trial=4, replicas_per_wg=2), seed=s, replicas=R)
               for s, R in ((1, 64), (2, 1000), (3, 4000))]
        say("[gpu] batch results")
        b.run(ids)
        b.wait()
        for g in ids:
            H, cut, spins = b.results(g, return_spins=True)
            Hr, cr = reference(spins)
            assert np.array_equal(H, Hr) and np.array_equal(cut, cr)
