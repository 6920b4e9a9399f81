"""The batch's word schedule (one |J|, one replica set per workgroup) and FP32's wrap at
the twists against single states: vertex counts either side of the room for the dummy
rows at each row width, classes of one slot and of odd and even numbers of them with
last slots of few lanes, an empty class, every storage format with and without the
grid, and runs that mix graphs of either rule with graphs outside it (couplings of two
magnitudes, no twist, drifts past a turn)."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_batch import say, single

pytestmark = pytest.mark.gpu


def compare(reqs, max_n, runs):
    with cosm.Batch(storage=reqs[0][3].storage, max_graphs=len(reqs), max_n=max_n) as b:
        ids = [b.add(i.n, i.eu, i.ev, i.J, c, C, p, seed=50 + k, replicas=R)
               for k, (i, c, C, p, R) in enumerate(reqs)]
        for sel in runs:
            b.run([ids[k] for k in sel])
            b.wait()
            for k in sel:
                inst, c, C, p, R = reqs[k]
                say(f"[gpu] batch words {inst.name} n={inst.n} R={R} {b.shape(ids[k])}")
                H, cut, sp = b.results(ids[k], return_spins=True)
                Hs, cs, ss = single(inst, c, C, p, 50 + k, R)
                assert np.array_equal(H, Hs) and np.array_equal(cut, cs)
                assert np.array_equal(sp, ss)


def regular(n, seed, **kw):
    inst = ci.random_regular(n, 3, seed=seed, **kw)
    c, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_GREEDY)
    return inst, c, C


# rows of 4, 2 and 1 words: 163584 bytes less 2048 of angles and the class counts
@pytest.mark.parametrize("n", [1024, 2050, 6200, 10024, 10040, 10094, 20120, 20128, 20186])
def test_sizes(n):
    inst, c, C = regular(n, n)
    p = cosm.Params(sweeps_per_trial=13, dwt_ratio=1.0, dwt_period=6)
    # a class of no edges, and a set of its own for each row width
    reqs = [(inst, c, C, p, 5), (inst, np.where(c >= 1, c + 1, c), C + 1, p, 3)]
    for w in (1, 2, 4):
        if n * 4 * w + 2048 + 4 * C <= 163584:
            q = cosm.Params(sweeps_per_trial=13, dwt_ratio=1.0, dwt_period=6,
                            replicas_per_wg=w)
            reqs.append((inst, c, C, q, w))
    compare(reqs, n, [list(range(len(reqs)))])


def test_mixed_rules():
    p = dict(sweeps_per_trial=40)
    a = (*regular(6000, 1), cosm.Params(dwt_ratio=1.0, dwt_period=6, **p), 9)
    two = (*regular(6002, 2, weights="pm12"), cosm.Params(dwt_ratio=0.5, dwt_period=2, **p), 4)
    none = (*regular(6004, 3), cosm.Params(dwt_ratio=0.0, dwt_period=0, **p), 4)
    far = (*regular(6006, 4), cosm.Params(dwt_ratio=1.0, dwt_period=40, **p), 4)
    compare([a, two, none, far], 6006,
            [[0], [0, 1], [0, 1, 2, 3], [3], [1, 0], [0]])


@pytest.mark.parametrize("storage", [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16,
                                     cosm.STORE_FIX16, cosm.STORE_FIX32, cosm.STORE_FP16_PK])
def test_storages(storage):
    """The twist every 2 sweeps keeps the 16-bit formats inside their drift bound, every
    6 does not."""
    inst, c, C = regular(6400, 8)
    p = [cosm.Params(sweeps_per_trial=25, dwt_ratio=1.0, dwt_period=t, storage=storage)
         for t in (2, 6)]
    compare([(inst, c, C, q, 9) for q in p], 6400, [[0], [1], [0, 1]])


def test_continuous_schedule():
    inst, c, C = regular(6400, 9)
    p = cosm.Params(sweeps_per_trial=25, dwt_ratio=1.0, dwt_period=6,
                    schedule=cosm.SCHED_CONTINUOUS)
    compare([(inst, c, C, p, 9)], 6400, [[0]])
