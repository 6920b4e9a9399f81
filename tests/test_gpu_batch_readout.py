"""The batch's readout, four replicas per workgroup, against single states: replica
counts off a multiple of four, graphs whose units end within an XCD's share, large
couplings (64-bit sums), the most bisectors of the grouped form and one more (which
reads one replica per workgroup), every storage format."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_batch import say, single

pytestmark = pytest.mark.gpu

STORAGES = [cosm.STORE_FP32, cosm.STORE_FP16, cosm.STORE_BF16, cosm.STORE_FIX16,
            cosm.STORE_FIX32, cosm.STORE_FP16_PK]


@pytest.mark.parametrize("storage,B", [(s, 100) for s in STORAGES]
                         + [(cosm.STORE_FP32, b) for b in (1, 127, 128)])
def test_batch_readout(storage, B):
    reqs = []
    for k, R in enumerate((1, 3, 4, 70, 257)):
        inst = ci.random_regular(60 + 34 * k, 3, seed=k)
        c, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_GREEDY)
        large = k == 3 and storage == cosm.STORE_FP32
        inst.J = (inst.J * (1 << 24 if large else 1)).astype(np.int32)
        p = cosm.Params(sweeps_per_trial=40, n_bisectors=B, storage=storage,
                        **({"alpha0_deg": 1e-8} if large else {}))
        reqs.append((inst, c, C, p, 20 + k, R))
    with cosm.Batch(storage=storage, max_graphs=8, max_n=400, max_bisectors=B) as b:
        ids = [b.add(i.n, i.eu, i.ev, i.J, c, C, p, seed=s, replicas=R)
               for i, c, C, p, s, R in reqs]
        b.run(ids)
        b.wait()
        for gid, (inst, c, C, p, seed, R) in zip(ids, reqs):
            say(f"[gpu] batch readout {inst.name} R={R} B={B} storage {storage}")
            H, cut, sp = b.results(gid, return_spins=True)
            Hs, cs, ss = single(inst, c, C, p, seed, R)
            assert np.array_equal(H, Hs) and np.array_equal(cut, cs)
            assert np.array_equal(sp, ss)
