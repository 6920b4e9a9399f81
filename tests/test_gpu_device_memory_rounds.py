"""Graphs past the LDS whose pairs of colour classes are large or small: rounds that take
two classes per pass and rounds that run class by class, in one sweep; against the plain
form (one replica and one class per launch) bit for bit."""
import numpy as np
import pytest

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from test_gpu_device_memory_two_class import against_plain

pytestmark = pytest.mark.gpu


def hub(n, m, degree, seed):
    """m edges, at most 4 at a vertex, and vertex 0 with `degree` of them."""
    rng = np.random.default_rng(seed)
    deg = np.zeros(n, int)
    edges = {(0, int(v)) for v in 1 + rng.permutation(n - 1)[:degree]}
    for _, v in edges:
        deg[v] += 1
    deg[0] = 4
    while len(edges) < m:
        u, v = sorted(int(x) for x in rng.integers(1, n, size=2))
        if u != v and deg[u] < 4 and deg[v] < 4 and (u, v) not in edges:
            edges.add((u, v))
            deg[u] += 1
            deg[v] += 1
    e = np.array(sorted(edges), np.int32)
    return ci.Instance(f"hub{n}_{degree}", n, e[:, 0].copy(), e[:, 1].copy(),
                       rng.choice(np.array([-2, -1, 1, 2], np.int32), size=m))


HUB = hub(40503, 76000, 24, seed=5)  # 0.43 n to 0.31 n edges in the first 5 of 25 classes
CUBIC = ci.random_regular(40502, 3, seed=6, weights="pm1")


@pytest.mark.parametrize("storage", [cosm.STORE_FP32, cosm.STORE_BF16, cosm.STORE_FIX16])
@pytest.mark.parametrize("R", [1, 6, 260])
def test_large_and_small_rounds(storage, R):
    against_plain(HUB, cosm.COLOR_MISRA_GRIES, None, R, storage=storage, dwt_ratio=1.0,
                  dwt_period=2)


@pytest.mark.parametrize("R", [1, 2, 5])
def test_every_round_a_pass(R):
    against_plain(CUBIC, cosm.COLOR_BALANCED, None, R, dwt_ratio=1.0, dwt_period=1)


def test_fields():
    rng = np.random.default_rng(1)
    against_plain(CUBIC, cosm.COLOR_BALANCED, None, 3, dwt_ratio=1.0, dwt_period=2,
                  h=rng.integers(-2, 3, size=CUBIC.n).astype(np.int32))
