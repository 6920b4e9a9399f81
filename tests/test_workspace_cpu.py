"""cosm_workspace_bytes of graphs past the LDS (no device needed): the tables of the
sweeps that take two classes per pass grow with the edges, not with vertices x classes."""
import ctypes

import pytest

from paper_2605_30355_amd.cosm import Params, load_library


def workspace(n, m, C, R=1, **kw):
    out = ctypes.c_size_t(0)
    cp = Params(**kw)._c()
    rc = load_library().cosm_workspace_bytes(n, m, C, R, ctypes.byref(cp), ctypes.byref(out))
    assert rc == 0
    return out.value


@pytest.mark.parametrize("n,m,C", [(50000, 49999, 49999), (50000, 75000, 1000),
                                   (100000, 300000, 60)])
def test_many_small_classes(n, m, C):
    extra = workspace(n, m, C) - workspace(n, m, C, residency=3)  # 3: the plain form
    # a second phase buffer, and 16 bytes per vertex for each pair of classes that can hold
    # a quarter as many edges as there are vertices, and one more
    assert extra <= 4 * n + (4 * m // n + 1) * 16 * (n + 2) + 4096
