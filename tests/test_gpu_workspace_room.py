"""Graphs past the LDS where there is no room for the buffers of the two-class sweeps: a
workspace of the least size, the static array, memory that runs out; the same trials."""
import ctypes

import numpy as np
import pytest
import torch

import cosm_inputs as ci
import paper_2605_30355_amd as cosm
from paper_2605_30355_amd.cosm import _check
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

INST = ci.cycle(40502)  # 2 classes
P = cosm.Params(sweeps_per_trial=6, dwt_ratio=0.5, dwt_period=2)


def graph(inst=INST):
    return cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_GREEDY)


def trial(R, **kw):
    colour, C = graph()
    with cosm.State(INST.n, INST.eu, INST.ev, INST.J, colour, C, P, seed=3, replicas=R, **kw) as st:
        st.sweep(6)
        return st.energy()


def workspace(n, m, C, R, residency):
    p = cosm.Params(sweeps_per_trial=6, dwt_ratio=0.5, dwt_period=2, residency=residency)._c()
    out = ctypes.c_size_t(0)
    _check(cosm.load_library().cosm_workspace_bytes(n, m, C, R, ctypes.byref(p), ctypes.byref(out)))
    return out.value


def test_least_workspace():
    colour, C = graph()
    L, R, cp = cosm.load_library(), 8, P._c()
    least = workspace(INST.n, INST.m, C, R, cosm.RES_PLAIN)
    full = workspace(INST.n, INST.m, C, R, cosm.RES_AUTO)
    assert full > least + 4 * INST.n * R
    want = trial(R)
    eu, ev, J, col = (np.ascontiguousarray(a, np.int32) for a in (INST.eu, INST.ev, INST.J, colour))
    for nbytes, status in ((least - 1, -5), (least, 0), (full - 1, 0), (full, 0)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        h = ctypes.c_void_p()
        say(f"[gpu] workspace of {nbytes} bytes")
        rc = L.cosm_init(ctypes.byref(h), INST.n, INST.m, eu.ctypes.data, ev.ctypes.data,
                         J.ctypes.data, None, col.ctypes.data, C, ctypes.byref(cp), 3, R, None,
                         ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(nbytes))
        assert rc == status
        if rc:
            continue
        H, cut, spins = np.zeros(R, np.int64), np.zeros(R, np.int64), np.zeros((R, INST.n), np.int8)
        _check(L.cosm_sweep(h, 6))
        _check(L.cosm_energy(h, None, spins.ctypes.data, H.ctypes.data, cut.ctypes.data))
        _check(L.cosm_destroy(h))
        for a, b in zip((H, cut, spins), want):
            assert np.array_equal(a, b)


def test_static_array():
    """40502 vertices, 64 replicas: 31 MB without the second phase buffer."""
    say("[gpu] static state past the LDS")
    for a, b in zip(trial(64, static_scratch=True), trial(64)):
        assert np.array_equal(a, b)


def test_memory_runs_out(monkeypatch):
    want = trial(8)
    empty, full = torch.empty, workspace(INST.n, INST.m, 2, 8, cosm.RES_AUTO)

    def short(size, *a, **kw):
        if size == full:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(size, *a, **kw)

    monkeypatch.setattr(torch, "empty", short)
    say("[gpu] no room for the whole workspace")
    for a, b in zip(trial(8), want):
        assert np.array_equal(a, b)


def test_graphs_that_still_fit_the_lds():
    n = 40300
    inst = ci.cycle(n)
    colour, C = graph(inst)
    assert workspace(n, n, C, 4, cosm.RES_AUTO) == workspace(n, n, C, 4, cosm.RES_PLAIN)
    say("[gpu] 40300 vertices in LDS")
    with cosm.State(n, inst.eu, inst.ev, inst.J, colour, C, P, seed=3, replicas=2) as st:
        assert st.info()["residency"] == cosm.RES_LDS
