"""The workloads whose speed is followed: whole trials through the public entry points.

Every case is one pass of a program that solves Ising / Max-Cut / QUBO instances: draw the
initial phases (``reset``), run the trial's sweeps (``sweep``), read the spins out
(``energy``), or the same for many instances at once (``Batch.run`` / ``wait`` / ``results``).
The state or the batch with its graph, colouring and tuned kernel shape is what such a
program keeps between trials; ``prepare`` makes it.

The cases differ in the graph (tori, 3- and 5-regular, capped Erdos-Renyi, sparse QUBO), its
size (144 to 90000 spins), the replicas (1 to 4096), the phase storage, the update rule, the
readout and the sweeps per trial, so that each sweep form is met: schedules held in registers
and streamed, register owners, device memory, the multi-instance launch.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import cosm_inputs as ci
import paper_2605_30355_amd as cosm

STORAGE = {"fp32": cosm.STORE_FP32, "fp16": cosm.STORE_FP16, "bf16": cosm.STORE_BF16,
           "fix16": cosm.STORE_FIX16, "fix32": cosm.STORE_FIX32, "fp16pk": cosm.STORE_FP16_PK}
ELEM_BYTES = {"fp32": 4, "fix32": 4, "fp16": 2, "bf16": 2, "fix16": 2, "fp16pk": 2}

# twist ratio and period of each family (Table X): tori, the unweighted graph, +-1 graphs
TWIST = {"torus": (0.5, 3), "torus12": (1.0, 3), "rr3": (1.0, 6), "rr5": (1.5, 3),
         "er": (1.5, 3), "qubo": (1.0, 6)}


def _case(name, graph, size, replicas, sweeps, storage="fp32", update="scs",
          readout="bisectors", **over):
    c = {"graph": graph, "size": size, "replicas": replicas, "sweeps": sweeps,
         "storage": storage, "update": update, "readout": readout, **over}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one trial at a time on a small +-1/+-2 lattice: a pass is latency and launches
        _case("one_trial_torus12", "torus12", 12, 1, 1000),
        # the small +-1 lattice: 64 replicas of a 20x20 torus
        _case("torus20", "torus", 20, 64, 2000),
        # unweighted Max-Cut on a 3-regular graph, the everyday instance
        _case("maxcut3", "rr3", 2000, 1024, 10000),
        # the same in 16-bit fixed point, read out at the best of all bisectors, short trials
        _case("maxcut3_fix16_optimal", "rr3", 2000, 1024, 1000, "fix16", readout="optimal"),
        # a large even lattice, 16-bit phases
        _case("torus100_fp16", "torus", 100, 4096, 1000, "fp16"),
        # the largest lattice, odd: two seam classes; phases of 19881 spins fill a CU's LDS
        _case("torus141", "torus", 141, 4096, 1000),
        # a dense bounded-degree graph with +-1 couplings
        _case("regular5_n20000", "rr5", 20000, 2048, 1000),
        # an irregular graph, nine uneven classes, brain-float phases
        _case("erdos_renyi_bf16", "er", 10000, 2048, 1000, "bf16"),
        # a service's micro-batch: requests of mixed families and sizes in one launch
        _case("mixed_batch", "mixed", 20000, 256, 500, count=24),
        # a sparse QUBO: bias fields, the single-semicircle readout
        _case("qubo_fields", "qubo", 2000, 1024, 2000),
        # the update without sequential classes (Eq. (8)), as ablation studies run it
        _case("full_gradient", "rr3", 2000, 2048, 1000, update="full"),
        # a lattice beyond a CU's LDS: phases stay in device memory
        _case("torus300_device", "torus", 300, 1024, 50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cap_sweeps(edges, replicas, sweeps, budget):
    """Sweeps of a pass within a budget of edge updates."""
    return max(8, min(sweeps, int(budget // max(1, edges * replicas))))


def draw(rng):
    """One more case of the listed ranges: sizes, replicas, sweeps and storage at random."""
    storage = rng.choice(["fp32", "fp32", "fp32", "fp16", "bf16", "fix16", "fix32", "fp16pk"])
    kind = rng.choice(["small", "torus", "rr3", "rr5", "er", "mixed", "qubo", "full", "device"])
    replicas = _log_int(rng, 16, 4096)
    sweeps = _log_int(rng, 100, 5000)
    if kind == "small":
        return _case(None, "torus12", rng.randint(12, 20), _log_int(rng, 1, 256), sweeps, storage)
    if kind == "torus":
        side = _log_int(rng, 20, 141)
        return _case(None, "torus", side, replicas,
                     _cap_sweeps(2 * side * side, replicas, sweeps, 1.2e11), storage)
    if kind in ("rr3", "rr5", "er"):
        n = 2 * _log_int(rng, 200, 10000)
        deg = {"rr3": 3, "rr5": 5, "er": 4}[kind]
        readout = rng.choice(["bisectors", "bisectors", "optimal"])
        return _case(None, kind, n if kind != "er" else n - rng.randint(0, 1), min(replicas, 2048),
                     _cap_sweeps(n * deg // 2, min(replicas, 2048), sweeps, 6e10), storage,
                     readout=readout)
    if kind == "mixed":
        return _case(None, "mixed", _log_int(rng, 1000, 20000), _log_int(rng, 16, 256),
                     _log_int(rng, 50, 500), rng.choice(["fp32", "fp32", "fix16", "bf16"]),
                     count=rng.randint(2, 24))
    if kind == "qubo":
        n = 2 * _log_int(rng, 50, 4000)
        replicas = min(replicas, 1024)
        return _case(None, "qubo", n, replicas, _cap_sweeps(3 * n, replicas, sweeps, 1e10), storage)
    if kind == "full":
        n = 2 * _log_int(rng, 100, 5000)
        replicas = min(replicas, 2048)
        return _case(None, rng.choice(["rr3", "er"]), n, replicas,
                     _cap_sweeps(2 * n, replicas, sweeps, 6e9), storage, update="full")
    return _case(None, "torus", rng.randint(290, 320), rng.choice([256, 384, 512, 768]),
                 rng.randint(10, 40), storage)


# ---- inputs -----------------------------------------------------------------

@functools.lru_cache(maxsize=8)
def _graph(family, n, seed):
    """A graph of the family and the colouring a program computes once for it."""
    if family in ("torus", "torus12"):
        inst = ci.torus(n, seed=seed)
        colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_TORUS, [n, n])
    elif family in ("rr3", "qubo"):
        inst = ci.random_regular(n, 3, seed=seed)
        colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_BALANCED)
    elif family == "rr5":
        inst = ci.random_regular(n, 5, seed=seed)
        colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_BALANCED)
    else:
        inst = ci.erdos_renyi_capped(n, 4, 8, seed=seed)
        colour, C = cosm.build_partitions(inst.n, inst.eu, inst.ev, cosm.COLOR_MISRA_GRIES)
    return inst.n, inst.eu, inst.ev, colour, C


def _instance(family, size, seed):
    """n, eu, ev, J, h, colour, C: the graph of the size, couplings and fields of the seed."""
    n, eu, ev, colour, C = _graph(family, size, 1000 + size)
    rng = np.random.default_rng(seed)
    m = len(eu)
    h = None
    if family == "torus12":
        J = rng.choice(np.array([-2, -1, 1, 2], np.int32), size=m)
    elif family == "rr3":
        J = np.full(m, -1, np.int32)  # Max-Cut weights +1
    elif family == "qubo":
        # min sum q_ij x_i x_j + sum q_i x_i with small integer weights, in Ising form
        q = rng.choice(np.array([-2, -1, 1, 2], np.int32), size=m)
        d = rng.integers(-3, 4, size=n).astype(np.int32)
        J = -q
        h = -2 * d
        np.subtract.at(h, eu, q)
        np.subtract.at(h, ev, q)
        h = h.astype(np.int32)
    else:
        J = rng.choice(np.array([-1, 1], np.int32), size=m)
    return n, eu, ev, J, h, colour, C


def _params(family, case):
    ratio, period = TWIST[family]
    return cosm.Params(
        alpha0_deg=25.0 if family == "torus12" else 14.0, dwt_ratio=ratio, dwt_period=period,
        sweeps_per_trial=case["sweeps"], storage=STORAGE[case["storage"]],
        update=cosm.UPDATE_FULL_GRADIENT if case["update"] == "full" else cosm.UPDATE_SCS,
        readout=cosm.READOUT_OPTIMAL if case["readout"] == "optimal" else cosm.READOUT_BISECTORS)


def _requests(case, seed):
    """The requests of a micro-batch: sizes and families by the case, couplings by the seed."""
    rng = np.random.default_rng(case["size"] + case["count"])
    out = []
    for k in range(case["count"]):
        n = int(rng.integers(400, case["size"] + 1))
        family = ("torus", "rr3", "rr5")[k % 3]
        size = max(3, int(round(math.sqrt(n)))) if family == "torus" else n + n % 2
        out.append((family, size, seed * 1000 + k))
    return out


def _solver_seed(seed):
    return (seed * 2654435761 + 12345) & 0xFFFFFFFF


def prepare(case, seed):
    if case["graph"] == "mixed":
        reqs = _requests(case, seed)
        batch = cosm.Batch(storage=STORAGE[case["storage"]], max_graphs=case["count"],
                           max_n=case["size"] + 1 + 2 * int(math.sqrt(case["size"])))
        ids = []
        for k, (family, size, s) in enumerate(reqs):
            n, eu, ev, J, _, colour, C = _batch_instance(family, size, s)
            ids.append(batch.add(n, eu, ev, J, colour, C, _params(family, case),
                                 seed=_solver_seed(s), replicas=case["replicas"]))
        return {"batch": batch, "ids": ids}
    family = case["graph"]
    n, eu, ev, J, h, colour, C = _instance(family, case["size"], seed)
    st = cosm.State(n, eu, ev, J, colour, C, _params(family, case), seed=_solver_seed(seed),
                    replicas=case["replicas"], h=h)
    return {"state": st, "seed": _solver_seed(seed), "sweeps": case["sweeps"]}


@functools.lru_cache(maxsize=96)
def _batch_graph(family, size):
    return _graph.__wrapped__(family, size, 1000 + size)


def _batch_instance(family, size, seed):
    n, eu, ev, colour, C = _batch_graph(family, size)
    rng = np.random.default_rng(seed)
    J = (np.full(len(eu), -1, np.int32) if family == "rr3"
         else rng.choice(np.array([-1, 1], np.int32), size=len(eu)))
    return n, eu, ev, J, None, colour, C


def run(state):
    if "batch" in state:
        b = state["batch"]
        b.run(state["ids"])
        b.wait()
        res = [b.results(g, return_spins=True) for g in state["ids"]]
        return [np.stack([r[0] for r in res]), np.stack([r[1] for r in res]),
                *(r[2] for r in res)]
    st = state["state"]
    st.reset(state["seed"])
    st.sweep(state["sweeps"])
    H, cut, spins = st.energy()
    return [H, cut, spins]


# ---- the work a pass cannot do without ---------------------------------------

def _sizes(family, size):
    if family in ("torus", "torus12"):
        return size * size, 2 * size * size
    if family == "er":
        return size, 2 * size
    deg = 5 if family == "rr5" else 3
    return size, size * deg // 2


def work(case):
    """Bytes: the graph in; spins, energies and cuts out (the phases are drawn, not given).
    Operations: per edge update a difference, a sign, a scaled step and two sums; per spin
    and twist a test and a sum; per edge of the readout two additions."""
    if case["graph"] == "mixed":
        items = [(f, s) for f, s, _ in _requests(case, 0)]
    else:
        items = [(case["graph"], case["size"])]
    R, S = case["replicas"], case["sweeps"]
    b = f = 0
    for family, size in items:
        n, m = _sizes(family, size)
        fields = family == "qubo"
        b += 16 * m + (4 * n if fields else 0) + R * (n + 16)
        f += R * S * (5 * m + (4 * n if fields else 0) + 3 * n // TWIST[family][1]) + 2 * R * m
    return {"bytes": b, "flops": f}


# ---- the same in 64 bits, with plain torch -----------------------------------
# Phases in units of 2^-23 turn are whole numbers, so the whole trial is exact in int64.

def _philox(c0, c1, c2, c3, key):
    """Words 0 and 1 of Philox4x32-10 for int64 tensors holding 32-bit counters."""
    M = 0xFFFFFFFF
    k0, k1 = key & M, (key >> 32) & M

    def mul(a, b):  # 32 x 32 -> (hi, lo) without overflow of int64
        lo = a * (b & 0xFFFF)
        hi = a * (b >> 16)
        t = lo + ((hi & 0xFFFF) << 16)
        return ((hi >> 16) + (t >> 32)) & M, t & M
    for _ in range(10):
        h0, l0 = mul(c0, 0xD2511F53)
        h1, l1 = mul(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1


def _exact_trial(case, seed):
    n, eu, ev, J, h, colour, C = _instance(case["graph"], case["size"], seed)
    p = _params(case["graph"], case)
    R, S, key = case["replicas"], case["sweeps"], _solver_seed(seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    i64 = dict(dtype=torch.int64, device=dev)
    ONE, HALF = 1 << 23, 1 << 22  # a turn and half a turn
    rid = torch.arange(R, **i64)
    v = torch.arange(n, **i64)[:, None].expand(n, R).contiguous()
    zero = torch.zeros_like(v)
    x = _philox(v, zero, rid[None, :] + zero, zero + 0x494E4954, key)[0] >> 9
    classes = []
    for c in range(C):
        k = np.flatnonzero(colour == c)
        classes.append((torch.as_tensor(eu[k].astype(np.int64), device=dev),
                        torch.as_tensor(ev[k].astype(np.int64), device=dev),
                        torch.as_tensor(J[k].astype(np.int64), device=dev)[:, None]))
    hh = None if h is None else torch.as_tensor(h.astype(np.int64), device=dev)[:, None]
    tu, tv = (torch.as_tensor(a.astype(np.int64), device=dev) for a in (eu, ev))
    tJ = torch.as_tensor(J.astype(np.int64), device=dev)[:, None]
    a0 = math.floor(p.alpha0_deg / 360.0 * HALF + 0.5)
    win = round(p.dwt_window_deg / 360.0 * ONE)
    for t in range(1, S + 1):
        step = 2 * ((a0 * (S - t + 1) + S // 2) // S)
        if case["update"] == "full":
            d = torch.where((x[tu] - x[tv]) % ONE < HALF, step * tJ, -step * tJ)
            acc = torch.zeros_like(x)
            acc.index_add_(0, tu, -d)
            acc.index_add_(0, tv, d)
            x = (x + acc) % ONE
        else:
            for cu, cv, cJ in classes:
                xu, xv = x[cu], x[cv]
                d = torch.where((xu - xv) % ONE < HALF, step * cJ, -step * cJ)
                x[cu] = (xu - d) % ONE
                x[cv] = (xv + d) % ONE
            if hh is not None:
                x = (x - torch.where(x < HALF, step * hh, -step * hh)) % ONE
        if t % p.dwt_period == 0:
            z = torch.zeros_like(rid)
            w0, w1 = _philox(z, z + t, rid, z + 0x44575420, key)
            theta = w0 >> 9
            twist = int(round(2 * p.dwt_ratio)) * (step // 2)
            if hh is not None:
                twist = torch.where(w1 >> 31 > 0, -twist, twist)
            inside = (2 * x - 2 * theta + win) % ONE < 2 * win
            x = torch.where(inside, (x + twist) % ONE, x)
    w = -tJ[:, 0]
    if hh is not None:
        s = torch.where((x + ONE // 4) % ONE < HALF, 1, -1)
        H = -(tJ * s[tu] * s[tv]).sum(0) - (hh * s).sum(0)
    else:
        B, H, s = p.n_bisectors, None, None
        for q in range(B):
            beta = ((q << 23) + B) // (2 * B)
            sq = torch.where((x - beta) % ONE < HALF, 1, -1).to(torch.int8)
            Hq = -(tJ * (sq[tu] * sq[tv])).sum(0)
            if H is None:
                H, s = Hq, sq
            else:
                better = Hq < H
                H, s = torch.where(better, Hq, H), torch.where(better[None, :], sq, s)
    cut = (w[:, None] * (s[tu] != s[tv])).sum(0)
    return [H.cpu().numpy(), cut.cpu().numpy(), s.to(torch.int8).t().contiguous().cpu().numpy()]


def exact(case, seed):
    """32-bit phases under the grid schedule only (16-bit ones round by their own rules), and
    not where the plain form takes too long."""
    if (case["graph"] == "mixed" or case["storage"] not in ("fp32", "fix32")
            or case["readout"] != "bisectors"):
        return None
    n, m = _sizes(case["graph"], case["size"])
    seconds = case["sweeps"] * (3e-4 + 2e-11 * 8 * m * case["replicas"] * 4)
    if seconds > 12 or n * case["replicas"] > 1e8:
        return None
    return _exact_trial(case, seed)
