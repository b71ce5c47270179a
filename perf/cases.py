"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from a
seed, ``run`` takes them through the framework's public entry points once and
``exact`` computes the same outputs with plain torch/numpy in 64 bits.  Grids are
buses on a square lattice in a random numbering: a random spanning tree plus
chords between lattice neighbours, with the branch parameter ranges, bus kinds
and smooth planted voltages of the framework's own synthetic workloads.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_28203_amd as dpf

PV_SHARE = 1445 / 9241  # PV buses per bus
DEV = "cuda"


# ---------------------------------------------------------------- the cases


def listed():
    return [
        # the smallest solve: one operating point of a 14-bus grid from a flat start,
        # an interactive or embedded call whose latency and launches count
        {"name": "solve-14x1", "kind": "solve", "n": 14, "branches": 20, "B": 1, "iters": 100, "start": "flat",
         "outage": False, "numbering": "file", "kernel": "default", "opt": "adam", "sched": "constant", "lr": 1e-2,
         "resume": False},
        # a batch of load scenarios on a mid-size transmission grid from flat starts
        {"name": "solve-1354x64", "kind": "solve", "n": 1354, "branches": 1991, "B": 64, "iters": 200,
         "start": "flat", "outage": False, "numbering": "rcm", "kernel": "default", "opt": "adam",
         "sched": "constant", "lr": 1e-3, "resume": False},
        # scenarios on a larger grid as its file numbers it, default routing, solved in
        # chunks: optimizer and schedule state come in and go out with the call
        {"name": "solve-3000x256", "kind": "solve", "n": 3000, "branches": 4500, "B": 256, "iters": 60,
         "start": "warm", "outage": False, "numbering": "file", "kernel": "default", "opt": "adam",
         "sched": "plateau", "lr": 1e-4, "resume": True},
        # the framework's main workload: 1024 outages of a 9241-bus grid sharing one
        # matrix, warm-started, in the numbering and with the kernel meant for it
        {"name": "outages-9241x1024", "kind": "solve", "n": 9241, "branches": 16049, "B": 1024, "iters": 60,
         "start": "warm", "outage": True, "numbering": "rcm", "kernel": "banded", "opt": "adam", "sched": "plateau",
         "lr": 1e-4, "resume": False},
        # one operating point of a 9241-bus grid: the latency of a single large solve
        {"name": "solve-9241x1", "kind": "solve", "n": 9241, "branches": 16049, "B": 1, "iters": 100,
         "start": "warm", "outage": False, "numbering": "rcm", "kernel": "default", "opt": "adam",
         "sched": "constant", "lr": 1e-4, "resume": False},
        # a day's time series, solved in warm-started windows of 16 steps
        {"name": "series-9241x32", "kind": "series", "n": 9241, "branches": 16049, "T": 32, "window": 16,
         "iters": 40, "numbering": "rcm", "lr": 1e-4},
        # a collection of grids of very different sizes, solved in one call
        {"name": "collection-48", "kind": "collection", "grids": 48, "lo": 100, "hi": 40000, "pick": 1, "iters": 30,
         "lr": 1e-4},
        # the residual, loss and gradient of every outage of a screening batch, for a
        # user's own optimizer or ranking (the largest evaluation)
        {"name": "evaluate-9241x256", "kind": "evaluate", "n": 9241, "branches": 16049, "B": 256, "outage": True,
         "numbering": "rcm", "shared_s": True, "want_dS": True, "want_grad": True},
        # the loss as a term of a torch model, forward and backward through autograd, on
        # a small grid: what a training step pays per call
        {"name": "autograd-118x8", "kind": "autograd", "n": 118, "branches": 186, "B": 8, "outage": False,
         "numbering": "file", "shared_s": False},
        # gradients with respect to branch parameters and injections (identification)
        {"name": "parameters-1354x64", "kind": "parameters", "n": 1354, "branches": 1991, "B": 64, "outage": False,
         "numbering": "file", "shared_s": False},
        # DC angles as the start points of a batch
        {"name": "dc-1354x64", "kind": "dc", "n": 1354, "branches": 1991, "B": 64, "outage": True,
         "numbering": "file"},
        # the admittance matrix of a large grid from its branch list
        {"name": "ybus-9241", "kind": "ybus", "n": 9241, "branches": 16049, "parallel": 0.02, "noalloc": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _branches(rng, n):
    return max(n, int(round(rng.uniform(1.35, 1.75) * n)))


# bus-iterations of the largest listed solve
_MOST = 9241 * 1024 * 60


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["series", "collection", "evaluate", "evaluate", "autograd", "parameters", "dc",
                                       "ybus"])
    if kind == "solve":
        n = _log_int(rng, 14, 9241)
        iters = _log_int(rng, 20, 200)
        B = _log_int(rng, 1, max(1, min(1024, _MOST // (n * iters))))
        opt = rng.choice(["adam"] * 4 + ["rmsprop", "sgd"])
        numbering = rng.choice(["file", "rcm"])
        banded = n > 1000 and numbering == "rcm" and rng.random() < 0.5
        flat = n <= 2000 and rng.random() < 0.5
        return {"kind": kind, "n": n, "branches": _branches(rng, n), "B": B, "iters": iters,
                "start": "flat" if flat else "warm", "outage": rng.random() < 0.4, "numbering": numbering,
                "kernel": "banded" if banded else "default", "opt": opt,
                "sched": rng.choice(["constant", "plateau", "step"]),
                "lr": 1e-2 if opt == "sgd" else 1e-3 if flat else 1e-4, "resume": rng.random() < 0.3}
    if kind == "series":
        n = _log_int(rng, 118, 9241)
        window = rng.choice([1, 2, 5, 16, 24])
        return {"kind": kind, "n": n, "branches": _branches(rng, n), "T": min(48, window * rng.randint(1, 3)),
                "window": window, "iters": _log_int(rng, 10, 40), "numbering": rng.choice(["file", "rcm"]),
                "lr": 1e-4}
    if kind == "collection":
        lo = _log_int(rng, 30, 300)
        return {"kind": kind, "grids": _log_int(rng, 2, 48), "lo": lo, "hi": _log_int(rng, 4 * lo, 40000),
                "pick": rng.randint(1, 1 << 20), "iters": _log_int(rng, 10, 60), "lr": 1e-4}
    if kind == "ybus":
        n = _log_int(rng, 14, 200000)
        return {"kind": kind, "n": n, "branches": _branches(rng, n), "parallel": rng.choice([0.0, 0.02, 0.2]),
                "noalloc": rng.random() < 0.4}
    if kind == "dc":
        n = _log_int(rng, 14, 3000)
        return {"kind": kind, "n": n, "branches": _branches(rng, n), "B": _log_int(rng, 1, 256),
                "outage": rng.random() < 0.5, "numbering": rng.choice(["file", "rcm"])}
    n = _log_int(rng, 14, 20000)
    B = _log_int(rng, 1, max(1, min(1024, 9241 * 512 // n)))
    case = {"kind": kind, "n": n, "branches": _branches(rng, n), "B": B, "outage": rng.random() < 0.5,
            "numbering": rng.choice(["file", "rcm"]), "shared_s": rng.random() < 0.5}
    if kind == "evaluate":
        case["want_dS"] = rng.random() < 0.5
        case["want_grad"] = not case["want_dS"] or rng.random() < 0.7
    return case


# ---------------------------------------------------------------- inputs


def _lattice(rng, n, n_branch):
    """(from, to, chord, x, y): a random spanning tree of the lattice and chords, buses in
    lattice order; chord marks the branches whose removal leaves the grid connected."""
    w = max(2, int(math.ceil(math.sqrt(n))))
    k = np.arange(1, n, dtype=np.int64)
    row, col = k // w, k % w
    left = (col > 0) & ((row == 0) | (rng.random(n - 1) < 0.5))
    parent = np.where(left, k - 1, k - w)
    other = np.where(left, k - w, k - 1)
    ok = np.where(left, row > 0, (row > 0) & (col > 0))
    diag = (row > 0) & (col > 0)
    anti = (row > 0) & (col < w - 1)
    cf = np.concatenate([other[ok], (k - w - 1)[diag], (k - w + 1)[anti]])
    ct = np.concatenate([k[ok], k[diag], k[anti]])
    m = min(max(0, n_branch - (n - 1)), len(cf))
    pick = rng.choice(len(cf), size=m, replace=False)
    f = np.concatenate([parent, cf[pick]])
    t = np.concatenate([k, ct[pick]])
    chord = np.arange(len(f)) >= n - 1
    p = rng.permutation(len(f))
    pos = np.arange(n)
    return f[p], t[p], chord[p], (pos % w) / w, (pos // w) / w


def _field(rng, x, y):
    """A smooth field in [-1, 1] over the positions."""
    v = np.zeros(len(x))
    for _ in range(4):
        a, b = rng.uniform(-2.5, 2.5, size=2)
        v += rng.uniform(0.3, 1.0) * np.cos(2 * np.pi * (a * x + b * y + rng.random()))
    return v / max(1e-9, np.abs(v).max())


def _grid(rng, n, n_branch, numbering, parallel=0.0):
    f, t, chord, x, y = _lattice(rng, n, n_branch)
    if parallel:
        twin = rng.integers(0, len(f), size=int(round(parallel * len(f))))
        f, t, chord = np.concatenate([f, f[twin]]), np.concatenate([t, t[twin]]), np.concatenate([chord, chord[twin]])
    nb = len(f)
    perm = rng.permutation(n)  # bus k of the lattice is bus perm[k] of the file
    f, t = perm[f], perm[t]
    vm, va = np.empty(n), np.empty(n)
    vm[perm] = 1.0 + 0.05 * _field(rng, x, y)
    va[perm] = 0.2 * _field(rng, x, y)
    kinds = rng.permutation(n)
    bt = np.zeros(n, dtype=np.int8)
    bt[kinds[0]] = dpf.SLACK
    bt[kinds[1:1 + int(round(PV_SHARE * n))]] = dpf.PV
    va -= va[kinds[0]]
    g = {"n": n, "f": f, "t": t, "r": rng.uniform(0.01, 0.1, nb), "x": rng.uniform(0.05, 0.3, nb),
         "b": rng.uniform(0.0, 0.05, nb), "bt": bt, "vm": vm, "va": va, "chord": np.flatnonzero(chord)}
    return _renumber(g, None, 0) if numbering == "rcm" else g


def _renumber(g, offsets, group):
    """The grid in the framework's small-bandwidth numbering, rows of similar degree
    grouped as far as the banded kernels' block of 4096 buses allows (one grid), or in
    windows of ``group``."""
    for w in ((group,) if group else (2560, 1536, 1024, 512, 256)):
        perm, bw = dpf.rcm_order(g["n"], g["f"], g["t"], sub_offset=offsets, group=w)
        if bw <= 4096 or offsets is not None:
            break
    inv = np.empty(g["n"], dtype=np.int64)
    inv[perm] = np.arange(g["n"])
    return dict(g, f=inv[g["f"]], t=inv[g["t"]], bt=g["bt"][perm], vm=g["vm"][perm], va=g["va"][perm])


def _injections(g):
    """S = V conj(Y V) at the planted voltages, from the branch flows."""
    V = g["vm"] * np.exp(1j * g["va"])
    y, ysh = 1.0 / (g["r"] + 1j * g["x"]), 0.5j * g["b"]
    vf, vt = V[g["f"]], V[g["t"]]
    i_f, i_t = (y + ysh) * vf - y * vt, (y + ysh) * vt - y * vf
    cur = np.zeros(g["n"], dtype=np.complex128)
    for end, i in ((g["f"], i_f), (g["t"], i_t)):
        cur += np.bincount(end, i.real, g["n"]) + 1j * np.bincount(end, i.imag, g["n"])
    return V * np.conj(cur)


def _gpu(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device=DEV, dtype=dtype)


def _case_grid(case, rng):
    if case["kind"] != "collection":
        return _grid(rng, case["n"], case["branches"], case.get("numbering", "file"), case.get("parallel", 0.0)), None
    pick = np.random.default_rng(case["pick"])
    sizes = np.exp(pick.uniform(np.log(case["lo"]), np.log(case["hi"]), case["grids"])).astype(np.int64)
    sizes = np.sort(sizes)[::-1]
    parts = [_grid(rng, int(n), int(round(1.4 * n)), "file") for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    g = {k: np.concatenate([p[k] for p in parts]) for k in ("r", "x", "b", "bt", "vm", "va")}
    g.update(n=int(off[-1]), chord=np.zeros(0, dtype=np.int64),
             f=np.concatenate([p["f"] + o for p, o in zip(parts, off)]),
             t=np.concatenate([p["t"] + o for p, o in zip(parts, off)]))
    return _renumber(g, off, 1536), off


def _inputs(case, seed):
    """The inputs of a case as a dict: the grid (numpy), and on the GPU the bus kinds,
    the injections ([n] shared or [B, n]), the start voltages [B, n] and the outages."""
    rng = np.random.default_rng(seed)
    g, off = _case_grid(case, rng)
    n, kind = g["n"], case["kind"]
    B = case.get("B", case.get("T", 1))
    d = {"g": g, "off": off, "B": B}
    if kind == "ybus":
        return d
    S = _gpu(_injections(g), torch.complex128)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))

    def spread(rows, by):
        return 1.0 + by * (2.0 * torch.rand(rows, n, generator=gen, dtype=torch.float64, device=DEV) - 1.0)

    flat = case.get("start") == "flat"
    shared = case.get("shared_s", kind == "dc" or (kind == "solve" and case["outage"]))
    # loads and generation move by up to 10% of a flat start's base, 2% of a warm one's
    d["s"] = (S * spread(1 if shared else B, 0.1 if flat else 0.02)).contiguous()
    if shared:
        d["s"] = d["s"][0].contiguous()
    d["bt"] = _gpu(g["bt"], torch.int8)
    vm, va = _gpu(g["vm"], torch.float64), _gpu(g["va"], torch.float64)
    if flat:
        vm, va = torch.where(d["bt"] == dpf.PQ, torch.ones_like(vm), vm), torch.zeros_like(va)
    rows = 1 if kind == "series" else B
    d["vm"], d["va"] = vm.expand(rows, n).contiguous(), va.expand(rows, n).contiguous()
    if kind in ("evaluate", "autograd", "parameters"):
        d["vm"] = d["vm"] * spread(B, 0.01)
        d["va"] = d["va"] + spread(B, 0.01) - 1.0
    if case.get("outage") and len(g["chord"]):
        d["outage"] = _gpu(g["chord"][rng.integers(0, len(g["chord"]), size=B)], torch.int32)
    else:
        d["outage"] = None
    return d


def _options(case):
    flat = case.get("start") == "flat"
    sched = {"constant": dpf.SCHED_CONSTANT, "plateau": dpf.SCHED_PLATEAU, "step": dpf.SCHED_STEP}[
        case.get("sched", "constant")]
    opt = {"adam": dpf.OPT_ADAM, "rmsprop": dpf.OPT_RMSPROP, "sgd": dpf.OPT_SGD}[case.get("opt", "adam")]
    b1, b2, eps = (0.9, 0.999, 1e-8) if flat else (0.995, 0.995, 1e-14)
    if opt == dpf.OPT_SGD:
        b1 = 0.9
    return dpf.Options(lr=case["lr"], beta1=b1, beta2=b2, eps=eps, tol=1e-6, max_iter=case["iters"], sched=sched,
                       factor=0.5, patience=25, threshold=1e-3, optimizer=opt)


def prepare(case, seed):
    d = _inputs(case, seed)
    g, kind = d["g"], case["kind"]
    nb = [_gpu(g[k], torch.int32) for k in ("f", "t")] + [_gpu(g[k], torch.float64) for k in ("r", "x", "b")]
    if kind == "ybus":
        return {"case": case, "n": g["n"], "branches": nb}
    if kind == "dc":
        grid = dpf.build_dc_grid(g["n"], g["f"], g["t"], g["x"])
    else:
        grid = dpf.build_ybus(g["n"], *nb)
    st = {"case": case, "grid": grid, "bt": d["bt"], "s": d["s"], "outage": d["outage"], "vm0": d["vm"], "va0": d["va"]}
    if kind in ("solve", "collection"):
        st["v0"] = torch.stack([d["vm"], d["va"]])
        st["v"] = st["v0"].clone()
        st["ws"], st["opts"] = dpf.SolveWorkspace(), _options(case)
        if d["off"] is not None:
            st["off"], st["off_dev"] = d["off"].tolist(), _gpu(d["off"], torch.int32)
        if case.get("kernel") == "banded":
            st["route"] = dpf.Route(variant=next(v["index"] for v in dpf.variants() if v["kind"] == "banded-pair"
                                                 and v["threads"] * v["buses_per_thread"] >= min(g["n"], 4096)))
        if case.get("resume"):
            B = case["B"]
            st["m0"] = torch.zeros(4, B, g["n"], dtype=torch.float64, device=DEV)
            st["q0"] = dpf.fresh_sched_state(B, case["lr"])
            st["m"], st["q"] = st["m0"].clone(), st["q0"].clone()
    elif kind == "series":
        st["ws"], st["opts"] = dpf.SolveWorkspace(), _options(case)
        st["vm0"], st["va0"] = d["vm"][0].contiguous(), d["va"][0].contiguous()
    elif kind == "autograd":
        st["vm0"].requires_grad_(True)
        st["va0"].requires_grad_(True)
    elif kind == "dc":
        st["va"] = torch.zeros_like(d["va"])
    return st


# ---------------------------------------------------------------- one pass


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "ybus":
        y = dpf.build_ybus(st["n"], *st["branches"], noalloc=case["noalloc"])
        return {"row_ptr": y.row_ptr, "col_idx": y.col_idx, "val": y.val, "nnz": y.nnz, "max_row_nnz": y.max_row_nnz}
    if kind in ("solve", "collection"):
        v = st["v"]
        v.copy_(st["v0"])
        if "m" in st:
            st["m"].copy_(st["m0"])
            st["q"].copy_(st["q0"])
        r = dpf.solve(st["grid"], st["bt"], st["s"], v[0], v[1], opts=st["opts"], outage=st["outage"],
                      sub_offset=st.get("off"), sub_offset_dev=st.get("off_dev"), adam_state=st.get("m"),
                      sched_state=st.get("q"), workspace=st["ws"], route=st.get("route"))
        out = {k: r[k] for k in ("iters", "status", "max_mis", "loss")}
        out.update(vm=v[0], va=v[1])
        if "m" in st:
            out.update(moments=st["m"], schedule=st["q"])
        return out
    if kind == "series":
        r = dpf.solve_series(st["grid"], st["bt"], st["s"], st["vm0"], st["va0"], window=case["window"],
                             opts=st["opts"], workspace=st["ws"])
        return {k: r[k] for k in ("vm", "va", "iters", "status", "max_mis", "loss")}
    if kind == "evaluate":
        r = dpf.mismatch_grad(st["grid"], st["bt"], st["s"], st["vm0"], st["va0"], outage=st["outage"],
                              want_dS=case["want_dS"], want_grad=case["want_grad"])
        return {k: v for k, v in r.items() if v is not None}
    if kind == "autograd":
        loss, mx = dpf.DPFLoss.apply(st["vm0"], st["va0"], st["grid"], st["bt"], st["s"], st["outage"])
        gv, ga = torch.autograd.grad(loss.sum(), (st["vm0"], st["va0"]))
        return {"loss": loss, "max_mis": mx, "g_vm": gv, "g_va": ga}
    if kind == "parameters":
        return dpf.param_grad(st["grid"], st["bt"], st["s"], st["vm0"], st["va0"], outage=st["outage"])
    # DC angles to the default accuracy; how many conjugate gradient steps that took and the
    # residual they ended at are rounding-level properties of the way there, not results
    st["va"].zero_()
    dpf.dc_init(st["grid"], st["bt"], st["s"], st["va"], outage=st["outage"])
    return {"va": st["va"]}


# ---------------------------------------------------------------- what a pass cannot do without


def _sizes(case):
    if case["kind"] == "collection":
        pick = np.random.default_rng(case["pick"])
        n = int(np.exp(pick.uniform(np.log(case["lo"]), np.log(case["hi"]), case["grids"])).astype(np.int64).sum())
        return n, int(round(1.4 * n))
    return case["n"], case["branches"] + int(round(case.get("parallel", 0.0) * case["branches"]))


def work(case):
    n, nb = _sizes(case)
    nnz = n + 2 * nb
    kind, B = case["kind"], case.get("B", case.get("T", 1))
    matrix = 20 * nnz + 4 * n
    if kind == "ybus":
        return {"bytes": 32 * nb + matrix, "flops": 20 * nb}
    s = 16 * n * (B if not case.get("shared_s", kind == "dc" or (kind == "solve" and case["outage"])) else 1)
    if kind in ("solve", "collection", "series"):
        # start and result once, and per iteration two products and about 150 operations a bus
        state = 80 * n * B if case.get("resume") else 0
        return {"bytes": 32 * n * B + s + matrix + state, "flops": case["iters"] * B * (16 * nnz + 150 * n)}
    if kind == "dc":
        return {"bytes": 8 * n * B + s + matrix, "flops": B * 4 * nnz}
    if kind == "parameters":
        return {"bytes": 16 * n * B + s + matrix + 40 * nb + 24 * nb * B + 16 * n * B,
                "flops": B * (8 * nnz + 100 * n + 40 * nb)}
    out = (16 * n * B if case.get("want_dS") else 0) + (16 * n * B if case.get("want_grad", True) else 0)
    return {"bytes": 16 * n * B + s + matrix + out, "flops": B * (16 * nnz + 100 * n)}


# ---------------------------------------------------------------- the same in 64 bits


class _Plain:
    """Plain torch arithmetic of a case's grid: products with Y, residuals, gradients."""

    def __init__(self, d):
        g = d["g"]
        n, f, t = g["n"], g["f"], g["t"]
        y, ysh = 1.0 / (g["r"] + 1j * g["x"]), 0.5j * g["b"]
        diag = np.zeros(n, dtype=np.complex128)
        np.add.at(diag, f, y + ysh)
        np.add.at(diag, t, y + ysh)
        row, col, val = np.concatenate([f, t]), np.concatenate([t, f]), np.concatenate([-y, -y])
        order = np.argsort(row, kind="stable")
        row, col, val = row[order], col[order], val[order]
        at = np.arange(len(row)) - np.searchsorted(row, row)
        cols = np.tile(np.arange(n)[:, None], (1, int(at.max(initial=0)) + 1))
        vals = np.zeros(cols.shape, dtype=np.complex128)
        cols[row, at], vals[row, at] = col, val
        self.diag = _gpu(diag, torch.complex128)
        self.cols = [_gpu(c, torch.int64) for c in cols.T]
        self.vals = [_gpu(v, torch.complex128) for v in vals.T]
        self.y, self.yd = _gpu(y, torch.complex128), _gpu(y + ysh, torch.complex128)
        self.f, self.t = _gpu(f, torch.int64), _gpu(t, torch.int64)
        self.d, self.n, self.B = d, n, d["B"]
        self.s, self.out = d.get("s"), d.get("outage")
        self.seg = None
        if d["off"] is not None:
            self.seg = _gpu(np.repeat(np.arange(len(d["off"]) - 1), np.diff(d["off"])), torch.int64)
        bt = d["bt"]
        self.pq, self.free = bt == dpf.PQ, bt != dpf.SLACK
        self.m = self.total((self.pq.double() + self.free.double())[None])

    def total(self, x):
        """Sums over each item: [B, n] -> [B, items of a case]."""
        if self.seg is None:
            return x.sum(1, keepdim=True)
        return torch.zeros(x.shape[0], int(self.seg[-1]) + 1, dtype=x.dtype, device=DEV).index_add_(1, self.seg, x)

    def largest(self, x):
        if self.seg is None:
            return x.max(1, keepdim=True).values
        z = torch.zeros(x.shape[0], int(self.seg[-1]) + 1, dtype=x.dtype, device=DEV)
        return z.index_reduce_(1, self.seg, x, "amax")

    def bus(self, x):
        """An item's value at each of its buses."""
        return x if self.seg is None else x[:, self.seg]

    def times(self, z):
        acc = self.diag * z
        for c, v in zip(self.cols, self.vals):
            acc += v * z[:, c]
        if self.out is not None:
            k = self.out.long()
            at = torch.arange(z.shape[0], device=DEV)
            f, t, y, yd = self.f[k], self.t[k], self.y[k], self.yd[k]
            zf, zt = z[at, f], z[at, t]
            acc[at, f] -= yd * zf - y * zt
            acc[at, t] -= yd * zt - y * zf
        return acc

    def forward(self, vm, va, s):
        V = torch.polar(vm, va)
        cur = self.times(V)
        dS = V * cur.conj() - s
        rP, rQ = dS.real * self.free, dS.imag * self.pq
        loss = self.total(rP * rP + rQ * rQ) / self.m
        a = torch.complex(rP, rQ) * (2.0 / self.bus(self.m))
        return V, cur, dS, a, loss, self.largest(torch.maximum(rP.abs(), rQ.abs()))

    def gradient(self, V, cur, a, vm):
        G = a * cur + self.times(a * V.conj()).conj()
        z = G.conj() * V
        return z.real / vm * self.pq, -z.imag * self.free

    def solve(self, vm, va, s, o, m, q):
        """vm, va, moments m [4, B, n] and schedule rows q [B, items, 6] after up to max_iter updates."""
        iters = torch.zeros(q.shape[:2], dtype=torch.int32, device=DEV)
        live = torch.ones(q.shape[:2], dtype=torch.bool, device=DEV)
        pq, free = self.pq[None], self.free[None]
        for it in range(o.max_iter + 1):
            V, cur, _, a, l2, mu = self.forward(vm, va, s)
            live &= mu >= o.tol
            if it == o.max_iter or not bool(live.any()):
                break
            gv, ga = self.gradient(V, cur, a, vm)
            q[..., 0] += live
            q[..., 4] = torch.where(live, q[..., 4] * o.beta1, q[..., 4])
            q[..., 5] = torch.where(live, q[..., 5] * o.beta2, q[..., 5])
            lr, c1, c2 = self.bus(q[..., 1]), self.bus(1 - q[..., 4]), self.bus(1 - q[..., 5])
            go = self.bus(live)
            for x, grad, j, mask in ((vm, gv, 0, pq & go), (va, ga, 1, free & go)):
                m1, m2 = m[j], m[2 + j]
                if o.optimizer == dpf.OPT_SGD:
                    n1, n2 = o.beta1 * m1 + grad, m2
                    step = lr * n1
                elif o.optimizer == dpf.OPT_RMSPROP:
                    n1, n2 = m1, o.beta2 * m2 + (1 - o.beta2) * grad * grad
                    step = lr * grad / (n2.sqrt() + o.eps)
                else:
                    n1, n2 = o.beta1 * m1 + (1 - o.beta1) * grad, o.beta2 * m2 + (1 - o.beta2) * grad * grad
                    step = lr * (n1 / c1) / ((n2 / c2).sqrt() + o.eps)
                x.copy_(torch.where(mask, x - step, x))
                m1.copy_(torch.where(mask, n1, m1))
                m2.copy_(torch.where(mask, n2, m2))
            if o.sched == dpf.SCHED_PLATEAU:
                better = l2 < q[..., 2] * (1 - o.threshold)
                bad = torch.where(better, 0.0, q[..., 3] + 1)
                cut = bad > o.patience
                lower = q[..., 1] * o.factor
                q[..., 2] = torch.where(live & better, l2, q[..., 2])
                q[..., 3] = torch.where(live, torch.where(cut, 0.0, bad), q[..., 3])
                q[..., 1] = torch.where(live & cut & (q[..., 1] - lower > o.sched_eps), lower, q[..., 1])
            elif o.sched == dpf.SCHED_STEP:
                q[..., 1] = torch.where(live & (q[..., 0] % o.patience == 0), q[..., 1] * o.factor, q[..., 1])
            iters += live
        status = torch.where(mu < o.tol, 0, 1).to(torch.int32)
        return {"iters": iters.reshape(-1), "status": status.reshape(-1), "max_mis": mu.reshape(-1),
                "loss": l2.reshape(-1), "vm": vm, "va": va}


def _exact_ybus(d):
    g = d["g"]
    n, f, t = g["n"], g["f"], g["t"]
    y, ysh = 1.0 / (g["r"] + 1j * g["x"]), 0.5j * g["b"]
    k = np.arange(n)
    key = np.concatenate([k * n + k, f * n + f, t * n + t, f * n + t, t * n + f])
    val = np.concatenate([np.zeros(n), y + ysh, y + ysh, -y, -y])
    u, at = np.unique(key, return_inverse=True)
    v = np.bincount(at, val.real, len(u)) + 1j * np.bincount(at, val.imag, len(u))
    row_ptr = np.searchsorted(u // n, np.arange(n + 1)).astype(np.int32)
    return {"row_ptr": torch.as_tensor(row_ptr), "col_idx": torch.as_tensor((u % n).astype(np.int32)),
            "val": torch.as_tensor(v), "nnz": len(u), "max_row_nnz": int(np.diff(row_ptr).max())}


def _exact_dc(d):
    g = d["g"]
    n, f, t, w = g["n"], g["f"], g["t"], 1.0 / g["x"]
    lap = np.zeros((n, n))
    for i, j, v in ((f, f, w), (t, t, w), (f, t, -w), (t, f, -w)):
        np.add.at(lap, (i, j), v)
    keep = np.flatnonzero(g["bt"] != dpf.SLACK)
    at = np.full(n, -1)
    at[keep] = np.arange(n - 1)
    P = d["s"].cpu().numpy().real
    P = np.broadcast_to(P, (d["B"], n))[:, keep].T
    cols = [P[:, :1] if d["s"].dim() == 1 else P]
    out = None if d["outage"] is None else d["outage"].cpu().numpy()
    if out is not None:
        e = np.zeros((n - 1, d["B"]))
        for c, k in enumerate(out):
            for bus, sign in ((f[k], 1.0), (t[k], -1.0)):
                if at[bus] >= 0:
                    e[at[bus], c] += sign
        cols.append(e)
    sol = np.linalg.solve(lap[np.ix_(keep, keep)], np.concatenate(cols, 1))
    theta = np.broadcast_to(sol[:, :cols[0].shape[1]], (n - 1, d["B"])).copy()
    if out is not None:  # the matrix without the branch, by its rank-1 inverse update
        u = sol[:, cols[0].shape[1]:]
        theta += u * (w[out] * (e * theta).sum(0) / (1.0 - w[out] * (e * u).sum(0)))
    va = np.zeros((d["B"], n))
    va[:, keep] = theta.T
    return {"va": torch.as_tensor(va)}


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "ybus":
        return _exact_ybus(d)
    if kind == "dc":
        return _exact_dc(d)
    p = _Plain(d)
    n, B = p.n, p.B
    if kind in ("solve", "collection"):
        items = p.m.shape[1]
        m = torch.zeros(4, B, n, dtype=torch.float64, device=DEV)
        q = dpf.fresh_sched_state(B * items, case["lr"]).reshape(B, items, 6)
        out = p.solve(d["vm"].clone(), d["va"].clone(), p.s, _options(case), m, q)
        if case.get("resume"):
            out.update(moments=m, schedule=q.reshape(-1, 6))
        return out
    if kind == "series":
        parts, vm, va = [], d["vm"], d["va"]
        for t0 in range(0, case["T"], case["window"]):
            s = p.s[t0:t0 + case["window"]]
            k = s.shape[0]
            r = p.solve(vm.expand(k, n).clone(), va.expand(k, n).clone(), s, _options(case),
                        torch.zeros(4, k, n, dtype=torch.float64, device=DEV),
                        dpf.fresh_sched_state(k, case["lr"]).reshape(k, 1, 6))
            vm, va = r["vm"][-1:], r["va"][-1:]
            parts.append(r)
        return {k: torch.cat([r[k] for r in parts]) for k in parts[0]}
    V, cur, dS, a, loss, mu = p.forward(d["vm"], d["va"], p.s)
    out = {"loss": loss[:, 0], "max_mis": mu[:, 0]}
    if kind in ("evaluate", "autograd"):
        if case.get("want_dS"):
            out["dS"] = dS
        if case.get("want_grad", True):
            out["g_vm"], out["g_va"] = p.gradient(V, cur, a, d["vm"])
        return out
    w = a * V.conj()
    f, t = p.f, p.t
    y2D = p.y * p.y * (w[:, f] - w[:, t]) * (V[:, f] - V[:, t])
    gb = -0.5 * (w[:, f] * V[:, f] + w[:, t] * V[:, t]).imag
    grads = {"g_r": -y2D.real, "g_x": y2D.imag, "g_b": gb}
    if p.out is not None:
        for v in grads.values():
            v[torch.arange(B, device=DEV), p.out.long()] = 0.0
    return dict(out, g_s=-a, **grads)
