"""Performance cases of the grain-envelope framework.

Each case is a piece of work that a program using the library has it do, driven
through the public binding (`Context`, `Batch`, the adjoint calls):

* ``grain``     one grain in a uniform melt, a 1 mm cube: step calls and the
                particles afterwards (the single-grain workload, its nucleus).
* ``columnar``  directional competitive growth in a linear field, optionally
                with periodic lateral faces or non-integer kinetic exponents: a
                window of steps from a grown state, then the grain map.
* ``equiaxed``  growth under the moving point source with nucleation (the
                columnar-to-equiaxed workload, or its scaled form, optionally
                with melting or periodic faces): a window of steps, then the
                deposition counts and the site states.
* ``coupled``   the inner loop of a coupled solver: hand over temperature and
                solute (device arrays), take a few steps, read the mushy-zone
                fraction.
* ``output``    the output step of a run: the grain map on a voxel grid and
                the particles of a window.
* ``regrid``    a coupled solver changes its mesh: the deposition grid is set
                anew (every reached site is counted) and the fraction read.
* ``adjoint``   gradient of the final positions: recorded forward and reverse
                sweep, or the reverse sweep alone (one more loss on a run).
* ``batch``     realisations of uneven size advanced together.

A pass that advances a state starts from the same state every time: the
program owns the device workspace of a context (or batch), keeps a copy of it
and copies it back before it steps, as a parameter study or a time-step
control does.  Steps per pass are whole re-sort intervals (16 steps), so the
context's step count and that of the restored state stay in phase.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2504_12858_amd import binding as B
from paper_2504_12858_amd import workloads as W

R = 16  # steps between re-sorts of the stopped store (the library's default)
DEV = "cuda:0"


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # The smallest calls: a nucleus stepped one call at a time with its
        # counters read back, as a program that watches every step does.
        {"name": "nucleus_calls", "kind": "grain", "shell": 0, "steps": 16, "per_call": 1},
        # The single-grain workload (shell 50, about 200 steps): ordinary
        # stepping of a small state, bound by launches and latency.
        {"name": "single_grain", "kind": "grain", "shell": 50, "steps": 208, "per_call": 208},
        # The scaled directional run with periodic lateral faces.
        {"name": "columnar_small_periodic", "kind": "columnar", "size": 0.3, "grains": 8,
         "cells": 1, "dt": 5e-4, "pre": 192, "steps": 64, "periodic": 3, "power": False, "map": 60},
        # The directional workload at its stated size (2 x 2 x 4 mm, 64
        # grains, about 2M stored particles).
        {"name": "columnar_full", "kind": "columnar", "size": 2.0, "grains": 64, "cells": 1,
         "dt": 5e-5, "pre": 2000, "steps": 192, "periodic": 0, "power": False, "map": 100},
        # The scaled moving-source run whose melt pool re-melts the grains.
        {"name": "equiaxed_small_melting", "kind": "equiaxed", "scaled": True, "size": 0.4,
         "lam": 4.0, "grid": 24, "pre": 240, "steps": 64, "periodic": 0, "melting": True},
        # The moving-source workload in half of its volume, about 13M active
        # particles: the largest states that are stepped.
        {"name": "equiaxed_large", "kind": "equiaxed", "scaled": False, "size": 3.2, "lam": 1.0,
         "grid": 256, "pre": 960, "steps": 96, "periodic": 0, "melting": False},
        # A coupled solver's loop on a 96 x 96 x 192 mesh, four steps of
        # growth for each of its own.
        {"name": "coupled_solute", "kind": "coupled", "size": 1.0, "grains": 32, "grid": 96,
         "pre": 320, "handovers": 8, "per_handover": 4},
        # The output step of a moving-source run with some hundred grains.
        {"name": "output_equiaxed", "kind": "output", "family": "equiaxed", "size": 3.0,
         "lam": 2.0, "grid": 128, "pre": 480, "map": 400, "window": 0.25},
        # A new mesh of the coupled solver on such a state.
        {"name": "regrid_equiaxed", "kind": "regrid", "family": "equiaxed", "size": 3.0,
         "lam": 2.0, "grid": 128, "pre": 480, "nodes": 120},
        # Gradient evaluation of a calibration: 16 grains that grow into each
        # other, recorded forward and reverse sweep.
        {"name": "adjoint_contacts", "kind": "adjoint", "grains": 16, "shell": 60,
         "field": "linear", "steps": 192, "ckpt": 50, "whole": True},
        # Another loss on the recorded run of 518 402 particles in a field on
        # a node grid, 500 steps: the reverse sweep alone.
        {"name": "gradient_grid", "kind": "adjoint", "grains": 1, "shell": 360, "field": "grid",
         "steps": 500, "ckpt": 50, "whole": False},
        # Realisations of uneven size in one batch.
        {"name": "batch_uneven", "kind": "batch", "members": 32, "size": 1.0, "pre": 640,
         "steps": 96},
    ]


def _log(rng, lo, hi):
    return float(lo * (hi / lo) ** rng.random())


def _whole(rng, lo, hi):
    return int(round(_log(rng, lo, hi)))


def _intervals(rng, lo, hi):
    return R * max(1, int(round(_log(rng, lo, hi) / R)))


def draw(rng):
    kind = rng.choice(["grain", "columnar", "equiaxed", "coupled", "output", "regrid", "adjoint",
                       "batch"])
    if kind == "grain":
        steps = _intervals(rng, 16, 208)
        return {"kind": kind, "shell": int(_log(rng, 1, 80)) - (1 if rng.random() < 0.2 else 0),
                "steps": steps, "per_call": rng.choice([1, steps, R])}
    if kind == "columnar":
        dt = rng.choice([5e-4, 2e-4, 5e-5])
        lo, hi = {5e-4: (64, 256), 2e-4: (128, 560), 5e-5: (320, 1600)}[dt]
        return {"kind": kind, "size": round(_log(rng, 0.2, 2.0), 3), "grains": _whole(rng, 3, 64),
                "cells": rng.choice([1, 2]), "dt": dt, "pre": _intervals(rng, lo, hi),
                "steps": _intervals(rng, 32, 96), "periodic": rng.choice([0, 0, 1, 3]),
                "power": rng.random() < 0.25, "map": _whole(rng, 20, 100)}
    if kind == "equiaxed":
        if rng.random() < 0.4:
            return {"kind": kind, "scaled": True, "size": round(_log(rng, 0.2, 0.8), 3), "lam": 4.0,
                    "grid": _whole(rng, 17, 49), "pre": _intervals(rng, 160, 256),
                    "steps": _intervals(rng, 32, 64), "periodic": rng.choice([0, 3]),
                    "melting": rng.random() < 0.6}
        lam = round(_log(rng, 1.0, 3.0), 2)
        return {"kind": kind, "scaled": False, "size": round(_log(rng, 0.6, 3.0), 3), "lam": lam,
                "grid": _whole(rng, 40, 256), "pre": _intervals(rng, 500 / lam, 960 / lam),
                "steps": _intervals(rng, 32, 48), "periodic": rng.choice([0, 0, 3]),
                "melting": rng.random() < 0.3}
    if kind == "coupled":
        return {"kind": kind, "size": round(_log(rng, 0.3, 1.2), 3), "grains": _whole(rng, 4, 32),
                "grid": _whole(rng, 16, 96), "pre": _intervals(rng, 96, 320),
                "handovers": rng.choice([4, 8, 16]), "per_handover": 4}
    if kind in ("output", "regrid"):
        lam = round(_log(rng, 1.5, 4.0), 2)
        c = {"kind": kind, "family": rng.choice(["columnar", "equiaxed"]), "lam": lam,
             "size": round(_log(rng, 0.8, 3.0), 3), "grid": _whole(rng, 33, 128),
             "pre": _intervals(rng, 320, 960 / lam)}
        if kind == "output":
            c["map"], c["window"] = _whole(rng, 30, 400 if c["family"] == "equiaxed" else 160), round(rng.uniform(0.05, 0.3), 3)
        else:
            c["nodes"] = _whole(rng, 20, 120)
        return c
    if kind == "adjoint":
        whole = rng.random() < 0.5
        return {"kind": kind, "grains": _whole(rng, 1, 16) if whole else 1,
                "shell": _whole(rng, 8, 60) if whole else _whole(rng, 20, 360),
                "field": rng.choice(["uniform", "linear", "grid"]),
                "steps": _intervals(rng, 48, 192) if whole else _whole(rng, 60, 500),
                "ckpt": rng.choice([16, 25, 50, 64, 7]), "whole": whole}
    return {"kind": kind, "members": _whole(rng, 3, 32), "size": round(_log(rng, 0.3, 1.0), 3),
            "pre": _intervals(rng, 320, 640), "steps": _intervals(rng, 32, 96)}


# --------------------------------------------------------------- workloads --
DT0 = {5e-4: 10.0, 2e-4: 14.0, 5e-5: 17.0}  # undercooling at the cold face [K] by time step


def _columnar(case, seed):
    s = case["size"] * 1e-3
    dt = case.get("dt", 5e-4)
    w = W.directional(seed=seed, n_grains=case.get("grains", 24), size=(s, s, 2 * s), dT0=DT0[dt],
                      dt=dt, h=5e-6 * case.get("cells", 2))
    if case.get("periodic"):
        n = max(3, int(round(s / w.h)))  # a whole number of cells per period
        w.hi = (n * w.h, n * w.h, w.hi[2])
        w.periodic = case["periodic"]
    if case.get("power"):
        w.b = (2.2, 2.9)
    return w


def _equiaxed(case, seed):
    s, lam = case["size"] * 1e-3, case["lam"] * 1e-6
    size = (s, s / 2, s / 4)
    if case.get("scaled"):
        w = W.cet(seed=seed, size=size, lambda0=lam, grid_n=case["grid"], dT0=6.0, rate=2.0,
                  bulk_density=2e12, face_density=2e8, dt=1.5e-3, U=0.005, q=0.004)
    else:
        w = W.cet(seed=seed, size=size, lambda0=lam, h=2 * lam, grid_n=case["grid"], dT0=12.0,
                  dt=5e-5 * case["lam"])
    if case.get("periodic"):
        w.hi = tuple(max(3, int(round(v / w.h))) * w.h for v in w.hi)
        w.periodic = case["periodic"]
    return w


def _active(case):
    """Rough number of active particles during the pass (sizes the stores and
    the stated work)."""
    if case["kind"] == "grain":
        return 4.0 * (case["shell"] + 1) ** 2 + 2
    if case["kind"] == "adjoint":
        return case["grains"] * (4.0 * case["shell"] ** 2 + 2)
    s = case["size"]
    if case.get("family", case["kind"]) == "equiaxed":
        grown = case["pre"] * case["lam"] / 960.0  # share of the time of the large case
        if case.get("scaled"):
            return 4e3 * (s / 0.4) ** 3
        return 1.3e7 * (s / 3.2) ** 3 / case["lam"] ** 2 * min(1.0, grown) ** 2
    return 3e5 * (s / 2.0) ** 2


def _caps(case, **more):
    n = _active(case)
    caps = dict(cap_particles=int(2.5 * n) + (1 << 18), cap_stopped=int((4 if n > 4e6 else 12) * n) + (1 << 18),
                cap_claim_bricks=max(1 << 16, int(n * 0.6)), cap_grains=4096)
    caps.update(more)
    return caps


def _grown(w, case, **caps):
    """A context of the workload after its first steps."""
    ctx = B.Context.from_workload(w, device=DEV, **_caps(case, **caps))
    if case.get("melting"):
        ctx.set_melting(True)
    ctx.step(w.dt, R * (case["pre"] // R))
    return ctx


def _keep(state):
    """Copy of the device workspace that the program owns."""
    state["snap"] = state["owner"].workspace.clone()
    return state


def _rewind(state):
    state["owner"].workspace.copy_(state["snap"])


# ----------------------------------------------------------------- prepare --
def prepare(case, seed):
    kind = case["kind"]
    g = W.rng(seed)
    if kind == "grain":
        w = W.single_grain(shell_r=case["shell"])
        w.grain_centre = w.grain_centre + 2e-5 * (g.random((1, 3)) - 0.5)
        w.grain_quat = W.shoemake_quaternions(g, 1)
        w.field.dT = 4.95 + 0.1 * g.random()
        ctx = B.Context.from_workload(w, device=DEV, **_caps(case, cap_grains=64))
        ctx.prepare_step(w.dt)
        return _keep({"case": case, "w": w, "ctx": ctx, "owner": ctx})
    if kind == "columnar":
        w = _columnar(case, seed)
        ctx = _grown(w, case)
        ctx.prepare_step(w.dt)
        return _keep({"case": case, "w": w, "ctx": ctx, "owner": ctx})
    if kind == "equiaxed":
        w = _equiaxed(case, seed)
        ctx = _grown(w, case)
        fd = w.field
        ctx.set_deposition_grid(fd.n, fd.origin, fd.spacing)
        ctx.prepare_step(w.dt)
        counts = torch.empty(fd.n[2], fd.n[1], fd.n[0], dtype=torch.int32, device=DEV)
        return _keep({"case": case, "w": w, "ctx": ctx, "owner": ctx, "counts": counts})
    if kind == "coupled":
        s, m = case["size"] * 1e-3, case["grid"]
        w, spec = W.directional_solute(seed=seed, n_grains=case["grains"], size=(s, s, 2 * s),
                                       grid=(m, m, 2 * m), amp=0.2 + 0.2 * g.random(), h=10e-6)
        ctx = _grown(w, case)
        ctx.set_deposition_grid(spec.n, spec.origin, spec.spacing)
        t0, per = (case["pre"] // R) * R * w.dt, case["per_handover"]
        fields = []
        for k in range(case["handovers"]):
            f = spec.field(t0 + k * per * w.dt)
            f.T, f.w = torch.from_numpy(f.T).to(DEV), torch.from_numpy(f.w).to(DEV)
            fields.append(f)
        gm = torch.empty(2 * m, m, m, dtype=torch.float32, device=DEV)
        return _keep({"case": case, "w": w, "ctx": ctx, "owner": ctx, "fields": fields, "gm": gm})
    if kind in ("output", "regrid"):
        if case["family"] == "columnar":
            w = _columnar(case, seed)
            m = case["grid"]
            ctx = _grown(w, case, field_n=(m, m, 2 * m))
        else:
            w = _equiaxed(case, seed)
            ctx = _grown(w, case)
        state = {"case": case, "w": w, "ctx": ctx}
        if kind == "output":
            vox = (w.hi[0] - w.lo[0]) / case["map"]
            state["grid"] = ([max(1, int(round((h - l) / vox))) for l, h in zip(w.lo, w.hi)],
                             w.lo, [vox] * 3)
            # A column through the box, somewhere in its middle half.
            size = np.subtract(w.hi, w.lo)
            side = case["window"] * size[:2]
            at = size[:2] * (0.25 + 0.5 * g.random(2)) - side / 2
            lo = np.maximum(np.append(at, 0.0), 0.0)
            state["window"] = (lo, np.append(side, size[2]))
            # The program's record buffer, larger than any window of this size.
            rows = 1 << int(np.ceil(np.log2(10 * _active(case) * case["window"] ** 2 + 16384)))
            state["records"] = torch.empty(rows, 12, dtype=torch.int32, device=DEV)
        else:
            top = w.field.n if any(w.field.n) else (case["grid"], case["grid"], 2 * case["grid"])
            n = tuple(max(2, min(case["nodes"], v)) for v in top)
            spacing = tuple((h - l) / (k - 1) for l, h, k in zip(w.lo, w.hi, n))
            state["nodes"] = (n, w.lo, spacing)
            state["gm"] = torch.empty(n[2], n[1], n[0], dtype=torch.float32, device=DEV)
        return state
    if kind == "adjoint":
        state = _adjoint_inputs(case, seed)
        ctx = B.Context(state["params"], device=DEV)
        ctx.set_thermal_field(state["field"])
        ctx.init_grains(state["centre"], state["quat"], np.full(case["grains"], case["shell"]))
        state.update(ctx=ctx, owner=ctx)
        if case["whole"]:
            return _keep(state)
        ctx.adjoint_forward(state["dt"], case["steps"], case["ckpt"])
        return state
    # batch
    s = case["size"] * 1e-3
    ws, ps = [], []
    for k in range(case["members"]):
        w = W.directional(seed=1000 * seed + k, n_grains=int(4 * 12 ** g.random()),
                          size=(s, s, 2 * s), h=10e-6)
        c = int(4e5 * case["size"] ** 2) + (1 << 16)
        ws.append(w)
        ps.append(B.params_from_workload(w, cap_particles=c, cap_stopped=c, cap_grains=64,
                                         cap_claim_bricks=1 << 15))
    batch = B.Batch(ps, device=DEV)
    for m, w in zip(batch.members, ws):
        m.init_from_workload(w)
    batch.step(ws[0].dt, R * (case["pre"] // R))
    return _keep({"case": case, "owner": batch, "batch": batch, "ws": ws})


def _adjoint_inputs(case, seed):
    g = W.rng(seed)
    n, r, lam = case["grains"], case["shell"], 5e-6
    # Envelopes of radius r lambda0 around centres about 1.7 r lambda0 apart
    # (neighbours meet during the run); one grain has the box to itself.
    side = int(np.ceil(n ** (1 / 3)))
    pitch = 1.7 * r * lam
    box = side * pitch + 2.4 * r * lam + 2e-4
    at = np.array([(i, j, k) for k in range(side) for j in range(side) for i in range(side)], float)
    centre = 0.5 * box + (at[:n] - (side - 1) / 2) * pitch + 2e-6 * (g.random((n, 3)) - 0.5)
    quat = W.shoemake_quaternions(g, n)
    lo, hi = (0.0, 0.0, 0.0), (box, box, box)
    if case["field"] == "uniform":
        f = W.Field(W.FIELD_UNIFORM, dT=5.0 + g.random())
    elif case["field"] == "linear":
        f = W.Field(W.FIELD_LINEAR, dT0=8.0 + g.random(), grad=(-1.5 / box, 1.0 / box, -2.0 / box),
                    rate=3.0)
    else:
        m = 64
        a = np.linspace(0.0, 2 * np.pi, m)
        z, y, x = np.meshgrid(a, a, a, indexing="ij")
        ph = 2 * np.pi * g.random(3)
        data = 7.0 + np.sin(x + ph[0]) + 0.8 * np.sin(2 * y + ph[1]) * np.cos(z + ph[2])
        f = W.Field(W.FIELD_GRID, n=(m, m, m), origin=lo, spacing=(box / (m - 1),) * 3,
                    data=np.ascontiguousarray(data, np.float32))
    cap = n * (4 * r * r + 2) + 64
    p = B.make_params(lo, hi, lam, 4 * lam, lam, W.KIN_A, W.KIN_B, branching=0, cap_particles=cap,
                      cap_stopped=cap, cap_grains=64,
                      cap_claim_bricks=1 << max(12, int(np.log2(n * r ** 3 / 100 + 1)) + 1),
                      field_n=f.n if case["field"] == "grid" else (0, 0, 0))
    dL = torch.from_numpy(g.normal(size=(n * (4 * r * r + 2), 3)).astype(np.float32)).to(DEV)
    return {"case": case, "params": p, "field": f, "centre": centre, "quat": quat, "dLdx": dL,
            "dt": 1e-4}


# --------------------------------------------------------------------- run --
COUNTS = ("n_active", "n_stopped", "n_grains", "n_claim_bricks", "advanced", "exited", "spawners",
          "children", "contained", "nucleated", "melted", "removed", "reactivated", "grains_melted",
          "step")


def _counts(stats):
    return {"counts": torch.tensor([[s[k] for k in COUNTS] for s in stats]),
            "clock": torch.tensor([[s["t"], s["max_step"]] for s in stats], dtype=torch.float64)}


def _digests(ctxs):
    return torch.from_numpy(np.array([c.digest() for c in ctxs], np.uint64).view(np.int64))


def _particles(ctx, window=None, buf=None):
    """Particles (of a window), in the order of their identity; in a buffer of
    the program's, its rows past the last particle zero."""
    args = None
    if window is not None:
        args = B.ge_query_args()
        args.n[:] = [1, 1, 1]
        args.origin[:] = [float(v) for v in window[0]]
        args.spacing[:] = [float(v) for v in window[1]]
    need = ctx.query_envelope(B.QUERY_PARTICLES, args=args)
    n = need // 48
    rec = torch.empty(n, 12, dtype=torch.int32, device=DEV) if buf is None else buf[:n]
    if need:
        ctx.query_envelope(B.QUERY_PARTICLES, rec, args=args)
    k = rec[:, 4:9].long()
    key = ((((k[:, 3] * 32768 + k[:, 0] + 16384) * 32768 + k[:, 1] + 16384) * 32768 +
            k[:, 2] + 16384) * 8 + (k[:, 4] & 7))
    order = torch.argsort(key)
    if buf is None:
        rec = rec[order]
    else:
        rec.copy_(rec[order])
        buf[n:].zero_()
        rec = buf
    return {"position": rec[:, :3].contiguous().view(torch.float32),
            "travel": rec[:, 3].contiguous().view(torch.float32),
            "lattice": rec[:, 4:9], "cell": rec[:, 9:]}


def _few_particles(ctx):
    """The same through the allocation-free query, on the host."""
    p, n = ctx.particles_noalloc()
    p = p[:n]
    p = p[np.lexsort((p["dir"], p["site"][:, 2], p["site"][:, 1], p["site"][:, 0], p["grain"]))]
    return {"position": np.stack([p["x"], p["y"], p["z"]], 1), "travel": p["s"].copy(),
            "lattice": np.column_stack([p["site"], p["grain"].astype(np.int32),
                                        p["dir"].astype(np.int32) | p["state"].astype(np.int32) << 8]),
            "cell": p["cell"].copy()}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if "snap" in state:
        _rewind(state)
    if kind == "grain":
        ctx, dt = state["ctx"], state["w"].dt
        stats = [ctx.step(dt, case["per_call"]) for _ in range(case["steps"] // case["per_call"])]
        out = _few_particles(ctx) if case["shell"] <= 4 else _particles(ctx)
        return {**out, **_counts(stats[-1:])}
    if kind == "columnar":
        ctx, w = state["ctx"], state["w"]
        st = ctx.step(w.dt, case["steps"])
        vox = (w.hi[0] - w.lo[0]) / case["map"]
        n = [max(1, int(round((h - l) / vox))) for l, h in zip(w.lo, w.hi)]
        return {"map": ctx.grain_map(n, w.lo, [vox] * 3, device_out=True),
                "digest": _digests([ctx]), **_counts([st])}
    if kind == "equiaxed":
        ctx, w = state["ctx"], state["w"]
        st = ctx.step(w.dt, case["steps"])
        ctx.query_envelope(B.QUERY_MUSHY_COUNTS, state["counts"])
        return {"reached": state["counts"], "sites": ctx.site_states(),
                "digest": _digests([ctx]), **_counts([st])}
    if kind == "coupled":
        ctx, w = state["ctx"], state["w"]
        for f in state["fields"]:
            ctx.set_thermal_field(f)
            ctx.step(w.dt, case["per_handover"], stats=False)
            ctx.query_envelope(B.QUERY_MUSHY, state["gm"])
        return {"mushy": state["gm"], "digest": _digests([ctx]), **_counts([ctx.counts()])}
    if kind == "output":
        ctx = state["ctx"]
        return {"map": ctx.grain_map(*state["grid"], device_out=True),
                **_particles(ctx, state["window"], state["records"])}
    if kind == "regrid":
        ctx = state["ctx"]
        ctx.set_deposition_grid(*state["nodes"])
        ctx.query_envelope(B.QUERY_MUSHY, state["gm"])
        return {"mushy": state["gm"]}
    if kind == "adjoint":
        ctx = state["ctx"]
        out = {}
        if case["whole"]:
            ctx.adjoint_forward(state["dt"], case["steps"], case["ckpt"])
            out["position"] = ctx.adjoint_positions()
        out["grad"] = torch.tensor(ctx.adjoint_backward(state["dLdx"]), dtype=torch.float64)
        return out
    batch = state["batch"]
    st = batch.step(state["ws"][0].dt, case["steps"])
    n = (24, 24, 48)
    maps = [m.grain_map(n, w.lo, [w.hi[0] / n[0]] * 3, device_out=True)
            for m, w in zip(batch.members, state["ws"])]
    return {"maps": torch.stack(maps), "digest": _digests(batch.members), **_counts(st)}


# -------------------------------------------------------------------- work --
def work(case):
    """Each active particle's 16-byte record read and written in every step
    (and each node of a field resampled or handed over), the results written
    once; about 60 operations per particle update."""
    kind, n = case["kind"], _active(case)
    if kind == "grain":
        return {"bytes": 32.0 * n * case["steps"] + 48.0 * n, "flops": 60.0 * n * case["steps"]}
    if kind == "columnar":
        return {"bytes": 32.0 * n * case["steps"] + 8.0 * case["map"] ** 3,
                "flops": 60.0 * n * case["steps"]}
    if kind == "equiaxed":
        nodes = float(case["grid"]) ** 3
        return {"bytes": (32.0 * n + 4.0 * nodes) * case["steps"] + 4.0 * nodes,
                "flops": (60.0 * n + 50.0 * nodes) * case["steps"]}
    if kind == "coupled":
        nodes = 2.0 * case["grid"] ** 3
        steps = case["handovers"] * case["per_handover"]
        return {"bytes": 32.0 * n * steps + 28.0 * nodes * case["handovers"],
                "flops": 60.0 * n * steps}
    if kind in ("output", "regrid"):
        # The reached sites of the state, one bit each, and the records.
        sites = 25.0 * n
        if kind == "regrid":
            return {"bytes": sites / 8 + 8.0 * case["nodes"] ** 3, "flops": 24.0 * sites}
        vox = case["map"] ** 3 * (2.0 if case["family"] == "columnar" else 0.125)
        return {"bytes": 4.0 * vox + sites / 8 + 5 * 16.0 * n, "flops": 40.0 * vox}
    if kind == "adjoint":
        per = 16.0 + (4.0 + 12.0) + 4.0 * (case["steps"] // case["ckpt"] + 1)
        if case["whole"]:
            per += 32.0 * case["steps"] + 12.0
        return {"bytes": n * per, "flops": 160.0 * n * case["steps"]}
    n = case["members"] * 4e4 * case["size"] ** 2
    return {"bytes": 32.0 * n * case["steps"], "flops": 60.0 * n * case["steps"]}


# ------------------------------------------------------------------- exact --
def _rotation(q):
    w, x, y, z = np.asarray(q, float) / np.linalg.norm(q)
    return np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                     [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                     [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]])


def _shell(r):
    """Sites and directions of an octahedral envelope of L1 radius r (r = 0:
    the nucleus), in the order in which its particles are created."""
    if r == 0:
        return np.zeros((6, 3), int), np.arange(6)
    s = [(x, y, z) for x in range(-r, r + 1) for y in range(-(r - abs(x)), r - abs(x) + 1)
         for z in sorted({-(r - abs(x) - abs(y)), r - abs(x) - abs(y)})]
    s = np.array(s)
    axis = np.argmax(np.abs(s), 1)
    return s, 2 * axis + (s[np.arange(len(s)), axis] < 0)


def _along(R3, d):
    return np.where(d % 2 == 0, 1.0, -1.0)[:, None] * R3[:, d // 2].T


def _exact_grain(case, seed):
    g = W.rng(seed)
    w = W.single_grain(shell_r=case["shell"])
    c = w.grain_centre[0] + 2e-5 * (g.random((1, 3)) - 0.5)[0]
    R3 = _rotation(W.shoemake_quaternions(g, 1)[0])
    dT = 4.95 + 0.1 * g.random()
    s = case["steps"] * w.dt * (w.a[0] * dT ** w.b[0] + w.a[1] * dT ** w.b[1])
    if s > 0.95 * w.lambda0:
        return None  # the envelope has branched
    site, d = _shell(case["shell"])
    o = np.lexsort((d, site[:, 2], site[:, 1], site[:, 0]))
    site, d = site[o], d[o]
    x = c + w.lambda0 * site @ R3.T + s * _along(R3, d)
    return {"position": x, "travel": np.full(len(d), s), "lattice": None, "cell": None,
            "counts": None, "clock": None}


def _exact_adjoint(case, seed):
    """The travel of each particle by the explicit scheme and its reverse,
    in 64 bits; one grain, which meets nothing."""
    if case["grains"] > 1:
        return None
    I = _adjoint_inputs(case, seed)
    f, dt, lam = I["field"], I["dt"], I["params"].lambda0
    R3 = _rotation(I["quat"][0])
    site, d = _shell(case["shell"])
    t = lambda v: torch.as_tensor(np.ascontiguousarray(v, float), device=DEV)  # noqa: E731
    u = t(_along(R3, d))
    x0 = t(I["centre"][0] + lam * site @ R3.T)
    if case["field"] == "grid":
        data, n, h = t(f.data).reshape(-1), f.n[0], f.spacing[0]

    def undercooling(s, k):
        """dT and its derivative along the travel."""
        if case["field"] == "uniform":
            return torch.full_like(s, f.dT), torch.zeros_like(s)
        x = x0 + s[:, None] * u
        if case["field"] == "linear":
            grad = t(f.grad)
            return f.dT0 + f.rate * k * dt + x @ grad, u @ grad
        i = torch.clamp(torch.floor(x / h), 0, n - 2)
        a = x / h - i
        i = i.long()
        v = [[[data[((i[:, 2] + dz) * n + i[:, 1] + dy) * n + i[:, 0] + dx] for dx in (0, 1)]
              for dy in (0, 1)] for dz in (0, 1)]
        ax, ay, az = a[:, 0], a[:, 1], a[:, 2]
        vx = [[v[z][y][0] + ax * (v[z][y][1] - v[z][y][0]) for y in (0, 1)] for z in (0, 1)]
        vy = [vx[z][0] + ay * (vx[z][1] - vx[z][0]) for z in (0, 1)]
        gx = [[v[z][y][1] - v[z][y][0] for y in (0, 1)] for z in (0, 1)]
        gx = [gx[z][0] + ay * (gx[z][1] - gx[z][0]) for z in (0, 1)]
        gx = gx[0] + az * (gx[1] - gx[0])
        gy = [vx[z][1] - vx[z][0] for z in (0, 1)]
        gy = gy[0] + az * (gy[1] - gy[0])
        g3 = torch.stack([gx, gy, vy[1] - vy[0]], 1) / h
        return vy[0] + az * (vy[1] - vy[0]), (g3 * u).sum(1)

    a0, a1 = W.KIN_A
    s = torch.zeros(len(d), dtype=torch.float64, device=DEV)
    tape = []
    for k in range(case["steps"]):
        tape.append(s)
        dT = undercooling(s, k)[0].clamp_min(0)
        s = s + dt * (a0 * dT ** 2 + a1 * dT ** 3)
    lam_s = (I["dLdx"].double() * u).sum(1)
    grad = torch.zeros(3, dtype=torch.float64, device=DEV)
    for k in range(case["steps"] - 1, -1, -1):
        dT, slope = undercooling(tape[k], k)
        dT = dT.clamp_min(0)
        vp = 2 * a0 * dT + 3 * a1 * dT ** 2
        grad += dt * torch.stack([(lam_s * dT ** 2).sum(), (lam_s * dT ** 3).sum(),
                                  -(lam_s * vp).sum()])
        lam_s = lam_s * (1 + dt * vp * slope)
    out = {"grad": grad}
    if case["whole"]:
        out["position"] = x0 + s[:, None] * u
    return out


def exact(case, seed):
    """What 64-bit arithmetic gives, where the pass has a closed or per-particle
    form; whole runs with contacts and branching have none."""
    if case["kind"] == "grain":
        return _exact_grain(case, seed)
    if case["kind"] == "adjoint":
        return _exact_adjoint(case, seed)
    return None
