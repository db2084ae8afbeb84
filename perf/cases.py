"""The work that users have this library do, as a list of timed cases.

Each case is one kind of call with its sizes:

  blocks        System.run_blocks over one sync interval (1/16 time unit)
                from the start-up state: a simulation's main loop
  shared        System.shared_steps: the fixed-step integration, as the
                conservation study runs it in every arithmetic
  evaluate      Context.h6_evaluate of an active set: a program that drives
                its own integrator, or a diagnostic, calls one stage
  startup       System.startup: first forces and initial steps
  energy_loss   adjoint.system_energy and its gradient
  adjoint       a loss through adjoint.hermite_shared_run and its gradients
  adjoint_block the same through adjoint.hermite_block_run

Particles are Plummer spheres (equal masses, or masses from a power law) in
Henon units, softening 1e-4 for the runs and 1e-3 for the gradients, steps
from eta = 0.4 and levels 4 to 30.
"""

import math

import numpy as np
import torch

from paper_1901_08532_amd import adjoint, h6, ics

PRECISIONS = {"fp64": h6.H6_FP64, "mixed": h6.H6_MIXED, "ex": h6.H6_EX, "sp": h6.H6_SP}
SYNC = 1 << (h6.TICK_BITS - 4)  # 1/16 time unit in ticks
ETA, ETA_S, LEV_MIN, LEV_MAX = 0.4, 0.1, 4, 30


def listed():
    return [
        # the simulation loop at its usual size: one sync interval of block steps
        {"name": "blocks-65536", "kind": "blocks", "n": 65536, "precision": "fp64", "masses": "equal"},
        # the same for a small cluster: thousands of tiny blocks, all latency
        {"name": "blocks-4096", "kind": "blocks", "n": 4096, "precision": "fp64", "masses": "equal"},
        # a cluster with a mass spectrum in the mixed arithmetic, odd size
        {"name": "blocks-mixed-20011", "kind": "blocks", "n": 20011, "precision": "mixed", "masses": "powerlaw"},
        # 100 fixed steps of a small system: three or four launches a step
        {"name": "shared-1024", "kind": "shared", "n": 1024, "precision": "fp64", "steps": 100},
        # the conservation study's double-single arithmetic
        {"name": "shared-ex-4096", "kind": "shared", "n": 4096, "precision": "ex", "steps": 16},
        # the smallest call: a few due particles of a small system
        {"name": "evaluate-1024-7", "kind": "evaluate", "n": 1024, "n_act": 7, "precision": "fp64"},
        # an ordinary block of a large system
        {"name": "evaluate-65536-1000", "kind": "evaluate", "n": 65536, "n_act": 1000, "precision": "fp64"},
        # every particle in single precision, odd size
        {"name": "evaluate-sp-10007", "kind": "evaluate", "n": 10007, "n_act": 10007, "precision": "sp"},
        # the first forces and steps of a run
        {"name": "startup-32768", "kind": "startup", "n": 32768, "masses": "powerlaw"},
        # an energy-based loss and its gradient
        {"name": "energy-loss-16384", "kind": "energy_loss", "n": 16384},
        # fitting initial conditions through fixed steps
        {"name": "adjoint-16384", "kind": "adjoint", "n": 16384, "steps": 8},
        # and through block steps
        {"name": "adjoint-block-4096", "kind": "adjoint_block", "n": 4096, "ticks": SYNC // 2},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["blocks", "shared", "evaluate", "evaluate", "startup", "energy_loss", "adjoint", "adjoint_block"])
    if kind == "blocks":
        return {"kind": kind, "n": _size(rng, 512, 50000), "precision": rng.choice(["fp64", "fp64", "mixed"]),
                "masses": rng.choice(["equal", "powerlaw"])}
    if kind == "shared":
        precision = rng.choice(["fp64", "fp64", "ex", "mixed", "sp"])
        n = _size(rng, 256, 8192 if precision == "ex" else 20000)
        return {"kind": kind, "n": n, "precision": precision, "steps": rng.randint(8, 100 if n <= 2048 else 16)}
    if kind == "evaluate":
        n = _size(rng, 512, 65536)
        return {"kind": kind, "n": n, "n_act": min(n, rng.choice([_size(rng, 1, 64), _size(rng, 64, n), n])),
                "precision": rng.choice(["fp64", "fp64", "fp64", "mixed", "ex", "sp"])}
    if kind == "startup":
        return {"kind": kind, "n": _size(rng, 512, 50000), "masses": rng.choice(["equal", "powerlaw"])}
    if kind == "energy_loss":
        return {"kind": kind, "n": _size(rng, 256, 50000)}
    if kind == "adjoint":
        return {"kind": kind, "n": _size(rng, 256, 16384), "steps": rng.randint(4, 12)}
    return {"kind": kind, "n": _size(rng, 256, 8192), "ticks": SYNC // 4}


# ---------------------------------------------------------------- inputs


def _particles(case, seed):
    n = case["n"]
    x, v, m = ics.plummer(n, seed)
    if case.get("masses") == "powerlaw":
        m = ics.salpeter_masses(n, seed + 30)
    return x, v, m


def _predicted(case, seed):
    """(9, n) positions, velocities and accelerations of a Plummer sphere,
    the accelerations those of the model's mean field."""
    x, v, m = _particles(case, seed)
    b = 3.0 * math.pi / 16.0
    a = -x / ((x * x).sum(axis=1, keepdims=True) + b * b) ** 1.5
    P = torch.from_numpy(np.ascontiguousarray(np.concatenate([x.T, v.T, a.T]))).cuda()
    return P, torch.from_numpy(m).cuda()


def _active(case, x):
    """The n_act innermost particles in index order (the dense core holds the
    short steps); None for all of them."""
    n, n_act = case["n"], case["n_act"]
    if n_act == n:
        return None
    near = torch.argsort((x * x).sum(0))[:n_act]
    return torch.sort(near).values.to(torch.int32).contiguous()


def _eps(case):
    return 1e-3 if case["kind"] in ("energy_loss", "adjoint", "adjoint_block") else 1e-4


def _step(case):
    return 1.0 / 256 if case["kind"] == "adjoint" else 1.0 / 1024


def _target(x, seed):
    rng = np.random.Generator(np.random.PCG64(seed + 40))
    return x + 0.01 * rng.standard_normal(x.shape)


def prepare(case, seed):
    kind, n, eps = case["kind"], case["n"], _eps(case)
    if kind == "evaluate":
        P, m = _predicted(case, seed)
        return {"case": case, "ctx": h6.Context(n, eps), "P": P, "m": m, "active": _active(case, P[0:3]),
                "F": torch.empty((9, case["n_act"]), dtype=torch.float64, device="cuda")}
    x, v, m = _particles(case, seed)
    if kind in ("blocks", "shared", "startup"):
        s = h6.System(x, v, m, eps)
        if kind != "startup":
            s.startup(ETA_S, LEV_MIN, LEV_MAX)
        return {"case": case, "system": s, "S0": s.S.clone(), "T0": s.T.clone()}
    st = {"case": case, "ctx": h6.Context(n, eps)}
    for name, arr in (("x", x), ("v", v), ("m", m)):
        st[name] = torch.from_numpy(arr).cuda().requires_grad_(True)
    st["target"] = torch.from_numpy(_target(x, seed)).cuda()
    return st


# ---------------------------------------------------------------- the calls


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "evaluate":
        state["ctx"].h6_evaluate(state["P"], state["m"], state["active"], case["n_act"],
                                 PRECISIONS[case["precision"]], state["F"])
        return state["F"]
    if kind in ("blocks", "shared", "startup"):
        # every pass starts from the same snapshot, as a restarted run does
        s = state["system"]
        s.S.copy_(state["S0"])
        s.T.copy_(state["T0"])
        if kind == "blocks":
            rc, stats = s.run_blocks(SYNC, ETA, LEV_MIN, LEV_MAX, PRECISIONS[case["precision"]])
            return {"S": s.S, "T": s.T, "blocks": int(stats.blocks), "steps": int(stats.particle_steps)}
        if kind == "shared":
            s.shared_steps(_step(case), case["steps"], PRECISIONS[case["precision"]])
            return {"S": s.S}
        s.startup(ETA_S, LEV_MIN, LEV_MAX)
        return {"S": s.S, "T": s.T}
    x, v, m = state["x"], state["v"], state["m"]
    if kind == "energy_loss":
        out = adjoint.system_energy(x, v, m, state["ctx"])
        loss = out * out
    elif kind == "adjoint":
        out = adjoint.hermite_shared_run(x, v, m, state["ctx"], _step(case), case["steps"], checkpoint=8)
        loss = ((out - state["target"]) ** 2).sum()
    else:
        out, _ = adjoint.hermite_block_run(x, v, m, state["ctx"], case["ticks"], ETA, LEV_MIN, LEV_MAX, ETA_S)
        loss = ((out - state["target"]) ** 2).sum()
    gx, gv, gm = torch.autograd.grad(loss, (x, v, m))
    return {"out": out.detach(), "gx": gx, "gv": gv, "gm": gm}


# ---------------------------------------------------------------- what a pass cannot do without

# operations of one pair (a fused multiply-add counts two, a reciprocal
# square root one): a, j, s; the start-up's two passes; potential and
# acceleration; the gradient of a, j, s
_AJS, _STARTUP, _ENERGY, _VJP = 78, 42 + 112, 12 + 22, 235


def _steps_per_particle(case):
    """Block steps a particle takes in 1/16 time unit from the start-up
    state, measured for Plummer spheres (8.1 at n = 1024, 16 at 16384, 23 at
    65536; a few percent fewer with power-law masses)."""
    return 8.0 * (case["n"] / 1024.0) ** 0.254


def work(case):
    kind, n = case["kind"], float(case["n"])
    if kind == "evaluate":
        return {"bytes": 80 * n + 76 * case["n_act"], "flops": _AJS * n * case["n_act"]}
    if kind == "blocks":
        return {"bytes": 2 * 160 * n, "flops": _AJS * n * n * _steps_per_particle(case)}
    if kind == "shared":
        return {"bytes": 2 * 144 * n + 8 * n, "flops": _AJS * n * n * case["steps"]}
    if kind == "startup":
        return {"bytes": (56 + 112) * n, "flops": _STARTUP * n * n}
    if kind == "energy_loss":
        return {"bytes": 2 * 56 * n, "flops": _ENERGY * n * n}
    pairs = n * n * (case["steps"] if kind == "adjoint" else _steps_per_particle(case) * case["ticks"] / SYNC)
    return {"bytes": 2 * 56 * n + 24 * n, "flops": (_AJS + _VJP) * pairs}


# ---------------------------------------------------------------- 64-bit values


def _pair_block(x, v, a, j, m, xi, vi, ai, ji, eps2, outputs):
    """Softened a, j, s, c (those named in outputs) of the targets xi.. from
    every source, each (3, targets)."""
    r = x[:, None, :] - xi[:, :, None]
    w = v[:, None, :] - vi[:, :, None]
    rinv2 = 1.0 / ((r * r).sum(0) + eps2)
    mr3 = m * rinv2 * rinv2.sqrt()
    alpha = (r * w).sum(0) * rinv2
    J = w - 3 * alpha * r
    out = {"a": lambda: r, "j": lambda: J}
    if "s" in outputs:
        d = a[:, None, :] - ai[:, :, None]
        beta = ((w * w).sum(0) + (r * d).sum(0)) * rinv2 + alpha * alpha
        Sn = d - 6 * alpha * J - 3 * beta * r
        out["s"] = lambda: Sn
    if "c" in outputs:
        e = j[:, None, :] - ji[:, :, None]
        gamma = (3 * (w * d).sum(0) + (r * e).sum(0)) * rinv2 + alpha * (3 * beta - 4 * alpha * alpha)
        out["c"] = lambda: e - 9 * alpha * Sn - 9 * beta * J - 3 * gamma * r
    return [(out[k]() * mr3).sum(-1) for k in outputs]


def _pairs(x, v, a, j, m, eps2, outputs, idx=None):
    n = x.shape[1]
    idx = torch.arange(n, device=x.device) if idx is None else idx.long()
    rows = max(1, min(len(idx), (1 << 24) // n))
    res = [torch.empty((3, len(idx)), dtype=x.dtype, device=x.device) for _ in outputs]
    for lo in range(0, len(idx), rows):
        t = idx[lo:lo + rows]
        got = _pair_block(x, v, a, j, m, x[:, t], v[:, t], None if a is None else a[:, t],
                          None if j is None else j[:, t], eps2, outputs)
        for q, g in enumerate(got):
            res[q][:, lo:lo + rows] = g
    return res


class _Ajs(torch.autograd.Function):
    """The pair sums with a gradient that is taken block by block."""

    @staticmethod
    def forward(ctx, x, v, a, j, m, eps2, outputs):
        ctx.save_for_backward(x, v, a, j, m)
        ctx.eps2, ctx.outputs = eps2, outputs
        with torch.no_grad():
            return torch.cat(_pairs(x, v, a, j, m, eps2, outputs))

    @staticmethod
    def backward(ctx, g):
        ins = ctx.saved_tensors
        n = ins[0].shape[1]
        tot = [torch.zeros_like(t) for t in ins]
        rows = max(1, min(n, (1 << 22) // n))
        for lo in range(0, n, rows):
            with torch.enable_grad():
                q = [t.detach().requires_grad_(True) for t in ins]
                x, v, a, j, m = q
                t = slice(lo, lo + rows)
                out = torch.cat(_pair_block(x, v, a, j, m, x[:, t], v[:, t], a[:, t], j[:, t], ctx.eps2, ctx.outputs))
                got = torch.autograd.grad(out, q, g[:, t], allow_unused=True)
            for k, d in enumerate(got):
                if d is not None:
                    tot[k] += d
        return (*tot, None, None)


def _start(x, v, m, eps2):
    z = torch.zeros_like(x)
    aj = _Ajs.apply(x, v, z, z, m, eps2, ("a", "j"))
    a, j = aj[0:3], aj[3:6]
    sc = _Ajs.apply(x, v, a, j, m, eps2, ("s", "c"))
    return a, j, sc[0:3], sc[3:6]


def _shared(x, v, a, j, s, c, m, eps2, h, steps):
    for _ in range(steps):
        ap = a + h * (j + h / 2 * (s + h / 3 * c))
        vp = v + h * (a + h / 2 * (j + h / 3 * (s + h / 4 * c)))
        xp = x + h * (v + h / 2 * (a + h / 3 * (j + h / 4 * (s + h / 5 * c))))
        f = _Ajs.apply(xp, vp, ap, torch.zeros_like(x), m, eps2, ("a", "j", "s"))
        a1, j1, s1 = f[0:3], f[3:6], f[6:9]
        v1 = v + h / 2 * (a + a1) - h * h / 10 * (j1 - j) + h ** 3 / 120 * (s + s1)
        x1 = x + h / 2 * (v + v1) - h * h / 10 * (a1 - a) + h ** 3 / 120 * (j + j1)
        c = (60 * (a1 - a) - h * (24 * j + 36 * j1) + h * h * (9 * s1 - 3 * s)) / h ** 3
        x, v, a, j, s = x1, v1, a1, j1, s1
    return x, v, a, j, s, c


def exact(case, seed):
    kind, n, eps2 = case["kind"], case["n"], _eps(case) ** 2
    if kind == "evaluate":
        P, m = _predicted(case, seed)
        return torch.cat(_pairs(P[0:3], P[3:6], P[6:9], None, m, eps2, ("a", "j", "s"), _active(case, P[0:3])))
    if kind in ("blocks", "adjoint_block"):
        return None  # the block sequence is part of the result
    x0, v0, m0 = _particles(case, seed)
    x, v = (torch.from_numpy(np.ascontiguousarray(t.T)).cuda() for t in (x0, v0))
    m = torch.from_numpy(m0).cuda()
    if kind == "startup":
        return {"S": torch.cat([x, v, *_start(x, v, m, eps2)]), "T": None}
    if kind == "shared":
        with torch.no_grad():
            return {"S": torch.cat(_shared(x, v, *_start(x, v, m, eps2), m, eps2, _step(case), case["steps"]))}
    if kind == "energy_loss":
        a = torch.empty_like(x)
        phi = torch.empty_like(m)
        rows = max(1, min(n, (1 << 24) // n))
        for lo in range(0, n, rows):
            t = slice(lo, lo + rows)
            r = x[:, None, :] - x[:, t, None]
            rinv = ((r * r).sum(0) + eps2).rsqrt()
            a[:, t] = (r * (m * rinv ** 3)).sum(-1)
            w = m * rinv
            i = torch.arange(lo, min(n, lo + rows), device=x.device)
            w[i - lo, i] = 0.0
            phi[t] = -w.sum(-1)
        vv = (v * v).sum(0)
        e = (m * (vv + phi)).sum() / 2
        return {"out": e, "gx": -2 * e * (m * a).T, "gv": 2 * e * (m * v).T, "gm": 2 * e * (vv / 2 + phi)}
    for t in (x, v, m):
        t.requires_grad_(True)
    y = _shared(x, v, *_start(x, v, m, eps2), m, eps2, _step(case), case["steps"])[0]
    loss = ((y.T - torch.from_numpy(_target(x0, seed)).cuda()) ** 2).sum()
    gx, gv, gm = torch.autograd.grad(loss, (x, v, m))
    return {"out": y.detach().T, "gx": gx.T, "gv": gv.T, "gm": gm}
