"""The work that a user of the library has it do, as cases to be timed.

A program makes a `Simulation` (one periodic box, or a batch of boxes), sets
the fields, advances it and reads rho and u back.  Three kinds of pass:

* "run": `steps` time steps, then the fields as device tensors in the run's own
  precision (a snapshot).  With `fresh` the pass starts from new fields
  (`init`), as in a parameter study; otherwise it continues the run.
* "batch": the same for `boxes` boxes of different sizes, each with its own tau.
* "check": what a program does around the steps: new fields, the conserved
  totals, the error against reference fields, and a snapshot.

`tune` stands for programs that run long and let the library time its kernels
once, beforehand; the others take the defaults.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2002_02503_amd import lbm

TYPES = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
Q_OF = {"D2Q9": 9, "D3Q15": 15, "D3Q19": 19, "D3Q39": 39}
DEFAULT_K = {"D2Q9": 3, "D3Q15": 3, "D3Q19": 3, "D3Q39": 4}


def _box(name, lattice, dims, tau, dtype, steps, *, fresh=False, tune=False, K=0, collision="filtered", theta=0.0,
         background=0.0):
    return {"name": name, "kind": "run", "lattice": lattice, "nx": dims[0], "ny": dims[1], "nz": dims[2], "tau": tau,
            "dtype": dtype, "steps": steps, "fresh": fresh, "tune": tune, "K": K, "collision": collision,
            "theta": theta, "background": background}


def _batch(name, lattice, boxes, lo, hi, dtype, steps, *, tune=False):
    return {"name": name, "kind": "batch", "lattice": lattice, "boxes": boxes, "lo": lo, "hi": hi, "dtype": dtype,
            "steps": steps, "tune": tune, "fresh": False, "K": 0, "collision": "filtered", "theta": 0.0,
            "background": 0.1}


def _check(name, lattice, dims, dtype):
    return {"name": name, "kind": "check", "lattice": lattice, "nx": dims[0], "ny": dims[1], "nz": dims[2],
            "tau": 0.6, "dtype": dtype, "steps": 0, "fresh": True, "tune": False, "K": 0, "collision": "filtered",
            "theta": 0.0, "background": 0.0}


def listed():
    return [
        # a coupled program: one step of a small box, then its fields, over and over
        _box("call16_fp32", "D3Q19", (16, 16, 16), 0.6, "fp32", 1),
        # the Taylor-Green vortex of the 2-D tests, from its fields to the fields after 1000 steps
        _box("vortex64_fp64", "D2Q9", (64, 64, 1), 0.8, "fp64", 1000, fresh=True),
        # a small box run long, as the 32^3 recipe of the error figures
        _box("box32_fp32", "D3Q19", (32, 32, 32), 0.51, "fp32", 500, tune=True),
        # the README's program: a box on a background flow, default kernel
        _box("shear128_fp32", "D3Q19", (128, 128, 128), 0.55, "fp32", 200, fresh=True, background=0.1),
        # a ragged box with the energy-flux term, default kernel
        _box("ragged_flux_fp32", "D3Q19", (201, 150, 77), 0.55, "fp32", 50, theta=0.5),
        # the headline box in each storage type that the benchmark runs long
        _box("turb256_fp32", "D3Q19", (256, 256, 256), 0.51, "fp32", 50, tune=True),
        _box("turb256_fp16", "D3Q19", (256, 256, 256), 0.51, "fp16", 50, tune=True),
        _box("turb256_fp64", "D3Q19", (256, 256, 256), 0.51, "fp64", 30, tune=True),
        # the 39-velocity lattice on the benchmark's box
        _box("d3q39_192_fp32", "D3Q39", (192, 192, 192), 0.6, "fp32", 30, tune=True, background=0.1),
        # the benchmark's batch of 256 boxes of sides 16 to 64
        _batch("batch256_fp32", "D3Q19", 256, 16, 64, "fp32", 50, tune=True),
        _batch("batch256_fp16", "D3Q19", 256, 16, 64, "fp16", 50, tune=True),
        # set-up, totals, residual and snapshot of the headline box
        _check("check256_fp32", "D3Q19", (256, 256, 256), "fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    n = _log(rng, lo, hi)
    r = rng.random()
    if r < 0.3 and n >= 64:
        n = n // 64 * 64
    elif r < 0.5 and n >= 8:
        n = n // 8 * 8
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choices(["run", "run2d", "batch", "check"], [9, 4, 4, 3])[0]
    dtype = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"])
    tau = round(rng.uniform(0.51, 1.0), 3)
    steps = _log(rng, 1, 100)
    if kind == "run2d":
        dims = (_side(rng, 16, 2048), _side(rng, 16, 2048), 1)
        c = _box("", "D2Q9", dims, tau, dtype, steps, fresh=rng.random() < 0.5, tune=rng.random() < 0.4)
    elif kind == "batch":
        lo = _log(rng, 4, 32)
        hi = _log(rng, max(lo, 16), 64)
        lattice = rng.choice(["D3Q15", "D3Q19", "D3Q19"])
        c = _batch("", lattice, _log(rng, 2, 256), lo, hi, dtype, min(steps, 50), tune=rng.random() < 0.4)
    else:
        lattice = rng.choice(["D3Q15", "D3Q19", "D3Q19", "D3Q39"])
        most = 192 if lattice == "D3Q39" else 256
        dims = tuple(_side(rng, 8, most) for _ in range(3))
        if kind == "check":
            c = _check("", lattice, dims, dtype)
        else:
            kinds = [("filtered", 0.0, 0), ("filtered", 0.0, 0), ("bgk", 0.0, 0), ("filtered", 0.0, 2),
                     ("filtered", 0.3, 0)]
            if lattice == "D3Q39":
                kinds += [("filtered", 0.0, 5)]
            collision, theta, K = rng.choice(kinds)
            if theta:
                tau = max(tau, 0.55)  # the term's stability bound
            c = _box("", lattice, dims, tau, dtype, min(steps, 30), fresh=rng.random() < 0.4,
                     tune=rng.random() < 0.5, K=K, collision=collision, theta=theta,
                     background=rng.choice([0.0, 0.1]))
    del c["name"]
    # no more work than the listed cases
    n = sum(x * y * z for x, y, z in _geometry(c)[0])
    c["steps"] = min(c["steps"], max(1, int(5e10 / (n * Q_OF[c["lattice"]] * lbm.DTYPE_BYTES[c["dtype"]]))))
    return c


# -- inputs -------------------------------------------------------------------

def _geometry(case):
    """[(nx, ny, nz)] and [tau] of the case's boxes; the same for every seed."""
    if case["kind"] != "batch":
        return [(case["nx"], case["ny"], case["nz"])], [case["tau"]]
    rng = np.random.default_rng([case["boxes"], case["lo"], case["hi"]])
    dims, tau = [], []
    for _ in range(case["boxes"]):
        dims.append(tuple(int(v) for v in rng.integers(case["lo"], case["hi"] + 1, size=3)))
        tau.append(float(rng.uniform(0.52, 1.0)))
    return dims, tau


def _flow(dims, rng, background, modes, D):
    """A solenoidal field of random long waves, rms 0.04 a component, on a
    uniform background, and a density of small waves: (rho, u) as [nz, ny, nx]
    and [D, nz, ny, nx] on the GPU."""
    nx, ny, nz = dims
    axes = [2 * math.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n for n in (nx, ny, nz)]
    rho = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
    u = torch.zeros((D, nz, ny, nx), dtype=torch.float64, device="cuda")
    for _ in range(modes):
        k = np.array([rng.integers(-min(4, (n - 1) // 2), min(4, (n - 1) // 2) + 1) for n in dims], dtype=np.float64)
        if not k.any():
            k[0] = 1.0
        wave = k * 2 * np.pi / np.array(dims, dtype=np.float64)  # physical wave vector
        a = rng.normal(size=3)
        if D == 2:
            a[2] = 0.0
        a -= wave * (a @ wave) / (wave @ wave)
        a /= max(1e-6, math.sqrt(a @ a))
        phase, dens = rng.uniform(0, 2 * np.pi), rng.normal()
        s = torch.sin((k[2] * axes[2] + phase)[:, None, None] + (k[1] * axes[1])[:, None] + k[0] * axes[0])
        for b in range(D):
            u[b].add_(s, alpha=float(a[b]))
        rho.add_(s, alpha=float(dens))
    u.mul_(0.04 / max(1e-12, math.sqrt(float(u.square().sum()) / (D * nx * ny * nz))))
    rho.mul_(1e-3 / max(1e-12, math.sqrt(float(rho.square().mean())))).add_(1.0)
    U = rng.normal(size=3)
    U *= background * rng.uniform(0.5, 1.0) / math.sqrt(U @ U)
    for b in range(D):
        u[b].add_(float(U[b]))
    return rho, u


def _fields(case, seed):
    """(rho, u) of the case from the seed, in the library's layout."""
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 7])
    D = 2 if case["lattice"] == "D2Q9" else 3
    boxes, _ = _geometry(case)
    if len(boxes) == 1 and case["kind"] != "batch":
        return _flow(boxes[0], rng, case["background"], 8, D)
    parts = [_flow(b, rng, case["background"], 2, D) for b in boxes]
    return torch.cat([r.reshape(-1) for r, _ in parts]), torch.cat([v.reshape(D, -1) for _, v in parts], dim=1)


def prepare(case, seed):
    boxes, taus = _geometry(case)
    options = {"dtype": case["dtype"], "collision": case["collision"], "theta": case["theta"]}
    if case["K"]:
        options["K"] = case["K"]
    if case["kind"] == "batch":
        sim = lbm.Simulation(case["lattice"], boxes, taus, **options)
    else:
        sim = lbm.Simulation(case["lattice"], boxes[0], taus[0], **options)
    rho, u = _fields(case, seed)
    state = {"case": case, "sim": sim}
    if case["kind"] == "check":
        state["ref"] = _fields(case, seed + 1000003)
    else:
        sim.init(rho, u)
        if case["tune"]:
            sim.tune()
    if case["fresh"]:
        state["fields"] = (rho, u)
    return state


def run(state):
    case, sim = state["case"], state["sim"]
    if case["fresh"]:
        sim.init(*state["fields"])
    out = {}
    if case["kind"] == "check":
        out["totals"] = sim.totals()
        out["residual"] = sim.residual(*state["ref"])
    else:
        sim.step(case["steps"])
    rho, u = sim.moments(device=True)
    out["rho"], out["u"] = rho.to(TYPES[case["dtype"]]), u.to(TYPES[case["dtype"]])
    return out


# -- what a pass cannot do without ----------------------------------------------

def work(case):
    """Bytes: the populations (or the fields) in, the populations and the fields
    out, once a pass, however many steps it takes.  Operations: the moments,
    the operator and the conservation of every site and step, about 14 a
    population (24 with the energy-flux term)."""
    boxes, _ = _geometry(case)
    n = sum(x * y * z for x, y, z in boxes)
    Q, S = Q_OF[case["lattice"]], lbm.DTYPE_BYTES[case["dtype"]]
    fields = (3 if case["lattice"] == "D2Q9" else 4) * n
    state = Q * S * n
    into = 8 * fields if case["fresh"] else state
    if case["kind"] == "check":
        return {"bytes": into + 8 * fields + state + S * fields, "flops": 14.0 * Q * n}
    return {"bytes": into + state + S * fields, "flops": (24.0 if case["theta"] else 14.0) * Q * n * case["steps"]}


# -- the same in 64 bits, in plain torch ------------------------------------------

def _lattice(name):
    """(c, w, T0) from the velocity shells."""
    shells = {"D2Q9": (2, [((0, 0), 4 / 9), ((1, 0), 1 / 9), ((1, 1), 1 / 36)], 1 / 3),
              "D3Q15": (3, [((0, 0, 0), 2 / 9), ((1, 0, 0), 1 / 9), ((1, 1, 1), 1 / 72)], 1 / 3),
              "D3Q19": (3, [((0, 0, 0), 1 / 3), ((1, 0, 0), 1 / 18), ((1, 1, 0), 1 / 36)], 1 / 3),
              "D3Q39": (3, [((0, 0, 0), 1 / 12), ((1, 0, 0), 1 / 12), ((1, 1, 1), 1 / 27), ((2, 0, 0), 2 / 135),
                            ((2, 2, 0), 1 / 432), ((3, 0, 0), 1 / 1620)], 2 / 3)}
    D, parts, T0 = shells[name]
    c, w = [], []
    for proto, weight in parts:
        each = {tuple(s * p for s, p in zip(signs, perm)) for perm in itertools.permutations(proto)
                for signs in itertools.product((1, -1), repeat=D)}
        c += sorted(each)
        w += [weight] * len(each)
    return c, w, T0


def _series(a, v, K):
    """P_m = sum_{n <= m} h_n / n! for m = 0..K, h_{n+1} = a h_n - n v h_{n-1}."""
    h = [torch.ones_like(v), a.clone()]
    for n in range(1, K):
        h.append(a * h[n] - n * v * h[n - 1])
    P = [h[0]]
    for n in range(1, K + 1):
        P.append(P[-1] + h[n] / math.factorial(n))
    return P


def _dot(x, y):
    return sum(float(s) * t for s, t in zip(x, y) if s) if any(x) else torch.zeros_like(y[0])


def _exact_collide(f, c, w, T0, omega, K, collision, theta):
    """f' of eq. lbe-reg for f [Q, ...], in place."""
    D, Q = len(c[0]), len(c)
    rho = f.sum(0)
    u = [sum(float(c[i][a]) * f[i] for i in range(Q) if c[i][a]) / rho for a in range(D)]
    v = sum(x * x for x in u) / T0

    def feq(i, P=None):
        return w[i] * rho * (P or _series(_dot(c[i], u) / T0, v, K))[K]

    if collision == "bgk":
        for i in range(Q):
            e = feq(i)
            f[i] = e + omega * (f[i] - e)
        return
    pi = {}
    for a in range(D):
        for b in range(a, D):
            m = sum(float(c[i][a] * c[i][b]) * f[i] for i in range(Q) if c[i][a] * c[i][b])
            pi[a, b] = pi[b, a] = m - rho * (u[a] * u[b] + (T0 if a == b else 0.0))
    trace = sum(pi[a, a] for a in range(D))
    piu = [sum(pi[a, b] * u[b] for b in range(D)) for a in range(D)]
    upu = sum(u[a] * piu[a] for a in range(D)) / T0
    q = {}
    if theta:  # the relative energy flux
        for t in itertools.combinations_with_replacement(range(D), 3):
            a, b, g = t
            flux = sum(float(c[i][a] * c[i][b] * c[i][g]) * (f[i] - feq(i)) for i in range(Q)
                       if c[i][a] * c[i][b] * c[i][g])
            if not isinstance(flux, torch.Tensor):
                flux = torch.zeros_like(rho)
            flux = flux - (u[a] * pi[b, g] + u[b] * pi[a, g] + u[g] * pi[a, b])
            for s in set(itertools.permutations(t)):
                q[s] = flux
        qt = [sum(q[a, a, g] for a in range(D)) for g in range(D)]
        qu = {(a, b): sum(q[a, b, g] * u[g] for g in range(D)) for a in range(D) for b in range(D)}
        quu = [sum(qu[a, b] * u[b] for b in range(D)) for a in range(D)]
        qtu = sum(qt[a] * u[a] for a in range(D))
    zero = torch.zeros_like(rho)
    for i in range(Q):
        P = _series(_dot(c[i], u) / T0, v, K)
        get = lambda m: P[m] if m >= 0 else zero  # noqa: E731
        A = sum(float(c[i][a] * c[i][b]) * pi[a, b] for a in range(D) for b in range(D)
                if c[i][a] * c[i][b]) / T0 - trace
        neq = A * get(K - 2) - 2 / T0 * _dot(c[i], piu) * get(K - 3) + upu * get(K - 4)
        out = feq(i, P) + omega * w[i] / (2 * T0) * neq
        if theta:
            d0 = sum(float(c[i][a] * c[i][b] * c[i][g]) * q[a, b, g] for a in range(D) for b in range(D)
                     for g in range(D) if c[i][a] * c[i][b] * c[i][g]) - 3 * T0 * _dot(c[i], qt)
            d1 = 3 * T0 * qtu - 3 * sum(float(c[i][a] * c[i][b]) * qu[a, b] for a in range(D) for b in range(D)
                                        if c[i][a] * c[i][b])
            d2 = 3 * _dot(c[i], quu)
            out = out + omega * theta * w[i] / (6 * T0 ** 3) * (d0 * get(K - 3) + d1 * get(K - 4) + d2 * get(K - 5))
        f[i] = out


def _source(dims, c, offset):
    """Flat indices of the sites x - c_i of one box, periodic."""
    nx, ny, nz = dims
    z, y, x = (torch.arange(n, device="cuda") for n in (nz, ny, nx))
    c = tuple(c) + (0,) * (3 - len(c))
    x, y, z = (x - c[0]) % nx, (y - c[1]) % ny, (z - c[2]) % nz
    return (offset + (z[:, None, None] * ny + y[:, None]) * nx + x).reshape(-1)


def exact(case, seed):
    boxes, taus = _geometry(case)
    n = sum(x * y * z for x, y, z in boxes)
    if 3e-9 * n * Q_OF[case["lattice"]] * max(1, case["steps"]) * (3 if case["theta"] else 1) > 60:
        return None  # too long
    c, w, T0 = _lattice(case["lattice"])
    D, Q = len(c[0]), len(c)
    K = case["K"] or DEFAULT_K[case["lattice"]]
    rho, u = _fields(case, seed)
    out = {}
    if case["kind"] == "check":
        nx, ny, nz = boxes[0]
        r2, u2 = _fields(case, seed + 1000003)
        sums = [float(rho.sum())] + [float((rho * u[a]).sum()) for a in range(D)] + [0.0] * (3 - D)
        out["totals"] = np.array([sums])
        out["residual"] = {"u_max": float((u - u2).abs().max()), "u_l2": float((u - u2).square().sum().sqrt()),
                           "rho_max": float((rho - r2).abs().max()), "rho_l2": float((rho - r2).square().sum().sqrt())}
        out["rho"], out["u"] = rho, u
        return out
    shapes = rho.shape, u.shape
    rho, u = rho.reshape(-1), u.reshape(D, -1)
    omega = torch.cat([torch.full((x * y * z,), 1 - 1 / t, dtype=torch.float64, device="cuda")
                       for (x, y, z), t in zip(boxes, taus)]) if len(boxes) > 1 else 1 - 1 / taus[0]
    starts = np.concatenate([[0], np.cumsum([x * y * z for x, y, z in boxes])])
    source = [torch.cat([_source(b, c[i], int(o)) for b, o in zip(boxes, starts)]) for i in range(Q)]
    v = sum(u[a] * u[a] for a in range(D)) / T0
    f = torch.stack([w[i] * rho * _series(_dot(c[i], u) / T0, v, K)[K] for i in range(Q)])
    for _ in range(case["steps"]):
        for i in range(Q):
            if any(c[i]):
                f[i] = f[i][source[i]]
        _exact_collide(f, c, w, T0, omega, K, case["collision"], case["theta"])
    rho = f.sum(0)
    out["rho"] = rho.reshape(shapes[0])
    out["u"] = torch.stack([sum(float(c[i][a]) * f[i] for i in range(Q) if c[i][a]) / rho
                            for a in range(D)]).reshape(shapes[1])
    return out
