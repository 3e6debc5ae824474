"""Workloads of the Tau1 framework whose time is watched.

Each case is one stretch of a user's program: a context over one or more
samples is at hand, the program advances it by some steps and reads the fields
(and, for porous samples, the permeability) back.  Sizes and settings come from
the benchmark, the tests and the smoke run of this repository, or are generic
(odd extents, row lengths between the lane layouts).

Fields are kept in the precision the run computes in: the library hands out
FP64 host arrays, an FP32 run's are kept as float32, a 16-bit-storage run's as
float16 or bfloat16.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2312_14742_amd import tau1

KEEP = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def _case(name, kind="porous", lattice=19, precision="f32", nx=64, ny=64, nz=64, phi=0.7,
          radius=8.0, steps=100, samples=1, g=1e-6, tune=False, restart=False):
    c = dict(name=name, kind=kind, lattice=lattice, precision=precision, nx=nx, ny=ny, nz=nz,
             phi=phi, radius=radius, steps=steps, samples=samples, g=g, tune=tune,
             restart=restart)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # The smallest call: the smoke run's lattice, a handful of steps and the
        # fields and permeability, as in an interactive check or a parity test;
        # host calls, launches and synchronisations count here.
        _case("smoke_48x40x36", nx=48, ny=40, nz=36, radius=4.0, steps=20, g=1e-5),
        # The paper's lid-driven cavity (D2Q9, FP64, L = 160): the stretch between
        # two looks at the flow rate, 1000 steps of a launch-bound lattice.
        _case("cavity_160_f64", kind="cavity", lattice=9, precision="f64", nx=160, ny=160, nz=1,
              steps=1000, g=0.0),
        # The paper's pressure-driven Poiseuille flow (D2Q9, FP64, 1000 x 100).
        _case("poiseuille_1000x100_f64", kind="poiseuille", lattice=9, precision="f64", nx=1000,
              ny=100, nz=1, steps=1000, g=0.0),
        # FP64 reference run of the force-driven channel of the tests.
        _case("channel_32_f64", kind="channel", precision="f64", nx=32, ny=32, nz=32, steps=200,
              g=1e-5, restart=True),
        # FP64 reference run of a porous crop (what FP32 results are checked against).
        _case("porous_128_f64", precision="f64", nx=128, ny=128, nz=128, phi=0.6, radius=12.0,
              steps=100),
        # A segmented image rarely has extents that are multiples of 32.
        _case("ragged_150x110x90", nx=150, ny=110, nz=90, phi=0.6, radius=8.0, steps=200,
              g=1e-5),
        # The precision workload's 128^3 crop: a mid-size sample.
        _case("crop_128", nx=128, ny=128, nz=128, phi=0.6, radius=12.0, steps=2000),
        # 16-bit storage, restarted from a saved flow field.
        _case("restart_256_f16", precision="f16", nx=256, ny=256, nz=256, phi=0.6, radius=12.0,
              steps=1000, g=1e-5, tune=True, restart=True),
        # Permeability sweep at low porosity: mostly solid rows.
        _case("tight_256", nx=256, ny=256, nz=256, phi=0.1, radius=8.0, steps=1000, tune=True),
        # D3Q27 on the sweep's 256^3 lattice.
        _case("d3q27_256", lattice=27, nx=256, ny=256, nz=256, phi=0.7, radius=8.0, steps=500,
              tune=True),
        # Uneven samples advanced as one batch (sides 64 to 192, as the batch recipe draws them).
        _case("batch_12", kind="batch", nx=192, ny=192, nz=192, phi=0.65, radius=8.0, steps=1000,
              samples=12, tune=True),
        # The headline lattice: D3Q19 FP32 512^3 sphere packing, two benchmark regions.
        _case("headline_512", nx=512, ny=512, nz=512, phi=0.7, radius=12.0, steps=1000, tune=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["porous", "porous", "ragged", "ragged", "small", "f64", "16bit", "tight",
                       "batch", "cavity", "poiseuille"])
    radius = rng.uniform(4.0, 14.0)
    phi = rng.uniform(0.4, 0.95)
    lattice = rng.choice([15, 19, 19, 19, 27])
    aligned = [64, 96, 128, 160, 192, 224, 256, 288, 320, 384, 512]
    if kind == "porous":        # row lengths of the tuned lane layouts
        nx = rng.choice(aligned)
        ny, nz = _log_int(rng, 48, 320), _log_int(rng, 48, 320)
        return _case(None, nx=nx, ny=ny, nz=nz, lattice=lattice, phi=phi, radius=radius,
                     steps=rng.randint(100, 600), tune=rng.random() < 0.5)
    if kind == "ragged":        # any row length
        nx = _log_int(rng, 20, 640)
        ny, nz = _log_int(rng, 20, 200), _log_int(rng, 20, 200)
        return _case(None, nx=nx, ny=ny, nz=nz, lattice=lattice, phi=phi, radius=radius,
                     steps=rng.randint(50, 300), g=1e-5)
    if kind == "small":         # short calls on small lattices
        nx, ny, nz = (_log_int(rng, 12, 72) for _ in range(3))
        return _case(None, nx=nx, ny=ny, nz=nz, lattice=lattice, phi=phi, radius=4.0,
                     steps=rng.randint(1, 120), g=1e-5)
    if kind == "f64":
        nx, ny, nz = (_log_int(rng, 16, 160) for _ in range(3))
        return _case(None, precision="f64", nx=nx, ny=ny, nz=nz, lattice=lattice, phi=phi,
                     radius=radius, steps=rng.randint(20, 200), g=1e-5)
    if kind == "16bit":
        nx = rng.choice(aligned)
        ny, nz = _log_int(rng, 48, 256), _log_int(rng, 48, 256)
        return _case(None, precision=rng.choice(["f16", "bf16"]), nx=nx, ny=ny, nz=nz,
                     lattice=lattice, phi=phi, radius=radius, steps=rng.randint(50, 200), g=1e-5,
                     tune=rng.random() < 0.5, restart=True)
    if kind == "tight":
        nx = rng.choice([128, 192, 256, 320])
        ny, nz = _log_int(rng, 64, 256), _log_int(rng, 64, 256)
        return _case(None, nx=nx, ny=ny, nz=nz, phi=rng.uniform(0.05, 0.3),
                     radius=rng.uniform(5.0, 10.0), steps=rng.randint(100, 600), tune=True)
    if kind == "batch":
        side = rng.choice([96, 128, 160, 192, 224])
        return _case(None, kind="batch", nx=side, ny=side, nz=side, phi=phi, radius=radius,
                     samples=rng.randint(2, 12), steps=rng.randint(50, 300), tune=True)
    if kind == "cavity":
        side = _log_int(rng, 40, 400)
        return _case(None, kind="cavity", lattice=9, precision=rng.choice(["f64", "f64", "f32"]),
                     nx=side, ny=side, nz=1, steps=rng.randint(100, 1000), g=0.0)
    return _case(None, kind="poiseuille", lattice=9, precision="f64", nx=_log_int(rng, 60, 1600),
                 ny=_log_int(rng, 12, 200), nz=1, steps=rng.randint(100, 1000), g=0.0)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _packing(nx, ny, nz, radius, phi, gen):
    """Overlapping spheres at seeded centres in a periodic box, as many as give
    the porosity on average; uint8 (nz, ny, nx), 1 = solid."""
    dev = torch.device("cuda:0")
    radius = min(radius, 0.3 * min(nx, ny, nz) if nz > 1 else radius)
    n = max(1, round(-math.log(phi) * nx * ny * nz / (4.0 / 3.0 * math.pi * radius ** 3)))
    dims = torch.tensor([nx, ny, nz], dtype=torch.float64)
    centres = (torch.rand(n, 3, generator=gen, dtype=torch.float64) * dims).to(dev)
    solid = torch.zeros(nx * ny * nz, dtype=torch.uint8, device=dev)
    width = int(math.floor(2.0 * radius)) + 2
    span = torch.arange(width, device=dev)
    per = max(1, (1 << 24) // width ** 3)
    for i in range(0, n, per):
        c = centres[i:i + per]
        at = torch.floor(c - radius).long()[:, :, None] + span          # (m, 3, width)
        off = (at - c[:, :, None]) ** 2
        x, y, z = at[:, 0] % nx, at[:, 1] % ny, at[:, 2] % nz
        inside = (off[:, 2, :, None, None] + off[:, 1, None, :, None]
                  + off[:, 0, None, None, :]) <= radius * radius
        flat = (z[:, :, None, None] * ny + y[:, None, :, None]) * nx + x[:, None, None, :]
        solid[flat[inside]] = 1
    return solid.reshape(nz, ny, nx).cpu().numpy()


def _flow(solid, gen):
    """A smooth low-speed field, as a saved run holds it: (rho - 1, u), zero at
    solid nodes; a few long waves per component with seeded amplitude and phase."""
    dev = torch.device("cuda:0")
    nz, ny, nx = solid.shape
    fluid = torch.from_numpy(solid == 0).to(dev)
    axes = [torch.arange(n, device=dev, dtype=torch.float64) * (2.0 * math.pi / n)
            for n in (nz, ny, nx)]
    z, y, x = axes[0][:, None, None], axes[1][None, :, None], axes[2][None, None, :]
    fields = []
    for amp in (2e-4, 0.02, 0.01, 0.01):
        a = torch.rand(6, generator=gen, dtype=torch.float64)
        f = (torch.sin(x + 6.3 * a[0]) * (0.5 + a[1]) + torch.sin(y + 6.3 * a[2]) * (0.5 + a[3])
             + torch.sin(z + 6.3 * a[4]) * (0.5 + a[5]))
        fields.append(amp * f * fluid)
    return fields[0].cpu().numpy(), torch.stack(fields[1:]).cpu().numpy()


def _sides(case):
    """Sides of a batch's cubes: steps of 32 from 64 up to the largest, in a mixed order."""
    n = (case["nx"] - 64) // 32 + 1
    return [case["nx"] - 32 * (7 * i % n) for i in range(case["samples"])]


def _inputs(case, seed):
    """[(solid, drho0, u0)] of the case's samples and the context's options."""
    gen = torch.Generator().manual_seed(int(seed))
    nx, ny, nz, kind = case["nx"], case["ny"], case["nz"], case["kind"]
    opts = dict(g=(case["g"], 0.0, 0.0))
    if kind in ("cavity", "poiseuille"):
        t = np.zeros((1, ny, nx), np.uint8)
        t[0, 0] = 1
        t[0, -1] = 1
        if kind == "cavity":
            t[0, :, 0] = 1
            t[0, :, -1] = 1
            t[0, -1] = 2
            opts["wall_u"] = (5.0 / 12.0, 0.0, 0.0)
        else:
            opts.update(x_boundary=1, rho_in=1.01, rho_out=0.99)
        drho, u = _flow(t, gen)     # the stretch starts from a flow, not from rest
        u[2] = 0.0
        return [(t, drho, u)], opts
    if kind == "channel":
        s = np.zeros((nz, ny, nx), np.uint8)
        s[0] = 1
        s[-1] = 1
        solids = [s]
    elif kind == "batch":
        solids = []
        for side in _sides(case):
            a = torch.rand(2, generator=gen)
            solids.append(_packing(side, side, side, 4.0 + 8.0 * float(a[0]),
                                   0.4 + 0.5 * float(a[1]), gen))
    else:
        solids = [_packing(nx, ny, nz, case["radius"], case["phi"], gen)]
    if case["restart"]:
        return [(s,) + _flow(s, gen) for s in solids], opts
    return [(s, None, None) for s in solids], opts


def prepare(case, seed):
    samples, opts = _inputs(case, seed)
    sim = tau1.Sim([tau1.Sample(*s) for s in samples], lattice=case["lattice"],
                   precision=case["precision"], **opts)
    if case["tune"]:
        sim.autotune(10)
    return {"sim": sim, "case": case}


def run(state):
    sim, case = state["sim"], state["case"]
    keep = KEEP[case["precision"]]
    sim.step(case["steps"])
    out = []
    for i in range(case["samples"]):
        got = {}
        if case["g"]:
            got["k"], got["mass"] = sim.permeability(i, 0)
        drho, u = sim.moments(i)
        got["drho"] = torch.from_numpy(drho).to(keep)
        got["u"] = torch.from_numpy(u).to(keep)
        out.append(got)
    return out


def work(case):
    """A step reads and writes the (d + 1) state values of every fluid node once
    and reads one mask bit per node; the fields come back once as FP64 arrays."""
    nodes = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "batch":
        nodes = sum(s ** 3 for s in _sides(case))
    phi = case["phi"] if case["kind"] == "porous" else 0.65 if case["kind"] == "batch" else 1.0
    dims = 2 if case["lattice"] == 9 else 3
    fluid = nodes * phi
    step = 2.0 * (dims + 1) * BYTES[case["precision"]] * fluid + nodes / 8.0
    # per direction: the equilibrium (4) and its sums (3); per node about 16 more
    return {"bytes": case["steps"] * step + 32.0 * nodes,
            "flops": case["steps"] * fluid * (7.0 * case["lattice"] + 16.0)}


# ---------------------------------------------------------------------------
# The same update in plain FP64 torch
# ---------------------------------------------------------------------------
def _directions(lattice):
    """[(c, weight)] of the DdQq set, the rest direction first."""
    weights = {9: {0: 4 / 9, 1: 1 / 9, 2: 1 / 36},
               15: {0: 2 / 9, 1: 1 / 9, 3: 1 / 72},
               19: {0: 1 / 3, 1: 1 / 18, 2: 1 / 36},
               27: {0: 8 / 27, 1: 2 / 27, 2: 1 / 54, 3: 1 / 216}}[lattice]
    zs = (0,) if lattice == 9 else (0, 1, -1)
    found = [((x, y, z), weights[abs(x) + abs(y) + abs(z)])
             for z in zs for y in (0, 1, -1) for x in (0, 1, -1)
             if abs(x) + abs(y) + abs(z) in weights]
    return sorted(found, key=lambda f: f[0] != (0, 0, 0))


def _exact_sample(case, solid, drho, u, opts):
    dev = torch.device("cuda:0")
    types = torch.from_numpy(solid).to(dev)
    shape = types.shape
    wall = types != 0
    fluid = (~wall).to(torch.float64)
    half = [0.5 * g for g in opts["g"]]
    zero = torch.zeros(shape, dtype=torch.float64, device=dev)
    d = zero.clone() if drho is None else torch.from_numpy(drho).to(dev) * fluid
    v = [((zero if u is None else torch.from_numpy(u[a]).to(dev)) + half[a]) * fluid
         for a in range(3)]
    dirs = _directions(case["lattice"])

    def shifted(t, c):
        for axis in range(3):
            if c[2 - axis]:
                t = torch.roll(t, c[2 - axis], axis)
        return t

    links = {}
    for c, _ in dirs[1:]:
        links[c] = shifted(wall, tuple(-a for a in c)) & ~wall      # x + c is solid
    moving, uw = {}, opts.get("wall_u", (0.0, 0.0, 0.0))
    if any(uw):
        for c, _ in dirs[1:]:
            moving[c] = shifted(types == 2, tuple(-a for a in c)) & ~wall
    pressure = opts.get("x_boundary", 0)
    for _ in range(case["steps"]):
        rho = 1.0 + d
        r3, r45 = 3.0 * rho, 4.5 * rho
        base = v[0] * v[0]
        base.addcmul_(v[1], v[1]).addcmul_(v[2], v[2])
        base = torch.addcmul(d, rho, base, value=-1.5)
        nd = dirs[0][1] * base
        j = [torch.zeros_like(d) for _ in range(3)]
        inlet, outlet = (nd.clone(), nd.clone()) if pressure else (None, None)
        for c, w in dirs[1:]:
            cu = None
            for a in range(3):
                if c[a]:
                    cu = c[a] * v[a] if cu is None else cu.add_(v[a], alpha=c[a])
            f = torch.addcmul(r3, r45, cu).mul_(cu).add_(base).mul_(w)
            back = f * links[c]
            if moving:
                back.add_(rho * moving[c], alpha=-6.0 * w * sum(c[a] * uw[a] for a in range(3)))
            f = shifted(f, c)
            if pressure:
                # populations along c arrive at x; those returned at x travel along -c
                for s, sign in ((inlet, -1), (outlet, 1)):
                    for t, cx in ((f, c[0]), (back, -c[0])):
                        if cx == 0 or cx == sign:
                            s.add_(t, alpha=1.0 if cx == 0 else 2.0)
            nd.add_(f).add_(back)
            for a in range(3):
                if c[a]:
                    j[a].add_(f, alpha=c[a]).sub_(back, alpha=c[a])
        d = nd.mul_(fluid)
        v = [(j[a].div_(1.0 + d) + 2.0 * half[a]) * fluid for a in range(3)]
        if pressure:
            for col, db, sign, s in ((0, opts["rho_in"] - 1.0, 1.0, inlet),
                                     (-1, opts["rho_out"] - 1.0, -1.0, outlet)):
                m = fluid[:, :, col]
                d[:, :, col] = db * m
                v[0][:, :, col] = (sign * (db - s[:, :, col]) / (1.0 + db) + 2.0 * half[0]) * m
                v[1][:, :, col] = 2.0 * half[1] * m
    got = {}
    out_u = torch.stack([(v[a] - half[a]) * fluid for a in range(3)])
    if case["g"]:
        nodes = float(fluid.numel())
        got["k"] = float(out_u[0].sum()) / nodes / 6.0 / case["g"]
        got["mass"] = float(fluid.sum() + d.sum())
    keep = torch.float64
    got["drho"], got["u"] = d.to(keep).cpu(), out_u.to(keep).cpu()
    return got


def exact(case, seed):
    # the plain FP64 update takes about 6e-11 s per node, direction and step: none
    # where that comes to more than about 20 s
    if work(case)["flops"] / 7.0 > 3.3e11:
        return None
    samples, opts = _inputs(case, seed)
    return [_exact_sample(case, s, d, u, opts) for s, d, u in samples]
