"""One Tau1 step in numpy, direction by direction in the lattice's order with
every operation rounded by itself, in FP64 or FP32 (storage FP32 or scaled
half): the arithmetic of the kernels that work node by node."""
import numpy as np

import oracle

WEIGHTS = {15: (2.0 / 9.0, 1.0 / 9.0, 0.0, 1.0 / 72.0),
           19: (1.0 / 3.0, 1.0 / 18.0, 1.0 / 36.0, 0.0),
           27: (8.0 / 27.0, 2.0 / 27.0, 1.0 / 54.0, 1.0 / 216.0)}
HALF = 2.0 ** 16       # default scale of the half storage


def store(x, prec):
    """x as the state holds it, back in the compute type."""
    if prec == "f16":
        return (x * np.float32(HALF)).astype(np.float16).astype(np.float32) * np.float32(1 / HALF)
    return x


def start(solid, drho, u, g, prec):
    """Initial state (drho, v = u + g/2)."""
    T = np.float64 if prec == "f64" else np.float32
    fl = solid == 0
    gh = [T(0.5 * x) for x in g]
    d = np.where(fl, drho.astype(T), T(0))
    v = np.stack([np.where(fl, u[a].astype(T) + gh[a], T(0)) for a in range(3)])
    return store(d, prec), store(v, prec)


def step(q, solid, d, v, g, prec):
    T = np.float64 if prec == "f64" else np.float32
    gh = [T(0.5 * x) for x in g]
    one, three, c45, c15 = T(1), T(3), T(4.5), T(1.5)
    n, j = np.zeros_like(d), np.zeros_like(v)
    for c in oracle.lattice(q)[0]:
        cx, cy, cz = (int(x) for x in c)
        w = T(WEIGHTS[q][abs(cx) + abs(cy) + abs(cz)])

        def src(a):
            return np.roll(a, (cz, cy, cx), axis=(0, 1, 2))

        wall = src(solid) != 0
        ds = np.where(wall, d, src(d))
        vx, vy, vz = (np.where(wall, v[a], src(v[a])) for a in range(3))
        sign = np.where(wall, T(-1), T(1))
        rho = one + ds
        cu = (sign * T(cx) * vx + sign * T(cy) * vy) + sign * T(cz) * vz
        vv = (vx * vx + vy * vy) + vz * vz
        p = (three * cu + (c45 * cu) * cu) - c15 * vv
        f = w * (ds + rho * p)
        n = n + f
        j = np.stack([j[0] + T(cx) * f, j[1] + T(cy) * f, j[2] + T(cz) * f])
    r = one / (one + n)
    out = np.stack([(j[a] * r + gh[a]) + gh[a] for a in range(3)])
    fl = solid == 0
    return store(np.where(fl, n, T(0)), prec), store(np.where(fl, out, T(0)), prec)


def fields(solid, d, v, g):
    """What the library reads back: drho and u = v - g/2 in FP64."""
    fl = solid == 0
    u = np.stack([np.where(fl, v[a].astype(np.float64) - 0.5 * g[a], 0.0) for a in range(3)])
    return d.astype(np.float64), u
