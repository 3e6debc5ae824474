"""One Tau1 step in numpy, FP64: direction by direction in the lattice's order with
every operation rounded by itself, as kernel 0 does in FP64 mode."""
import numpy as np

import oracle

WEIGHTS = {15: (2.0 / 9.0, 1.0 / 9.0, 0.0, 1.0 / 72.0),
           19: (1.0 / 3.0, 1.0 / 18.0, 1.0 / 36.0, 0.0),
           27: (8.0 / 27.0, 2.0 / 27.0, 1.0 / 54.0, 1.0 / 216.0)}


def start(solid, drho, u, g):
    """Initial state (drho, v = u + g/2)."""
    fl = solid == 0
    return drho * fl, np.stack([np.where(fl, u[a] + 0.5 * g[a], 0.0) for a in range(3)])


def step(q, solid, d, v, g):
    gh = [0.5 * x for x in g]
    n, j = np.zeros_like(d), np.zeros_like(v)
    for c in oracle.lattice(q)[0]:
        cx, cy, cz = (int(x) for x in c)
        w = WEIGHTS[q][abs(cx) + abs(cy) + abs(cz)]

        def src(a):
            return np.roll(a, (cz, cy, cx), axis=(0, 1, 2))

        wall = src(solid) != 0
        ds = np.where(wall, d, src(d))
        vx, vy, vz = (np.where(wall, v[a], src(v[a])) for a in range(3))
        sign = np.where(wall, -1.0, 1.0)
        cu = (sign * cx * vx + sign * cy * vy) + sign * cz * vz
        vv = (vx * vx + vy * vy) + vz * vz
        p = (3.0 * cu + (4.5 * cu) * cu) - 1.5 * vv
        f = w * (ds + (1.0 + ds) * p)
        n = n + f
        j = np.stack([j[0] + cx * f, j[1] + cy * f, j[2] + cz * f])
    r = 1.0 / (1.0 + n)
    out = np.stack([(j[a] * r + gh[a]) + gh[a] for a in range(3)])
    fl = solid == 0
    return np.where(fl, n, 0.0), np.where(fl, out, 0.0)


def fields(solid, d, v, g):
    """What the library reads back: drho and u = v - g/2."""
    fl = solid == 0
    return d, np.stack([np.where(fl, v[a] - 0.5 * g[a], 0.0) for a in range(3)])
