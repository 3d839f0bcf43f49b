"""Media of large grids for the tests of the block list and of the passes that it selects."""
import numpy as np

from paper_1709_02733_amd import scenarios as S


def clumps(shape_xyz, fluid: float, radius: float, seed: int = 5) -> np.ndarray:
    """Solid cells (nz, ny, nx) of a grid with fluid ellipsoids, three times as long along x (as a tile
    is wide), until their volumes add up to `fluid` of it."""
    rng = np.random.default_rng(seed)
    nx, ny, nz = shape_xyz
    solid = np.ones((nz, ny, nx), bool)
    r, rx = int(radius), int(3 * radius)
    z, y, x = np.ogrid[-r:r + 1, -r:r + 1, -rx:rx + 1]
    ball = (x / 3.0) ** 2 + y * y + z * z <= radius * radius
    for _ in range(int(fluid * nx * ny * nz / ball.sum())):
        c = [int(rng.integers(0, n)) for n in (nz, ny, nx)]
        lo = [max(v - q, 0) for v, q in zip(c, (r, r, rx))]
        hi = [min(v + q + 1, n) for v, q, n in zip(c, (r, r, rx), (nz, ny, nx))]
        part = ball[tuple(slice(a - v + q, b - v + q) for a, b, v, q in zip(lo, hi, c, (r, r, rx)))]
        solid[tuple(slice(a, b) for a, b in zip(lo, hi))] &= ~part
    return solid


# shape (x, y, z), npml, fluid part, radius of its ellipsoids, element bytes, planes per block, streaming
CASES = [
    ((192, 200, 190), 3, 0.30, 18.0, 4, 8, True),
    ((192, 180, 180), 0, 0.0, 1.0, 4, 8, True),
    ((128, 150, 170), 6, 0.90, 30.0, 8, 4, True),
    ((128, 120, 140), 4, 0.80, 20.0, 4, 4, False),
]


def scenario(shape_xyz, npml: int, fluid: float, radius: float, nsteps: int = 5, nrec: int = 300):
    sc = S.random_scenario(shape_xyz, seed=9, nsteps=nsteps, npml=npml, nrec=nrec, fluid_fraction=0.0)
    solid = clumps(shape_xyz, fluid, radius)
    sc.mu[~solid] = 0.0
    sc.lam[~solid] = 2.25e9
    sc.rho[~solid] = 1000.0
    sc.alpha[~solid] = 0.0
    return sc, solid
