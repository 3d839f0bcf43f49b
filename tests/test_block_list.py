"""The block list of the stencil passes, on the host (block_list_check.cpp): every plane of every
sub-tile is covered once by the update its columns ask for, s33 is stored on the planes of fluid
tiles that general tiles read, every receiver's increment lies where the stress pass reads it, and
the list keeps to its room; a list that would outgrow it is refused.  No GPU is touched."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1709_02733_amd import build as B
from paper_1709_02733_amd import el
from tests import large_media as LM

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("block_list") / "check.so")
    subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I" + os.path.join(B.ROOT, "include"), "-I" + B.CSRC, os.path.join(HERE, "block_list_check.cpp"),
                    "-x", "none", B.LIB, "-Wl,-rpath," + B.PKG, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.check_message.restype = ctypes.c_char_p

    def run(solid, npml=2, fluid=True, nrec=40, seed=0, medium=None, room=0):
        nz, ny, nx = solid.shape
        solid = np.ascontiguousarray(solid, np.uint8)
        medium = np.ascontiguousarray(solid if medium is None else medium, np.uint8)
        rng = np.random.default_rng(seed)
        base = np.stack([rng.integers(0, n - 1, nrec) for n in (nx, ny, nz)], 1)
        corners = np.array([[c & 1, c >> 1 & 1, c >> 2 & 1] for c in range(8)])
        pts = np.unique((base[:, None] + corners).reshape(-1, 3), axis=0)
        pts = np.ascontiguousarray(pts[np.lexsort((pts[:, 0], pts[:, 1], pts[:, 2]))], np.int32)
        out = np.zeros(6, np.int32)
        ptr = [a.ctypes.data_as(ctypes.c_void_p) for a in (solid, medium, pts, out)]
        rc = lib.check_blocks(nx, ny, nz, npml, ptr[0], ptr[1], int(fluid), ptr[2], len(pts), nrec, room, ptr[3])
        assert rc in (0, 2), lib.check_message().decode()
        return rc, dict(zip(("depth", "per", "cap", "general", "once", "touched"), out.tolist()))

    return run


def _medium(rng, shape_xyz):
    """Solid cells and media of a random kind: none, all, a ball, clumps, slabs, scattered cells."""
    nx, ny, nz = shape_xyz
    shp = (nz, ny, nx)
    kind = rng.integers(0, 6)
    z, y, x = np.ogrid[:nz, :ny, :nx]
    solid = np.zeros(shp, bool)
    if kind == 1:
        solid[:] = True
    elif kind in (2, 3):
        for _ in range(1 if kind == 2 else 6):
            c = rng.uniform(size=3) * (nx, ny, nz)
            r = rng.uniform(1, 0.4 * max(shp))
            solid |= (x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2 <= r * r
    elif kind == 4:
        a = rng.integers(0, nz, 4)
        for k in a:
            solid[k:k + int(rng.integers(1, 9))] = True
    elif kind == 5:
        solid = rng.uniform(size=shp) < rng.choice([1e-4, 1e-3, 1e-2])
    medium = solid.astype(np.uint8)
    if rng.integers(0, 2):
        medium[:, :, : nx // 2] += 2   # two fluids
    return solid, medium


def test_random_grids(check):
    rng = np.random.default_rng(12)
    for n in range(160):
        shape = tuple(int(v) for v in np.exp(rng.uniform(np.log(4), np.log((150, 70, 90)))))
        solid, medium = _medium(rng, shape)
        npml = int(rng.integers(0, max(1, min(6, (min(shape) - 2) // 2) + 1)))
        for fluid in (True, False):
            assert check(solid, npml, fluid, int(rng.integers(1, 80)), n, medium)[0] == 0, (n, shape)


@pytest.mark.parametrize("shape,solid,depth", [
    ((64, 4096, 19), 0, 2),      # chunks of six planes, blocks of two
    ((64, 8192, 7), 0, 2), ((2048, 256, 7), 0, 2),
    ((64, 4096, 19), 1, 4), ((64, 6000, 25), 0, 4),
    ((256, 130, 160), 1, 8), ((256, 256, 90), 0, 4), ((128, 128, 128), 1, 4), ((96, 96, 96), 1, 2)])
def test_shapes(check, shape, solid, depth):
    s = np.full(shape[::-1], solid, np.uint8)
    for fluid in (True, False):
        rc, got = check(s, 0, fluid, 500)
        assert rc == 0
        if fluid:
            assert got["depth"] == depth


def test_a_list_that_outgrows_its_room_is_refused(check):
    s = np.zeros((40, 70, 90), np.uint8)
    s[15:25, 20:50, 20:70] = 1
    rc, got = check(s)
    assert rc == 0
    assert check(s, room=got["per"])[0] == 0
    for room in (got["per"] - 1, got["per"] // 2, 1):
        assert check(s, room=room)[0] == 2


def test_the_state_that_a_step_touches(check):
    """All general: every cell's 13 arrays and six memory variables of each layer it is in (one cell more
    than npml on every face); all one fluid: 4 arrays and two of them.  The passes stream from 256 MiB on
    (float elements)."""
    for shape, npml in (((70, 21, 40), 3), ((64, 64, 64), 0), ((33, 9, 8), 2), ((160, 160, 160), 16), ((152, 152, 152), 16)):
        nx, ny, nz = shape
        lay = sum(2 * (npml + 1) * nx * ny * nz // n for n in shape) if npml else 0
        for solid, arrays, memory in ((1, 13, 6), (0, 4, 2)):
            got = check(np.full(shape[::-1], solid, np.uint8), npml)[1]
            want = arrays * nx * ny * nz + memory * lay
            assert got["touched"] == want // 1000 and got["once"] == int(4 * want > 2 ** 28)
            off = check(np.full(shape[::-1], solid, np.uint8), npml, fluid=False)[1]
            assert off["touched"] == (13 * nx * ny * nz + 6 * lay) // 1000


@pytest.mark.parametrize("case", range(len(LM.CASES)))
def test_large_media_take_the_path_they_are_meant_for(check, case):
    """The media that test_gpu_large.py runs: planes per block, streaming, room, with fluid tiles,
    fluid sub-tiles and general ones where they are meant to be mixed."""
    shape, npml, fluid, radius, size, depth, once = LM.CASES[case]
    solid = LM.clumps(shape, fluid, radius)
    rc, got = check(solid, npml, nrec=300)
    assert rc == 0 and got["depth"] == depth
    assert (got["touched"] * 1000 * size > 2 ** 28) == once
    assert not fluid or 20 < got["general"] < 980
    assert got["per"] <= got["cap"]


def test_boxes_that_need_more_than_their_room_give_way_to_bands(check):
    """A 96^3 grid deals its pieces to the XCDs in boxes; half of it solid, the fullest box has more
    entries than the fullest band."""
    s = np.zeros((96, 96, 96), np.uint8)
    s[:48] = 1
    boxes = check(s, 16)[1]
    rc, bands = check(s, 16, room=boxes["per"] - 1)
    assert rc == 0 and bands["per"] < boxes["per"] <= boxes["cap"]


def test_workspace_of_a_small_plan():
    """A 96^3 plan with 512 receivers took 103.4 MB with a list of tiles; its block lists and increments
    add 6% at most."""
    assert el.plan_bytes(el.make_grid(96, 96, 96, 1e-4, 1e-8, 10, 16), 512) < 1.06 * 103.4e6


def test_sizing_a_flat_grid_takes_no_time():
    """el_plan_bytes bounds the block lists band by band, not tile row by plane (26 ms for this grid)."""
    import time
    g = el.make_grid(30, 5000, 5000, 1e-4, 1e-8, 10, 2)
    best = 1.0
    for _ in range(10):
        t = time.perf_counter()
        el.plan_bytes(g, 100)
        best = min(best, time.perf_counter() - t)
    assert best < 5e-3
