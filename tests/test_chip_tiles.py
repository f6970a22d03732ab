"""Tiles of the on-chip Krylov runs, on the CPU: the library's partition of a
grid (its own function, no GPU), and the index arithmetic of the kernel redone
here.  Every unknown belongs to one tile; every staged cell and exchange slot
lies in its buffer; what a tile publishes in a slot is the node its neighbour
takes from there."""
import ctypes
import os

import numpy as np
import pytest

from paper_1711_04060_amd import pf

NT, LP, GMAX = 512, 616, 256


class Geom(ctypes.Structure):
    _fields_ = [("KZ", ctypes.c_int), ("o", ctypes.c_int * 3), ("n", ctypes.c_int * 3), ("c", ctypes.c_int * 3),
                ("G", ctypes.c_int), ("fx", ctypes.c_int), ("fy", ctypes.c_int), ("fz", ctypes.c_int),
                ("fstride", ctypes.c_int)]


def partition(nx, ny, nz, neu, cap=GMAX, kzmax=16):
    if not os.path.exists(pf.LIB_PATH):
        pytest.skip("library not built")
    f = getattr(ctypes.CDLL(pf.LIB_PATH), "_ZN3pfk14chip_partitionEiiiiii")
    f.restype, f.argtypes = Geom, [ctypes.c_int] * 6
    return f(nx, ny, nz, neu, cap, kzmax)


def halo_slots(kz):
    return 1 if kz <= 4 else 2 if kz <= 8 else 3


def face_slots(kz):
    return 3 if kz <= 4 else 4 if kz <= 8 else 5


def tile(ge, lb):
    cx, cy, _ = ge.c
    t = (lb % cx, lb // cx % cy, lb // (cx * cy))
    at = [ge.o[a] + t[a] * ge.n[a] // ge.c[a] for a in range(3)]
    size = [ge.o[a] + (t[a] + 1) * ge.n[a] // ge.c[a] - at[a] for a in range(3)]
    return t, at, size


def check(nx, ny, nz, neu, cap=GMAX, kzmax=16):
    ge = partition(nx, ny, nz, neu, cap, kzmax)
    if ge.KZ == 0:
        return False
    cx, cy, cz = ge.c
    fx, fy, fz, fs = ge.fx, ge.fy, ge.fz, ge.fstride
    assert ge.KZ in (4, 8, 16) and ge.KZ <= kzmax
    assert ge.G == cx * cy * cz <= min(cap, GMAX)
    assert fs == 2 * (fx + fy + fz) <= face_slots(ge.KZ) * NT
    assert fx % 32 == fy % 32 == fz % 32 == 0          # whole cache lines of any element
    owner = np.full((nz, ny, nx), -1)
    pub = np.full((ge.G, fs), -1)
    node = lambda x, y, z: x + nx * (y + ny * z)   # noqa: E731
    zlo, zhi = 2 * (fx + fy), 2 * (fx + fy) + fz
    for lb in range(ge.G):
        (tx, ty, tz), (x0, y0, z0), (bx, by, nk) = tile(ge, lb)
        assert bx * by <= NT and 1 <= nk <= ge.KZ and (bx + 2) * (by + 2) <= LP - 1
        assert (cx == 1 or bx >= 2) and (cy == 1 or by >= 2)
        own = owner[z0:z0 + nk, y0:y0 + by, x0:x0 + bx]
        assert own.size == bx * by * nk and (own == -1).all()
        own[:] = lb
        # mirror neighbours of a face on the grid's edge lie inside the tile
        assert not ((x0 == 0 or x0 + bx == nx) and bx < 2) and not ((y0 == 0 or y0 + by == ny) and by < 2)
        k, j = np.divmod(np.arange(by * nk), by)
        if tx > 0:
            pub[lb, :by * nk] = node(x0, y0 + j, z0 + k)
        if tx < cx - 1:
            pub[lb, fx:fx + by * nk] = node(x0 + bx - 1, y0 + j, z0 + k)
        k, i = np.divmod(np.arange(bx * nk), bx)
        if ty > 0:
            pub[lb, 2 * fx:2 * fx + bx * nk] = node(x0 + i, y0, z0 + k)
        if ty < cy - 1:
            pub[lb, 2 * fx + fy:2 * fx + fy + bx * nk] = node(x0 + i, y0 + by - 1, z0 + k)
        j, i = np.divmod(np.arange(bx * by), bx)
        if tz > 0:
            pub[lb, zlo:zlo + bx * by] = node(x0 + i, y0 + j, z0)
        if tz < cz - 1:
            pub[lb, zhi:zhi + bx * by] = node(x0 + i, y0 + j, z0 + nk - 1)
    assert (owner >= 0).sum() == ge.n[0] * ge.n[1] * ge.n[2]
    for lb in range(ge.G):
        (tx, ty, tz), (x0, y0, z0), (bx, by, nk) = tile(ge, lb)
        W = bx + 2
        h1 = by * nk
        h = np.arange(2 * (h1 + bx * nk))
        assert h.size <= halo_slots(ge.KZ) * NT
        cells = []
        for up in (0, 1):   # x, then y halo, as the kernel decodes its slots
            e = np.arange(h1)
            k, j = np.divmod(e, by)
            if (tx < cx - 1) if up else (tx > 0):
                assert (pub[lb + (1 if up else -1), (0 if up else fx) + e]
                        == node(x0 + (bx if up else -1), y0 + j, z0 + k)).all()
                cells.append(k * LP + (j + 1) * W + (bx + 1 if up else 0))
            e = np.arange(bx * nk)
            k, i = np.divmod(e, bx)
            if (ty < cy - 1) if up else (ty > 0):
                assert (pub[lb + (cx if up else -cx), 2 * fx + (0 if up else fy) + e]
                        == node(x0 + i, y0 + (by if up else -1), z0 + k)).all()
                cells.append(k * LP + ((by + 1) if up else 0) * W + i + 1)
            z = np.arange(bx * by)
            j, i = np.divmod(z, bx)
            if (tz < cz - 1) if up else (tz > 0):
                assert (pub[lb + (cx * cy if up else -cx * cy), (zlo if up else zhi) + z]
                        == node(x0 + i, y0 + j, z0 + (nk if up else -1))).all()
        if cells:
            c = np.concatenate(cells)
            assert len(np.unique(c)) == c.size and (c % LP < LP - 1).all() and c.max() < ge.KZ * LP
    return True


@pytest.mark.parametrize("neu", [0, 0b001111, 0b111111, 0b010110])
def test_tiles_of_small_and_ragged_grids(neu):
    rng = np.random.default_rng(neu)
    for nx, ny, nz in [(3, 3, 3), (5, 4, 3), (4, 29, 31), (130, 5, 9), (7, 131, 6), (6, 7, 133)]:
        assert check(nx, ny, nz, neu)
    for _ in range(25):
        n = rng.integers(3, 120, 3)
        check(*(int(v) for v in n), neu, cap=int(rng.choice([256, 256, 64, rng.integers(1, 257)])),
              kzmax=int(rng.choice([8, 16])))


@pytest.mark.parametrize("n", [17, 33, 49, 65, 81, 97, 113, 129])
def test_cubes_of_the_workloads_fit(n):
    assert check(n, n, n, 0)
    assert check(n, n, n, 0b001111) == (n < 129)      # 129 x 129 x 127 unknowns are more than the tiles hold


def test_what_does_not_fit():
    assert not check(161, 161, 161, 0)
    assert not check(129, 129, 129, 0, kzmax=8)
    assert not check(33, 33, 33, 0, cap=1)
