"""3D labeling at the sizes where its tiles (64 x 16 x 8 voxels, 4 slices under
6-connectivity) and their two-row, two-slice bundles begin, end and are cut,
against the 3D oracle, bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_3d import _cmp, noise

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 65), (1, 17, 64), (2, 16, 63), (3, 15, 129), (4, 33, 66), (5, 2, 192), (7, 31, 65), (8, 16, 64),
          (9, 17, 65), (16, 32, 128), (17, 33, 130), (25, 1, 70), (12, 48, 1)]


@pytest.mark.parametrize("conn", [6, 18, 26])
@pytest.mark.parametrize("p", [0.06, 0.2, 0.33, 0.6, 0.9])
def test_3d_tile_edges(conn, p):
    for k, shape in enumerate(SHAPES):
        _cmp(noise(shape, p, 9300 + k), conn, what="tile edges p=%.2f" % p)


@pytest.mark.parametrize("conn", [6, 18, 26])
def test_3d_dense_joins(conn):
    """Most intervals per bundle and most joins per tile: separate columns and
    planes, and the same joined once at a far corner."""
    D, H, W = 17, 33, 131
    zz, yy, xx = np.indices((D, H, W))
    for what, vol in (("planes x", xx % 2 == 0), ("rods z", (xx % 2 == 0) & (yy % 2 == 0)),
                      ("rods z, shifted", (xx + yy) % 2 == 0), ("rods y", (xx + zz) % 2 == 0),
                      ("corner touches", (xx % 2 == 0) & ((yy + zz + xx // 2) % 2 == 0)),
                      ("blocks", ((xx // 2) + (yy // 2) + (zz // 2)) % 2 == 0)):
        vol = vol.astype(np.uint8)
        _cmp(vol, conn, what=what)
        vol[D - 1, H - 1, :] = 1
        _cmp(vol, conn, what=what + ", joined")


@pytest.mark.parametrize("conn", [6, 18, 26])
def test_3d_pairs_across_corners(conn):
    """Two voxels at every offset around a tile corner, nothing else set."""
    for base in ((8, 16, 64), (4, 16, 64), (8, 15, 63)):
        cells = [(dz, dy, dx) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dz, dy, dx) != (0, 0, 0)]
        # stacked with empty slices between; every slab keeps the corner's
        # position modulo the tile (8 slices)
        vol = np.zeros((16 * len(cells), 32, 128), np.uint8)
        for i, (dz, dy, dx) in enumerate(cells):
            z, y, x = 16 * i + base[0], base[1], base[2]
            vol[z, y, x] = 1
            vol[z + dz, y + dy, x + dx] = 1
        _cmp(vol, conn, what="corner pairs at %s" % (base,))


def test_3d_near_threshold():
    _cmp(noise((64, 128, 256), 0.16, 9400), 18, what="noise near the threshold")
