"""The traversal where rays meet edges and corners of voxels: returns and sensors on a
lattice of voxel fractions, against the oracle (needs an MI355X).  Integers and height
bits are compared exactly, by the comparison rules of the other parity tests."""
import numpy as np
import pytest

from conftest import params
from parity_util import Pair, compare_all

pytestmark = pytest.mark.gpu

EYE = np.eye(3, dtype=np.float32)


def _pose(t):
    return np.concatenate([EYE, np.asarray(t, np.float32)[:, None]], 1).reshape(12)


@pytest.mark.parametrize("distinct", [False, True])
@pytest.mark.parametrize("dims,seg_len,frac", [
    ((16, 16, 16), 1, 1),        # every segment one move long; corners only
    ((24, 18, 12), 8, 1),
    ((24, 18, 12), 8, 2),        # sensor in the middle of voxels
    ((40, 26, 7), 5, 4),
    ((130, 6, 5), 8, 2),         # long along one axis: rays of 17 segments
    ((6, 130, 40), 1024, 2),     # one segment per ray
    ((20, 22, 128), 8, 1),
])
def test_lattice_rays(dims, seg_len, frac, distinct):
    nx, ny, nz = dims
    res = 0.25  # a power of two: lattice points are exact in world coordinates
    rng = np.random.default_rng(nx + 10 * ny + 100 * nz + frac)
    pair = Pair(params(nx, ny, nz, res, szv=nz // 2), seg_len)
    try:
        for k in range(3):  # the storage wrap moves through the window
            # on the lattice: boundaries (frac 1), boundaries and middles (2), quarters (4)
            cell = rng.integers(-40, 40, 3) if k else np.zeros(3, int)
            s = (cell + rng.integers(0, frac, 3) / frac) * res
            d = rng.integers(-12 * frac, 12 * frac + 1, (1500, 3)) * np.array([nx, ny, nz]) // 20
            d[rng.uniform(size=d.shape) < 0.2] = 0       # rays in planes and along axes
            d[:100, 1] = d[:100, 0]                      # diagonals: two or three axes at once
            d[100:200, 2] = -d[100:200, 0]
            d[200:300, 1], d[200:300, 2] = d[200:300, 0], d[200:300, 0]
            d[300] = 0                                   # ends in the sensor's point
            pts = (d / frac * res).astype(np.float32)
            assert pair.insert(pts, _pose(s), 1 | (2 if distinct else 0)) == 0
            compare_all(pair, distinct=distinct)
    finally:
        pair.close()


@pytest.mark.parametrize("seg_len", [1, 2])
def test_short_rays_over_the_storage_wrap(seg_len):
    """Rays whose dominant axis makes one or two moves while another makes as many, so
    that the other runs up to any number of times faster between them, at every offset
    of the storage's ring: sensors close to a voxel's faces, returns close to faces one
    and two voxels away."""
    nx, ny, nz, res = 6, 10, 5, 0.25
    rng = np.random.default_rng(seg_len)
    eps = 2.0 ** -16  # one unit of the fixed-point coordinates
    pair = Pair(params(nx, ny, nz, res, szv=2), seg_len)
    try:
        for k in range(2 * ny):
            cell = np.array([k % nx, k, -k % nz]) + (rng.integers(-2, 3, 3) if k % 3 == 0 else 0)
            face = rng.choice([eps, 0.0, 0.5, 1 - eps], 3)
            s = (cell + face) * res
            step = rng.integers(-2, 3, (400, 3))
            end = cell + step + rng.choice([0.0, eps, 2 * eps, 0.5, 1 - eps], (400, 3))
            pts = (end * res - s).astype(np.float32)
            assert pair.insert(pts, _pose(s), 1) == 0
        compare_all(pair)
    finally:
        pair.close()
