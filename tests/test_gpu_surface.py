"""The slope / roughness / negative-obstacle pass on hand-made height fields
against the oracle: window sizes around the edges of its 16-, 32- and 64-pixel
tiles, search distances on both sides of 31 and at the largest one, other fit
windows, sparse and dense maps, and imported heights far outside their voxels
(needs an MI355X).  The comparison rule is parity_util's: flags equal, slope
and roughness within 1e-5."""
import numpy as np
import pytest
import torch

from parity_util import compare_2d_arrays, host_2d

pytestmark = pytest.mark.gpu


def _field(nx, ny, nz, rng, fill, wild):
    """Lookup table and data array with at most one return per column: a smooth
    surface with steps, `fill` of the columns known, some clustered gaps."""
    x, y = np.meshgrid(np.arange(nx), np.arange(ny), indexing="ij")
    z = nz / 2 + nz / 5 * np.sin(x / 9.0 + rng.uniform(0, 6)) * np.cos(y / 7.0 + rng.uniform(0, 6))
    z = np.clip(z + (rng.uniform(size=z.shape) < 0.03) * rng.integers(-nz // 3, nz // 3 + 1, z.shape),
                0, nz - 1).astype(np.int64)
    known = rng.uniform(size=z.shape) < fill
    for _ in range(6):  # gaps wider than the search
        cx, cy = rng.integers(nx), rng.integers(ny)
        r = rng.integers(1, max(2, min(40, min(nx, ny) // 5)))
        known &= (x - cx) ** 2 + (y - cy) ** 2 > r * r
    lut = np.full((nx, ny, nz), -1, np.int32)
    idx = np.argwhere(known)
    lut[idx[:, 0], idx[:, 1], z[known]] = np.arange(len(idx))
    data = np.zeros((len(idx), 3), np.int32)
    data[:, 0] = 1
    if wild:  # any height the data array can hold
        data[:, 2] = rng.integers(-2 ** 31 + 1, 2 ** 31 - 1, len(idx))
    else:
        data[:, 2] = (z[known] << 16) + rng.integers(0, 65536, len(idx))
    return lut.reshape(-1), data


@pytest.mark.parametrize("nx,ny,nz,res,search,fit,fill,wild", [
    (2, 2, 4, 0.2, 1.0, 5, 0.9, False),        # smaller than any halo
    (16, 34, 8, 0.2, 0.2, 5, 0.5, False),      # search of one ring; halo = fit window
    (66, 94, 16, 0.2, 6.2, 5, 0.3, False),     # 31 rings, the last of the near lookup
    (130, 62, 16, 0.2, 6.4, 5, 0.02, False),   # 32 rings, mostly gaps
    (98, 126, 16, 0.1, 6.4, 5, 0.005, False),  # 64 rings, the most
    (130, 130, 16, 0.2, 5.0, 3, 0.4, False),
    (62, 98, 16, 0.2, 2.0, 15, 0.6, False),
    (64, 64, 16, 0.2, 5.0, 5, 0.5, True),
    (354, 278, 8, 0.25, 5.0, 5, 0.35, False),  # two 16-pixel tiles per compute unit
    (514, 386, 8, 0.2, 5.0, 5, 0.3, False),    # 32-pixel tiles
    (1030, 1026, 4, 0.2, 5.0, 5, 0.2, False),  # 64-pixel tiles
    (1026, 1030, 12, 0.1, 5.0, 5, 0.01, False),
])
def test_surface_matches_oracle(nx, ny, nz, res, search, fit, fill, wild):
    import oracle
    from paper_2109_13176_amd import gvom
    rng = np.random.default_rng(nx * 7 + ny)
    p = dict(nx=nx, ny=ny, nz=nz, res_m=res, sensor_z_voxel=nz // 2, obs_min_m=0.4, obs_max_m=2.0,
             dens_num=1, dens_den=2, fit_n=fit, neg_thresh_m=0.5, neg_search_m=search)
    lut, data = _field(nx, ny, nz, rng, fill, wild)
    origin = np.array([-nx // 2, 3, 0], np.int32)
    m, o = gvom.VoxelMap(p), oracle.OracleMap(p)
    st = gvom.map_import_voxels(m.h, torch.from_numpy(lut).cuda(), torch.from_numpy(data).cuda(), origin)
    assert st == 0 and o.import_voxels(lut, data, origin) == oracle.OK
    ref = o.export_2d()
    o.close()
    for tile in (32, 16):
        if tile == 16 and nx * ny > 400000:
            continue
        assert gvom.map_set_tuning(m.h, surface_tile=tile) == 0
        out = m.export_2d()
        torch.cuda.synchronize()
        g = host_2d(out)
        if wild:  # 64-bit sums of squares may wrap: the plane fits say nothing
            assert np.array_equal(g["flags"], ref["flags"])
        else:
            compare_2d_arrays(g, ref, res)
    m.close()
