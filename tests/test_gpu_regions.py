"""The kernels that take a map region by region (import, table, density and
feature exports, thinning, reset) against the oracle, on windows whose columns,
levels and scroll offsets do not fill the regions (needs an MI355X).  Everything
compared here is exact: integers, and floats by their bits (slope and roughness
features excepted, which follow the plain maps' tolerance and are not compared)."""
import numpy as np
import pytest
import torch

from oracle import sgt as osgt

pytestmark = pytest.mark.gpu


def _state(nx, ny, nz, seed, fill):
    """A random table and data array: occupied, passed and unseen voxels."""
    rng = np.random.default_rng(seed)
    V = nx * ny * nz
    occ = rng.uniform(size=V) < fill
    lut = np.where(rng.uniform(size=V) < 0.4, -1 - rng.integers(1, 1000, V), -1).astype(np.int32)
    lut[occ] = np.arange(occ.sum())
    data = np.stack([rng.integers(1, 50, occ.sum()), rng.integers(0, 90, occ.sum()),
                     rng.integers(-2 ** 20, 2 ** 20, occ.sum())], 1).astype(np.int32)
    return lut, data


@pytest.mark.parametrize("nx,ny,nz,origin", [
    (2, 2, 1, (0, 0, 0)),             # one voxel per column, one partial brick
    (6, 10, 3, (-3, 5, -1)),
    (18, 34, 41, (7, -11, 13)),       # odd levels: no 16-byte table words
    (64, 48, 64, (5, 2, -31)),
    (66, 94, 96, (-35, 17, 40)),      # two occupancy words per column
    (30, 130, 128, (1, 1, 127)),      # the most levels
    (514, 530, 4, (3, -9, 2)),        # 67 super groups of ranks
    (1026, 1030, 2, (-513, 0, 1)),    # 258 of them: scanned first
])
def test_region_kernels_match_oracle(nx, ny, nz, origin):
    import oracle
    from paper_2109_13176_amd import gvom
    p = dict(nx=nx, ny=ny, nz=nz, res_m=0.25, sensor_z_voxel=nz // 2, obs_min_m=0.3, obs_max_m=2.0,
             dens_num=1, dens_den=2, fit_n=5, neg_thresh_m=0.5, neg_search_m=2.0)
    m, o = gvom.VoxelMap(p), oracle.OracleMap(p)
    origin = np.array(origin, np.int32)
    V = nx * ny * nz
    sensor = np.array([0.3, -0.2, 1.1], np.float32)
    # each state over the one before it (other occupied voxels, other offsets)
    for k, fill in enumerate((0.1, 0.0, 0.02, 0.6)):
        org = origin + np.array([k, -2 * k, 3 * k], np.int32)
        lut, data = _state(nx, ny, nz, 10 * k + nz, fill)
        off = k & 1  # a table that is not 16-byte aligned
        lt = torch.zeros(V + 4, dtype=torch.int32, device="cuda")[off:off + V]
        lt.copy_(torch.from_numpy(lut))
        dt = torch.from_numpy(data).cuda() if len(data) else None
        assert gvom.map_import_voxels(m.h, lt, dt, org) == 0
        assert o.import_voxels(lut, data, org) == oracle.OK
        out = torch.zeros(V + 4, dtype=torch.int32, device="cuda")[off:off + V]
        back = torch.zeros((len(data) + 1, 3), dtype=torch.int32, device="cuda")
        st, n, org_g = gvom.map_export_voxels(m.h, out, back)
        assert st == 0 and n == len(data) and np.array_equal(org_g, org)
        assert np.array_equal(out.cpu().numpy(), lut)
        assert np.array_equal(back.cpu().numpy()[:n], data)
        den = m.export_density().cpu().numpy()
        assert np.array_equal(den.view(np.uint32), o.export_density().view(np.uint32).reshape(-1))
        mask = (np.random.default_rng(k).uniform(size=(nx, ny)) < 0.5).astype(np.uint8)
        thin = torch.from_numpy(mask).cuda()
        for step in range(2):  # features before and after the columns go
            plain = m.export_2d()
            f = gvom.sgt_features(m, plain, sensor, thin if step else None).cpu().numpy()
            of = osgt.features(o, o.export_2d(), sensor, mask if step else np.zeros_like(mask))
            exact = [i for i in range(16) if i not in (10, 11)]
            assert np.array_equal(f[..., exact].view(np.uint32), of[..., exact].view(np.uint32))
            if step == 0:
                assert gvom.sgt_thin(m, thin) == 0
                osgt.thin(o, mask)
        st, lut_o, data_o, n_o, _ = o.export_voxels()
        st, n, _ = gvom.map_export_voxels(m.h, out, back)
        assert n == n_o and np.array_equal(out.cpu().numpy(), lut_o.reshape(-1))
        assert np.array_equal(back.cpu().numpy()[:n], np.asarray(data_o).reshape(-1, 3)[:n])
    assert gvom.map_reset(m.h) == 0
    st, n, _ = gvom.map_export_voxels(m.h, out, back)
    assert st == 0 and n == 0 and bool((out == -1).all())
    assert bool(torch.isnan(m.export_density()).all())
    m.close()
    o.close()


@pytest.mark.parametrize("nx,ny,nz,origin", [(30, 22, 16, (3, -9, 5)), (22, 30, 17, (-8, 5, 9))])
def test_region_kernels_around_sixteen_levels(nx, ny, nz, origin):
    """The line between one and four waves per region of the thinning and the reset."""
    test_region_kernels_match_oracle(nx, ny, nz, origin)


def test_import_of_invalid_content_empties_the_map():
    from paper_2109_13176_amd import gvom
    nx, ny, nz = 34, 18, 9
    p = dict(nx=nx, ny=ny, nz=nz, res_m=0.25, sensor_z_voxel=4, obs_min_m=0.3, obs_max_m=2.0,
             dens_num=1, dens_den=2, fit_n=5, neg_thresh_m=0.5, neg_search_m=2.0)
    m = gvom.VoxelMap(p)
    org = np.zeros(3, np.int32)
    good, data = _state(nx, ny, nz, 3, 0.2)
    out = torch.zeros(nx * ny * nz, dtype=torch.int32, device="cuda")
    for kind in ("index", "hits", "min"):
        lut, d = good.copy(), data.copy()
        if kind == "index":
            lut[np.argmax(lut)] = len(d)
        elif kind == "hits":
            d[7, 0] = 0
        else:
            lut[5] = -2 ** 31
        assert gvom.map_import_voxels(m.h, torch.from_numpy(good).cuda(), torch.from_numpy(data).cuda(), org) == 0
        st = gvom.map_import_voxels(m.h, torch.from_numpy(lut).cuda(), torch.from_numpy(d).cuda(), org)
        assert st == gvom.MAP_E_INVALID, kind
        st, n, _ = gvom.map_export_voxels(m.h, out, None)
        assert n == 0 and bool((out == -1).all()), kind
    m.close()


@pytest.mark.parametrize("H,W", [(1, 1), (16, 32), (17, 33), (5, 130), (100, 7)])
def test_fill_at_tile_edges(H, W):
    from paper_2109_13176_amd import gvom
    rng = np.random.default_rng(H + W)
    ph = rng.normal(0, 2, (H, W)).astype(np.float32)
    ph[rng.uniform(size=(H, W)) < 0.7] = np.nan
    pr = rng.uniform(0, 0.1, (H, W)).astype(np.float32)
    pred = np.stack([np.where(np.isnan(ph), 0, ph) + rng.normal(0, 0.05, (H, W)),
                     rng.normal(0, 0.05, (H, W))], 2).astype(np.float32)
    plain = {"height": torch.from_numpy(ph).cuda(), "rough": torch.from_numpy(pr).cuda()}
    for k in ("slope", "density"):
        plain[k] = torch.zeros((H, W), dtype=torch.float32, device="cuda")
    plain["flags"] = torch.zeros((H, W), dtype=torch.uint8, device="cuda")
    gh, gr = gvom.sgt_fill(torch.from_numpy(pred).cuda(), plain, 0.04)
    oh, orr = osgt.fill(pred, ph, pr, 0.04)
    assert np.array_equal(gh.cpu().numpy().view(np.uint32), oh.view(np.uint32))
    assert np.array_equal(gr.cpu().numpy().view(np.uint32), orr.view(np.uint32))


@pytest.mark.parametrize("nx,ny,nz", [(6, 10, 3), (18, 34, 41), (64, 48, 64), (66, 94, 96)])
def test_scrolled_window_keeps_and_clears(nx, ny, nz):
    """The window moved over a random map by every kind of step (slabs that wrap
    in storage, that cut bricks, along one axis, all axes, past the window), with
    and without points in the same call."""
    import oracle
    from paper_2109_13176_amd import gvom
    p = dict(nx=nx, ny=ny, nz=nz, res_m=0.5, sensor_z_voxel=nz // 2, obs_min_m=0.5, obs_max_m=2.0,
             dens_num=1, dens_den=2, fit_n=5, neg_thresh_m=0.5, neg_search_m=2.0)
    rng = np.random.default_rng(nz)
    m, o = gvom.VoxelMap(p), oracle.OracleMap(p)
    V = nx * ny * nz
    out = torch.zeros(V, dtype=torch.int32, device="cuda")
    steps = [(0, 0, 0), (1, 0, 0), (0, -3, 0), (0, 0, 1), (-2, 1, 0), (nx // 2, -1, -nz // 2),
             (3, ny - 1, 1), (-nx + 1, 2, -1), (nx + 5, 0, 0), (0, 0, nz - 1), (5, 4, -2)]
    vox = np.array([0, 0, 0])
    for k, d in enumerate(steps):
        if k % 5 == 0:
            lut, data = _state(nx, ny, nz, k + nx, 0.3)
            org = vox - np.array([nx // 2, ny // 2, nz // 2])
            org = org.astype(np.int32)
            assert gvom.map_import_voxels(m.h, torch.from_numpy(lut).cuda(),
                                          torch.from_numpy(data).cuda(), org) == 0
            assert o.import_voxels(lut, data, org) == oracle.OK
        vox = vox + np.array(d)
        pose = np.eye(3, 4, dtype=np.float32)
        pose[:, 3] = (vox + 0.5) * 0.5
        pts = rng.uniform(-nx / 5, nx / 5, (0 if k & 1 else 700, 3)).astype(np.float32)
        x = torch.from_numpy(pts).cuda() if len(pts) else None
        assert gvom.map_insert_scan(m.h, x, pose.reshape(12), gvom.MAP_RECENTER) == 0
        assert o.insert_scan(pts, pose.reshape(12), oracle.RECENTER) == oracle.OK
        n_o = o.export_voxels()
        back = torch.zeros((n_o[3] + 1, 3), dtype=torch.int32, device="cuda")
        st, n, org_g = gvom.map_export_voxels(m.h, out, back)
        assert st == 0 and n == n_o[3] and np.array_equal(org_g, n_o[4]), k
        assert np.array_equal(out.cpu().numpy(), n_o[1].reshape(-1)), k
        assert np.array_equal(back.cpu().numpy()[:n], np.asarray(n_o[2]).reshape(-1, 3)[:n]), k
        assert m.stats()["n_cleared"] == o.stats()["n_cleared"], k
    m.close()
    o.close()


def test_import_time_does_not_follow_the_heights():
    """A table given another origin in z, so that every lowest return lies outside its
    voxel, is imported about as fast as one with all of them inside (a factor of 4
    leaves room for noise; one global update per such voxel took 12)."""
    import time
    from paper_2109_13176_amd import gvom
    nx, ny, nz = 512, 512, 64
    p = dict(nx=nx, ny=ny, nz=nz, res_m=0.2, sensor_z_voxel=32, obs_min_m=0.4, obs_max_m=2.0,
             dens_num=1, dens_den=2, fit_n=5, neg_thresh_m=0.5, neg_search_m=5.0)
    rng = np.random.default_rng(0)
    lut = np.full(nx * ny * nz, -1, np.int32)
    occ = np.flatnonzero(rng.uniform(size=len(lut)) < 0.01)
    lut[occ] = np.arange(len(occ))
    data = np.ones((len(occ), 3), np.int32)
    data[:, 2] = (occ % nz) << 16
    lt, dt = torch.from_numpy(lut).cuda(), torch.from_numpy(data).cuda()
    m = gvom.VoxelMap(p)
    took = []
    for oz in (0, 5):
        org = np.array([0, 0, oz], np.int32)
        t = []
        for _ in range(20):
            t0 = time.perf_counter()
            assert gvom.map_import_voxels(m.h, lt, dt, org) == 0
            t.append(time.perf_counter() - t0)
        took.append(sorted(t)[len(t) // 2])
    m.close()
    print(f"import: heights inside {took[0] * 1e6:.0f} us, outside {took[1] * 1e6:.0f} us", flush=True)
    assert took[1] < 4 * took[0]
