"""Launch tuning: a value the caller sets is what runs, and where the library
chooses (a map whose tuning was never set) results are the oracle's on both sides
of its lines (needs an MI355X).  Integers and height bits are compared exactly, by
the comparison rules of the other parity tests."""
import numpy as np
import pytest
import torch

from conftest import params
from parity_util import Pair, compare_2d, compare_all, compare_2d_arrays, host_2d

pytestmark = pytest.mark.gpu

POSE = np.concatenate([np.eye(3, dtype=np.float32),
                       np.array([[0.1], [0.2], [0.3]], np.float32)], 1).reshape(12)


def _cloud(n, radius, seed):
    rng = np.random.default_rng(seed)
    return rng.uniform(-radius, radius, (n, 3)).astype(np.float32)


def _insert_bytes(dims, n, seg_len):
    """Bytes of the work buffers of a map's first insert: a 16-byte record per ray of
    every block of 512, 8 bytes for every wave item a block's 8 waves can have (one per
    segment of the window's longest axis), 32 bytes of counters per block."""
    blocks = (n + 511) // 512
    return blocks * (512 * 16 + 8 * ((max(dims) - 1) // seg_len + 1) * 8 + 32)


# a map's own choice: 4 up to 2^24 points x longer side (1024 at most), 5 up to sides of 512
# and 196,608 points, then 8
@pytest.mark.parametrize("dims,n,set_len,runs", [
    ((64, 48, 16), 1500, 8, 8), ((512, 12, 16), 131072, 8, 8), ((512, 12, 16), 131072, 5, 5),
    ((64, 48, 16), 200000, 3, 3),
    ((64, 48, 16), 1500, 0, 4), ((64, 48, 16), 262144, 0, 4), ((64, 48, 16), 262145, 0, 8),
    ((512, 12, 16), 32768, 0, 4), ((512, 12, 16), 32769, 0, 5), ((12, 512, 16), 32769, 0, 5),
    ((512, 12, 16), 196608, 0, 5), ((512, 12, 16), 196609, 0, 8),
    ((514, 12, 16), 32640, 0, 4), ((514, 12, 16), 32641, 0, 8),
    ((4096, 6, 8), 16384, 0, 4), ((4096, 6, 8), 16385, 0, 8),
])
def test_segment_length_that_runs(dims, n, set_len, runs):
    from paper_2109_13176_amd import gvom
    pair = Pair(params(*dims, 0.5), set_len)
    try:
        used = gvom.lib().map_device_memory_in_use()
        assert pair.insert(_cloud(n, 20.0, n), POSE) == 0
        assert gvom.lib().map_device_memory_in_use() - used == _insert_bytes(dims, n, runs)
        compare_all(pair)
        assert gvom.map_get_tuning(pair.g.h)[1]["seg_len"] == (set_len or 8)
    finally:
        pair.close()


def test_no_memory_for_shorter_segments():
    """Under a memory limit that admits the work buffers of segments of 8 but not of
    5, the length of a scan of 131,072 points: 8 runs, and goes on running without
    another try while its buffers hold; a larger scan grows them again."""
    from paper_2109_13176_amd import gvom
    L = gvom.lib()
    dims, n = (512, 12, 16), 131072
    pair = Pair(params(*dims, 0.5))
    try:
        pts = _cloud(n, 20.0, 1)
        used = L.map_device_memory_in_use()
        assert L.map_set_device_memory_limit(used + _insert_bytes(dims, n, 8) - 1024) == 0
        x = torch.as_tensor(pts, device="cuda")
        assert gvom.map_insert_scan(pair.g.h, x, POSE, 0) == gvom.MAP_E_OOM
        assert pair.g.export_voxels()[2] == 0
        assert L.map_set_device_memory_limit(used + _insert_bytes(dims, n, 8) + 1024) == 0
        for k in range(3):
            assert pair.insert(_cloud(n, 20.0, k), POSE) == 0
            assert L.map_device_memory_in_use() - used == _insert_bytes(dims, n, 8)
            if k == 1:
                assert L.map_set_device_memory_limit(0) == 0
        compare_all(pair)
        for m in (1000, 150000, n):
            assert pair.insert(_cloud(m, 20.0, m), POSE) == 0
        assert L.map_device_memory_in_use() - used > _insert_bytes(dims, 150000, 5)
        compare_all(pair)
    finally:
        L.map_set_device_memory_limit(0)
        pair.close()


# windows where the library takes 16, 32 and 64 pixels by itself; 31 rings and more
@pytest.mark.parametrize("nx,ny,res", [(62, 98, 0.1), (258, 250, 0.2), (642, 514, 0.1),
                                       (1030, 1026, 0.2)])
def test_surface_tiles_set_and_chosen(nx, ny, res):
    from paper_2109_13176_amd import gvom
    pair = Pair(params(nx, ny, 16, res, szv=8))
    try:
        pts = _cloud(20000, 0.4 * nx * res, nx)
        pts[:, 2] *= 0.02
        assert pair.insert(pts, POSE, 1) == 0
        _, ref = compare_2d(pair)
        for tile in (32, 16):
            assert gvom.map_set_tuning(pair.g.h, surface_tile=tile) == 0
            out = pair.g.export_2d()
            torch.cuda.synchronize()
            compare_2d_arrays(host_2d(out), ref, res)
            assert gvom.map_get_tuning(pair.g.h)[1]["surface_tile"] == tile
    finally:
        pair.close()


def test_batch_follows_tuning_set_between_steps():
    """A batch whose maps' surface tile is set after its first step (its recorded
    launches then no longer fit): every step equals the single-map calls."""
    from paper_2109_13176_amd import gvom
    ps = [params(64, 48, 16, 0.5), params(98, 62, 16, 0.1)]
    maps, ref = [gvom.VoxelMap(p) for p in ps], [gvom.VoxelMap(p) for p in ps]
    batch = gvom.MapBatch(maps)
    try:
        for k, tile in enumerate((0, 32, 16, 32)):
            if tile:
                for m in maps:
                    assert gvom.map_set_tuning(m.h, surface_tile=tile) == 0
            xyz = [torch.as_tensor(_cloud(3000, 6.0, 10 * k + i), device="cuda") for i in range(2)]
            for x in xyz:
                x[:, 2] *= 0.05
            batch.step(xyz, [POSE, POSE], [1, 1], [True, False])
            torch.cuda.synchronize()
            for i, m in enumerate(ref):
                assert gvom.map_insert_scan(m.h, xyz[i], POSE, 1) == 0
                want = m.export_2d()
                torch.cuda.synchronize()
                for key in want:
                    assert torch.equal(maps[i].out2d[key].view(torch.uint8), want[key].view(torch.uint8)), \
                        (k, i, key)
    finally:
        batch.close()
        for m in maps + ref:
            m.close()
