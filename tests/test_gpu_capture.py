"""Exports and inserts captured into graphs, replayed between the program's own calls,
against the oracle (needs an MI355X): a table export has the ranks of the map as it is
when it runs.  Tables, data arrays and heights are compared exactly."""
import numpy as np
import pytest
import torch

import oracle
from conftest import params
from parity_util import compare_2d_arrays, compare_voxel_arrays, host_2d

pytestmark = pytest.mark.gpu

POSE = np.concatenate([np.eye(3, dtype=np.float32),
                       np.array([[0.1], [0.2], [0.3]], np.float32)], 1).reshape(12)
SMALL = (66, 48, 20)
LARGE = (1026, 1030, 2)  # 258 super groups of ranks: their sums are scanned in place


class Rig:
    """A map on a stream of its own, the oracle's map and graphs of the map's calls."""

    def __init__(self, dims):
        from paper_2109_13176_amd import gvom
        self.p = params(*dims, 0.5)
        self.s = torch.cuda.Stream()
        self.m, self.o = gvom.VoxelMap(self.p, stream=self.s), oracle.OracleMap(self.p)
        self.rng = np.random.default_rng(dims[0])
        self.m.export_voxels_async()  # (its output tensors exist before a capture)
        torch.cuda.synchronize()

    def cloud(self, n=3000):
        r = 0.5 * np.array([self.p["nx"], self.p["ny"], self.p["nz"]]) / 2
        return self.rng.uniform(-r, r, (n, 3)).astype(np.float32)

    def insert(self, pts):
        from paper_2109_13176_amd import gvom
        x = torch.as_tensor(pts, device="cuda")
        torch.cuda.synchronize()
        assert gvom.map_insert_scan(self.m.h, x, POSE, 0) == 0
        self.seen(pts)
        torch.cuda.synchronize()

    def seen(self, pts):
        assert self.o.insert_scan(pts, POSE, 0) == oracle.OK

    def capture(self, *calls):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=self.s, capture_error_mode="thread_local"):
            for c in calls:
                c()
        return g

    def replay(self, g):
        with torch.cuda.stream(self.s):
            g.replay()
        torch.cuda.synchronize()

    def check_table(self):
        torch.cuda.synchronize()
        st, lut, data, n, origin = self.o.export_voxels()
        assert st == oracle.OK
        m = self.m
        compare_voxel_arrays((m.lut, m.data, int(m.n_occ.item()), m.origin()), lut, data, n, origin)
        m.lut.fill_(-7)
        m.n_occ.fill_(-7)
        torch.cuda.synchronize()

    def close(self):
        self.m.close()
        self.o.close()


@pytest.mark.parametrize("dims", [SMALL, LARGE])
def test_captured_table_export_after_an_eager_2d_export(dims):
    r = Rig(dims)
    try:
        r.insert(r.cloud())
        r.m.export_2d()
        g = r.capture(r.m.export_voxels_async)
        for k in range(3):
            r.insert(r.cloud())
            if k == 1:
                r.m.export_2d()
            r.replay(g)
            r.check_table()
    finally:
        r.close()


@pytest.mark.parametrize("dims", [SMALL, LARGE])
def test_replayed_insert_between_the_exports(dims):
    from paper_2109_13176_amd import gvom
    r = Rig(dims)
    try:
        pts = r.cloud()
        x = torch.as_tensor(pts, device="cuda")

        def static():
            assert gvom.map_insert_scan_static(r.m.h, x, POSE, 0) == 0
        r.insert(r.cloud())
        g = r.capture(static)
        for _ in range(2):
            r.m.export_2d()
            torch.cuda.synchronize()
            r.replay(g)
            r.seen(pts)
            r.m.export_voxels_async()
            r.check_table()
            r.insert(r.cloud())
    finally:
        r.close()


@pytest.mark.parametrize("dims", [SMALL, LARGE])
def test_both_exports_in_one_graph_and_apart(dims):
    """The pair captured together uses the ranks of its own 2D export; captured apart,
    and eager calls between the replays, every table counts for itself."""
    r = Rig(dims)
    try:
        r.insert(r.cloud())
        both = r.capture(r.m.export_2d, r.m.export_voxels_async)
        first = r.capture(r.m.export_2d)
        second = r.capture(r.m.export_voxels_async)
        for k in range(3):
            r.insert(r.cloud())
            for g in ((both,), (first, second), (both, second))[k]:
                r.replay(g)
            r.check_table()
            r.insert(r.cloud())
            r.m.export_2d()
            torch.cuda.synchronize()
            r.replay(both)
            r.check_table()
            r.m.export_voxels_async()
            r.check_table()
            compare_2d_arrays(host_2d(r.m.out2d), r.o.export_2d(), 0.5)
    finally:
        r.close()


def test_captured_2d_export_and_imported_heights():
    """A graph of the 2D export made while every height lay in its voxel, replayed on
    imported heights of up to 2^28 (4,096 voxels; 32-bit sums of a 5 x 5 window's first
    moments, up to 30 times that, do not hold them), and back."""
    from paper_2109_13176_amd import gvom
    r = Rig(SMALL)
    nx, ny, nz = SMALL
    try:
        r.insert(r.cloud())
        g = r.capture(r.m.export_2d)
        org = np.array([-nx // 2, -ny // 2, -nz // 2], np.int32)
        for k, top in enumerate((2 ** 28, 2 ** 16, 2 ** 28, None)):
            lut = np.full((nx * ny, nz), -1, np.int32)
            known = np.flatnonzero(r.rng.uniform(size=nx * ny) < 0.7)
            z = r.rng.integers(0, nz, len(known))
            lut[known, z] = np.arange(len(known))
            data = np.ones((len(known), 3), np.int32)
            data[:, 2] = (org[2] + z << 16) + r.rng.integers(0, 65536, len(known))
            if top == 2 ** 28:
                data[:, 2] = r.rng.integers(-top, top, len(known))
            if top is None:  # refused: the map is empty afterwards
                data[3, 0] = 0
            lut = lut.reshape(-1)
            st = gvom.map_import_voxels(r.m.h, torch.from_numpy(lut).cuda(),
                                        torch.from_numpy(data).cuda(), org)
            assert st == (0 if top else gvom.MAP_E_INVALID)
            assert (r.o.import_voxels(lut, data, org) == oracle.OK) == (top is not None)
            if top is None:
                r.o.close()
                r.o = oracle.OracleMap(r.p)
            if k == 2:  # emptied and filled by scans alone
                assert gvom.map_reset(r.m.h) == 0
                r.o.close()
                r.o = oracle.OracleMap(r.p)
                r.insert(r.cloud())
            ref = r.o.export_2d()
            for _ in range(2):
                r.replay(g)
                compare_2d_arrays(host_2d(r.m.out2d), ref, 0.5)
                r.m.export_2d()
                torch.cuda.synchronize()
                compare_2d_arrays(host_2d(r.m.out2d), ref, 0.5)
    finally:
        r.close()
