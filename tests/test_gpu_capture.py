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
