"""Gradient of the gap-fill network on images at the edges of its kernels' tiles (8 and 4
rows, 16 rows a block, 64 columns), against the oracle (needs an MI355X).  The bound is
the one of the other gradient test: fp32 sums against fp64, 1e-3 of a layer's largest
entry; labels keep 0.05 from the oracle's output so that every sign is the same."""
import numpy as np
import pytest
import torch

from oracle import sgt as osgt

pytestmark = pytest.mark.gpu

CIN, COUT = (16, 32, 32, 32, 32), (32, 32, 32, 32, 2)


@pytest.mark.parametrize("H,W,offset", [(1, 1, 0), (8, 64, 0), (9, 65, 1), (17, 63, 0), (33, 129, 1)])
def test_gradient_at_tile_edges(H, W, offset):
    from paper_2109_13176_amd import gvom
    rng = np.random.default_rng(H * 1000 + W)
    p = np.concatenate([np.concatenate([rng.normal(0, np.sqrt(2.0 / (9 * ci)), co * ci * 9),
                                        rng.normal(0, 0.05, co)]) for ci, co in zip(CIN, COUT)])
    p = p.astype(np.float32)
    net = gvom.Surrogate(H, W, seed=1)
    try:
        net.set_params(p)
        x = rng.normal(size=(H, W, 16)).astype(np.float32)
        out = osgt.forward(x, p, True)
        lab = out + rng.choice([-1, 1], size=out.shape) * rng.uniform(0.05, 0.5, out.shape)
        lab = lab.astype(np.float32)
        if lab.size > 2:
            lab[rng.uniform(size=lab.shape) < 0.3] = np.nan
        # labels that are 4-byte aligned only
        lt = torch.zeros(lab.size + 2, device="cuda")[offset:offset + lab.size].view(H, W, 2)
        lt.copy_(torch.from_numpy(lab))
        loss, g = net.loss_grad(torch.from_numpy(x).cuda(), lt, True)
        ref_loss, ref_g = osgt.loss_grad(x, p, lab, True)
        assert loss == pytest.approx(ref_loss, rel=1e-4)
        o = 0
        for ci, co in zip(CIN, COUT):
            n = co * ci * 9 + co
            a, b = g[o:o + n], ref_g[o:o + n]
            o += n
            assert np.abs(a - b).max() <= 1e-3 * np.abs(b).max()
    finally:
        net.close()
