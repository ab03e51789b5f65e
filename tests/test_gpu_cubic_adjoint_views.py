"""The cubic blob's adjoint in perspective views from inside the points: some
behind the near plane, some out of view, world radii below, between and above
the clamps at 1 and 16 pixels, with and without a fixed pixel radius beside
them.  All four gradients against the float64 oracle, and 0 where culled."""
import numpy as np
import pytest

import synth
from oracle import cubic as ocubic
from oracle import splat as osplat
from paper_0811_2055_amd import lib

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_px,h_world", [(0.0, 0.001), (0.0, 0.01), (0.0, 0.2), (2.2, 0.01), (2.2, 0.0), (16.0, 0.0),
                                          (0.3, 0.0), (1.25, 0.0), (1.2501, 0.0)])
@pytest.mark.parametrize("n", [1, 65, 2000])
def test_view_from_inside(n, h_px, h_world):
    import torch
    s = synth.small_clustered(n, 31 + n)
    W, H = 96, 80
    cam = lib.Camera.look_at((0.5, 0.48, 0.5), (0.55, 0.5, 0.9), W, H, fov_deg=70.0)
    ocam = osplat.Camera(1, W, H, cam.pos, cam.right, cam.up, cam.fwd, cam.F, cam.near)
    g = np.random.default_rng(n).standard_normal((H, W)).astype(np.float32)
    got = lib.splat_backward(*to_dev(s), torch.from_numpy(g).cuda(), cam,
                             blob=lib.Blob.cubic(h_px=h_px, h_world=h_world))
    kw = dict(h_px=h_px, h_world=h_world)
    rm, rp = ocubic.render_backward(ocam, s.x, s.y, s.z, s.m, g.astype(np.float64), **kw)
    bm, bp = ocubic.render_backward(ocam, s.x, s.y, s.z, s.m, None, bound_weights=np.abs(g.astype(np.float64)), **kw)
    keep = osplat.project(ocam, s.x, s.y, s.z)[2]
    assert n < 2000 or 100 < np.count_nonzero(keep) < n - 100
    # float64 sums of float32 offsets, rounded once: 1e-6 of the absolute terms
    for k, want, bound in ((0, rm, bm), (1, rp[:, 0], bp[:, 0]), (2, rp[:, 1], bp[:, 1]), (3, rp[:, 2], bp[:, 2])):
        v = got[k].cpu().numpy().astype(np.float64)
        assert np.all(v[~keep] == 0.0), k
        bad = np.nonzero(~(np.abs(v - want) <= 1e-6 * bound + 1e-30))[0]
        assert bad.size == 0, (k, bad[:5], v[bad[:5]], want[bad[:5]], bound[bad[:5]])
