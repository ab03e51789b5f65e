"""The cubic blob's adjoint at the edges of its split (four lanes a point, points
of equally many pixels together), against the float64 oracle: windows of one to
three columns or rows, of up to 16, 20, 28 and more pixels, whole images
narrower than four pixels, points in view and out of it side by side, a last
wave of one point."""
import numpy as np
import pytest

import synth
from oracle import cubic as ocubic
from oracle import splat as osplat
from paper_0811_2055_amd import lib

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (2, 9), (3, 40), (5, 3), (70, 33)])
@pytest.mark.parametrize("h,n", [(0.6, 1), (1.0, 63), (1.7, 64), (2.2, 65), (2.6, 257), (5.0, 500), (16.0, 129)])
def test_windows(W, H, h, n):
    import torch
    s = synth.uniform(n, n)
    # a third of the points out of view or at its border
    s.x[::3] = np.float32(-0.2) + np.float32(1.4) * s.x[::3]
    cam, ocam = lib.Camera.ortho(W, H), osplat.Camera(0, W, H)
    g = np.random.default_rng(W * H).standard_normal((H, W)).astype(np.float32)
    got = lib.splat_backward(*to_dev(s), torch.from_numpy(g).cuda(), cam, blob=lib.Blob.cubic(h_px=h))
    rm, rp = ocubic.render_backward(ocam, s.x, s.y, s.z, s.m, g.astype(np.float64), h_px=h)
    bm, bp = ocubic.render_backward(ocam, s.x, s.y, s.z, s.m, None, h_px=h, bound_weights=np.abs(g.astype(np.float64)))
    # float64 sums of float32 offsets, rounded once: 1e-6 of the absolute terms
    for k, want, bound in ((0, rm, bm), (1, rp[:, 0], bp[:, 0]), (2, rp[:, 1], bp[:, 1]), (3, rp[:, 2], bp[:, 2])):
        v = got[k].cpu().numpy().astype(np.float64)
        bad = np.nonzero(np.abs(v - want) > 1e-6 * bound + 1e-30)[0]
        assert bad.size == 0, (k, bad[:5], v[bad[:5]], want[bad[:5]], bound[bad[:5]])
