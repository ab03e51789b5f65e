"""Rounding and range of the Gaussian blob's pixel values: isolated points (one
per 16 x 16 pixels, so that no pixel sums two), each pixel against the float64
oracle within the rounding of one float32 exponential per axis, for masses up
to the largest that leave every pixel finite."""
import math

import numpy as np
import pytest

from oracle import splat as osplat
from paper_0811_2055_amd import lib

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("sigma,radius", [(0.3, 3.0), (0.5, 3.0), (0.5, 6.0), (0.663, 6.0), (0.7, 3.0), (1.0, 0.9), (1.0, 3.0), (1.0, 3.97),
                                          (1.3, 3.0), (2.0, 1.95), (4.0, 0.97), (8.0, 0.49), (2.0, 3.0)])
@pytest.mark.parametrize("mass", [1.0, 3e36, 1e38])
def test_isolated_points(sigma, radius, mass):
    import torch
    rng = np.random.default_rng(4)
    W, H = 1024, 512
    gx, gy = np.meshgrid(np.arange(W // 16), np.arange(H // 16))
    n = gx.size
    x = ((16 * gx.ravel() + 7 + rng.random(n)) / W).astype(np.float32)
    y = ((16 * gy.ravel() + 7 + rng.random(n)) / H).astype(np.float32)
    z = rng.random(n).astype(np.float32)
    # the largest pixel stays below 2e38
    m = (mass * rng.uniform(0.5, 1.0, n) * min(1.0, 2 * math.pi * sigma * sigma)).astype(np.float32)
    d = [torch.from_numpy(a).cuda() for a in (x, y, z, m)]
    got = lib.splat(*d, lib.Camera.ortho(W, H), sigma, radius).cpu().numpy().astype(np.float64)
    want = osplat.render(osplat.Camera(0, W, H), x, y, z, m, sigma, radius)
    assert np.isfinite(got).all()
    assert np.array_equal(got > 0, want > 0)
    # an axis: the square, the factor and its float32 constant (three roundings
    # of an argument of at most o^2 / 2 sigma^2), an exponential (within an ulp);
    # the product with the mass, that of the axes and the image's own rounding
    arg = (radius * sigma) ** 2 / (2 * sigma * sigma)
    tol = 2 * (3 * U * arg + 2 * U) + 3 * U
    on = want > 1e-30
    rel = np.abs(got[on] - want[on]) / want[on]
    assert float(rel.max()) <= tol, (float(rel.max()), tol)


@pytest.mark.parametrize("sigma", [0.5, 0.7, 0.9, 1.0, 1.1, 1.3, 2.0])
def test_mass_of_a_dense_image(sigma):
    """Roundings that are the same for every point would not average out: the
    image's sum is the oracle's within a third of a rounding unit."""
    import torch
    rng = np.random.default_rng(9)
    W, H, n = 128, 96, 200000
    x, y, z = (rng.uniform(0.1, 0.9, n).astype(np.float32) for _ in range(3))
    m = rng.uniform(0.2, 1.0, n).astype(np.float32)
    d = [torch.from_numpy(a).cuda() for a in (x, y, z, m)]
    got = lib.splat(*d, lib.Camera.ortho(W, H), sigma, 3.0).cpu().numpy().astype(np.float64).sum()
    want = osplat.render(osplat.Camera(0, W, H), x, y, z, m, sigma, 3.0).sum()
    assert abs(got / want - 1.0) <= U / 3, got / want - 1.0
