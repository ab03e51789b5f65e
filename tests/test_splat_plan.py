"""Plans of the splat's workspace (no GPU): a plan for up to N points covers every
smaller number, for every blob and image size, and the allocation-free render
refuses the calls beyond its limit."""
import ctypes as C
import random

import pytest

from paper_0811_2055_amd import lib

BLOBS = {"gauss": {}, "wide": dict(sigma=4.0), "cubic": dict(blob=lib.Blob.cubic(h_px=2.5)),
         "cubic16": dict(blob=lib.Blob.cubic(h_px=16.0)), "cubic1": dict(blob=lib.Blob.cubic(h_px=1.0))}


@pytest.mark.parametrize("W,H", [(16, 16), (256, 256), (1024, 1024), (1920, 1080), (2048, 1024)])
@pytest.mark.parametrize("blob", sorted(BLOBS))
def test_a_plan_covers_fewer_points(W, H, blob):
    rng = random.Random(W + H)
    cam = lib.Camera.ortho(W, H)
    sizes = {int(2 ** rng.uniform(0, 27)) for _ in range(200)}
    for top in (17, 19, 20, 21, 22, 25, 26):
        for pairs_per_point in (1, 4, 9, 16):
            n = 2 ** top // pairs_per_point
            sizes |= {n - 1, n, n + 1, n + n // 50}
    sizes |= {514_627, 524_920, 173_155, 176_619, 459_162, 524_289}
    before = (0, 0, 0)
    for n in sorted(sizes):
        try:
            now = (lib.splat_workspace_bytes(n, cam, **BLOBS[blob]),
                   lib.splat_lod_workspace_bytes(5000, n, cam, **BLOBS[blob]),
                   lib.splat_lod_highlight_workspace_bytes(5000, 1000, n, cam, **BLOBS[blob]))
        except lib.LodError as e:
            assert e.code == lib.LOD_EUNSUPPORTED     # 32-bit pair counts
            break
        assert all(a >= b for a, b in zip(now, before)), n
        before = now


@pytest.mark.parametrize("W,H,count", [(1024, 1024, 1_300_000), (1024, 1024, 3_000_000), (256, 256, 1_400_000),
                                       (2048, 1024, 1_200_000)])
def test_noalloc_refuses_beyond_its_limit(W, H, count):
    """Refused before anything is read: any addresses do."""
    L = lib.load()
    cam, sp = lib.Camera.ortho(W, H).c(), lib._sp(1.0, 3.0, None)
    a = C.c_void_p(256)
    assert L.splat_render_noalloc(a, a, a, a, count, C.byref(cam), C.byref(sp), a, C.c_void_p()) == lib.LOD_ECAPACITY
