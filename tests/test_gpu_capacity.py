"""An image is a function of the points drawn, not of the sizes that its
workspace was planned for: one cut drawn under capacities up to 2^26 points, the
highlighted points under several bounds, the allocation-free render against the
planned one up to its limit, all bit for bit; a workspace planned for more points
draws fewer."""
import ctypes as C

import numpy as np
import pytest

import synth
from gpu_util import image_rel_err, to_dev
from oracle import splat as osplat
from paper_0811_2055_amd import lib

pytestmark = pytest.mark.gpu


def bits(t):
    import torch
    return t.view(torch.int32)


@pytest.mark.parametrize("blob", [None, "cubic"])
@pytest.mark.parametrize("N", [60_000, 900_000])
def test_one_cut_under_several_capacities(N, blob):
    import torch
    s = synth.small_clustered(N, 12)
    tree = lib.build(*to_dev(s), lib.BuildParams(n=3000, max_depth=6, seed=2))
    b = lib.Blob.cubic(h_px=2.5) if blob else None
    cam = lib.Camera.ortho(1024, 1024)
    ids, nsel = lib.select_nodes(tree, cam, 0.5, 3000)
    first = None
    for cap in (N, (1 << 19) + 1 if N < 1 << 19 else N + 1, 1_000_000, 1_100_000, 1 << 21, 1 << 23, 1 << 25, (1 << 25) + 1,
                1 << 26):
        img = lib.splat_lod(tree, ids, nsel, cap, cam, blob=b)
        first = img if first is None else first
        assert torch.equal(bits(img), bits(first)), cap
    assert float(first.max()) > 0
    assert int(lib._to_numpy(tree.counts)[2]) == 0
    flags = lib.highlight_flags(tree, lib.highlight_bits(np.arange(0, N, 2), N), N)
    first = None
    for cap in (N, 1_000_000, 1 << 20, 1 << 22, 1 << 25):
        img, hl = lib.splat_lod_highlight(tree, ids, nsel, max(cap, N), cam, flags, cap, blob=b)
        first = hl if first is None else first
        assert torch.equal(bits(hl), bits(first)), cap
    assert float(first.max()) > 0


@pytest.mark.parametrize("N,blob", [(900_000, None), (1_000_000, None), (1_050_000, None), (1_080_000, None), (500_000, 2.5),
                                    (800_000, 2.5), (60_000, 16.0), (150_000, 16.0)])
def test_allocation_free_up_to_its_limit(N, blob):
    import torch
    s = synth.uniform(N, 3)
    dev = to_dev(s)
    b = lib.Blob.cubic(h_px=blob) if blob else None
    cam = lib.Camera.ortho(1024, 1024)
    want = lib.splat(*dev, cam, blob=b)
    assert torch.equal(bits(lib.splat_noalloc(*dev, cam, blob=b)), bits(want))
    both, _ = lib.splat_aux(*dev, torch.ones_like(dev[0]), cam, blob=b)
    assert torch.equal(bits(both), bits(want))
    if blob is None:
        err, zeros_ok = image_rel_err(want.cpu().numpy(), osplat.render(osplat.Camera(0, 1024, 1024), s.x, s.y, s.z, s.m))
        assert zeros_ok and err <= 1e-5, err


@pytest.mark.parametrize("planned,drawn,blob", [(524_920, 514_627, None), (176_619, 173_155, 16.0)])
def test_a_planned_workspace_draws_fewer_points(planned, drawn, blob):
    import torch
    s = synth.uniform(drawn, 5)
    dev = to_dev(s)
    att = torch.ones_like(dev[0])
    b = lib.Blob.cubic(h_px=blob) if blob else None
    cam = lib.Camera.ortho(1024, 1024)
    ws = torch.empty(lib.splat_workspace_bytes(planned, cam, blob=b), dtype=torch.uint8, device="cuda")
    img, aimg = (torch.empty(1024, 1024, device="cuda") for _ in range(2))
    camc, sp = cam.c(), lib._sp(1.0, 3.0, b)
    p = [lib._ptr(t) for t in (*dev, att)]
    assert lib.load().splat_render_aux(*p, drawn, C.byref(camc), C.byref(sp), lib._ptr(ws), ws.numel(), lib._ptr(img),
                                       lib._ptr(aimg), lib._stream()) == lib.LOD_OK
    assert torch.equal(bits(img), bits(lib.splat(*dev, cam, blob=b)))
    assert torch.equal(bits(img), bits(aimg))
