"""The binning of points to tiles at its edges: rounds of 64 points that lie in
one 8x8 tile window, rounds that change windows, rounds spread over the image,
blobs several tiles wide; cuts and draw lists at the edges of their blocks.
Images against the float64 oracle within 1e-5 per pixel."""
import numpy as np
import pytest

from gpu_util import image_rel_err, to_dev
from oracle import cubic as ocubic
from oracle import cut as ocut
from oracle import lod as olod
from oracle import splat as osplat
from paper_0811_2055_amd import lib
import synth

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _points(order, n, seed):
    s = synth.small_clustered(n, seed)
    if order == "morton":
        key = olod.interleave(*(olod.cell_coords(a, 10) for a in (s.x, s.y, s.z)), 10)
        o = np.argsort(key, kind="stable")
    elif order == "corners":          # every round holds points of all four corners
        o = np.arange(n)
        s.x[:] = np.where(o & 1, 0.02, 0.98) + (s.x - 0.5) * 0.03
        s.y[:] = np.where(o & 2, 0.02, 0.98) + (s.y - 0.5) * 0.03
    elif order == "jumps":            # a window holds one round and not the next
        o = np.arange(n)
        s.x[:] = np.where((o // 64) & 1, 0.1, 0.9) + (s.x - 0.5) * 0.05
    else:
        o = np.arange(n)
    return [np.ascontiguousarray(a[o]) for a in (s.x, s.y, s.z, s.m)]


@pytest.mark.parametrize("order", ["morton", "random", "corners", "jumps"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 70001])
@pytest.mark.parametrize("blob", ["narrow", "wide", "cubic"])
def test_image_over_orders(order, n, blob):
    import torch
    W, H = 200, 136                   # 13 x 9 tiles: windows cut by both edges
    cam, ocam = lib.Camera.ortho(W, H), osplat.Camera(0, W, H)
    p = _points(order, n, 11 + n)
    d = [torch.from_numpy(a).cuda() for a in p]
    if blob == "cubic":
        img = lib.splat(*d, cam, blob=lib.Blob.cubic(h_px=16.0 if n < 5000 else 4.5)).cpu().numpy()
        ref = ocubic.render(ocam, *p, h_px=16.0 if n < 5000 else 4.5)
    else:
        sigma, rad = (1.0, 3.0) if blob == "narrow" else (8.0, 6.0 if n < 5000 else 2.0)
        img = lib.splat(*d, cam, sigma, rad).cpu().numpy()
        ref = osplat.render(ocam, *p, sigma, rad)
    err, zeros_ok = image_rel_err(img, ref)
    assert zeros_ok and err <= TOL, err


@pytest.mark.parametrize("n,depth", [(1, 1), (2, 6), (1, 7)])
def test_cut_and_draw_list_over_block_edges(n, depth):
    """Trees of a few nodes and of several 1024-node cut blocks and 1024-id
    offset blocks: the cut equals the oracle's, the render its points' render."""
    s = synth.small_clustered(60000, 5)
    ref = olod.lod_build(s.x, s.y, s.z, s.m, n=n, D=depth, seed=1)
    tree = lib.build(*to_dev(s), lib.BuildParams(n=n, max_depth=depth, seed=1))
    cam, ocam = lib.Camera.ortho(128, 128), osplat.Camera(0, 128, 128)
    for tau in (0.01, 1.0, 60.0):
        ids, nsel = lib.select_nodes(tree, cam, tau, n)
        k = int(lib._to_numpy(nsel)[0])
        want = ocut.select(ref, ocam, tau, n)
        assert np.array_equal(lib._to_numpy(ids[:k]).astype(np.int64), want), (tau, k, len(want))
        img = lib.splat_lod(tree, ids, nsel, tree.point_capacity, cam).cpu().numpy()
        px, py, pz, pm = olod.decoded_points(ref, want)
        err, zeros_ok = image_rel_err(img, osplat.render(ocam, px, py, pz, pm))
        assert zeros_ok and err <= TOL, (tau, err)


@pytest.mark.parametrize("order", ["morton", "random", "clump"])
@pytest.mark.parametrize("aux", [False, True])
def test_cubic_window_classes(order, aux):
    """World radii whose pixel windows span every class of the cubic
    accumulation (4, 5, 6, 8 pixels and wider) in one render, at chunk
    remainders, with a clump whose records all cover the same few pixels."""
    import torch
    n, W, H = 4096 + 77, 96, 80
    rng = np.random.default_rng(3)
    p = _points(order if order != "clump" else "random", n, 21)
    if order == "clump":
        p[0][:n // 2] = 0.5 + 0.004 * (p[0][:n // 2] - 0.5)
        p[1][:n // 2] = 0.5 + 0.004 * (p[1][:n // 2] - 0.5)
    pos = (0.5, 0.5, -1.0)
    cam = lib.Camera.look_at(pos, (0.5, 0.5, 0.5), W, H, fov_deg=60.0)
    ocam = osplat.Camera(1, W, H, cam.pos, cam.right, cam.up, cam.fwd, cam.F, cam.near)
    # pixel radii from the clamp at 1 to the clamp at 16
    hw = (np.exp(rng.uniform(np.log(0.8), np.log(20.0), n)) * 1.5 / cam.F).astype(np.float32)
    col = rng.random(n).astype(np.float32)
    d = [torch.from_numpy(a).cuda() for a in p]
    dh, dc = torch.from_numpy(hw).cuda(), torch.from_numpy(col).cuda()
    got = lib.splat_interp(d, d, 0.5, cam, blob=lib.Blob.cubic(h_world=0.01), hA=dh, hB=dh,
                           cA=dc if aux else None, cB=dc if aux else None)
    want = ocubic.render(ocam, *p, h_world=hw, aux=col if aux else None)
    pairs = zip(got, want) if aux else ((got, want[0] if isinstance(want, tuple) else want),)
    for g, w in pairs:
        err, zeros_ok = image_rel_err(g.cpu().numpy(), w)
        assert zeros_ok and err <= TOL, err


@pytest.mark.parametrize("sigma,radius", [(0.3, 1.0), (0.49, 6.0), (0.5, 0.8), (0.5, 1.0), (0.5, 6.0), (0.663, 6.0),
                                          (1.0, 2.5), (1.0, 3.49), (1.0, 3.5), (1.326, 3.0), (1.327, 3.0)])
def test_gaussian_window_edges(sigma, radius):
    """Truncation radii at the edges of the narrow form's windows (one to nine
    pixels, tests on none, one and two of them) and of its range, both image
    channels, points on pixel and tile edges and outside the image."""
    import torch
    W, H, n = 70, 50, 3000
    rng = np.random.default_rng(8)
    x = rng.uniform(-0.1, 1.1, n).astype(np.float32)
    y = rng.uniform(-0.1, 1.1, n).astype(np.float32)
    x[:400] = (rng.integers(0, 2 * W + 1, 400) / 2 / W).astype(np.float32)     # pixel edges and centres
    y[200:600] = (rng.integers(0, 2 * H + 1, 400) / 2 / H).astype(np.float32)
    x[600:700] = (16 * rng.integers(0, 5, 100) / W).astype(np.float32)          # tile edges
    z = rng.random(n).astype(np.float32)
    m = rng.uniform(0.1, 1.0, n).astype(np.float32)
    a = rng.uniform(0.0, 2.0, n).astype(np.float32)
    cam, ocam = lib.Camera.ortho(W, H), osplat.Camera(0, W, H)
    d = [torch.from_numpy(t).cuda() for t in (x, y, z, m)]
    img = lib.splat(*d, cam, sigma, radius)
    both, aimg = lib.splat_aux(*d, torch.from_numpy(a).cuda(), cam, sigma, radius)
    ma = (m.astype(np.float64) * a.astype(np.float64))
    for got, mass in ((img, m), (both, m)):
        err, zeros_ok = image_rel_err(got.cpu().numpy(), osplat.render(ocam, x, y, z, mass, sigma, radius))
        assert zeros_ok and err <= TOL, err
    # the oracle takes float32 masses: the rounding of m a is within the tolerance
    err, zeros_ok = image_rel_err(aimg.cpu().numpy(),
                                  osplat.render(ocam, x, y, z, ma.astype(np.float32), sigma, radius))
    assert zeros_ok and err <= TOL, err


@pytest.mark.parametrize("blob", [None, "cubic"])
@pytest.mark.parametrize("N", [400_000, 700_000, 900_000, 1_100_000, 1_400_000])
def test_first_channel_is_the_plain_render_around_the_fixed_scratch(N, blob):
    """The form of the slice sums changes where a render nears the fixed
    scratch's size; the attribute channel's larger records do not move that
    line, so the image is the plain render's, bit for bit, on both sides."""
    import torch
    s = synth.uniform(N, 3)
    dev = to_dev(s)
    cam = lib.Camera.ortho(1024, 1024)
    b = lib.Blob.cubic(h_px=2.5) if blob else None
    img, _ = lib.splat_aux(*dev, torch.ones_like(dev[0]), cam, blob=b)
    plain = lib.splat(*dev, cam, blob=b)
    assert torch.equal(img.view(torch.int32), plain.view(torch.int32))


@pytest.mark.parametrize("size", [None, 256, "planned"])
def test_splat_workspace_forms(size):
    """A given workspace is tried before the plan is asked: the image is the
    same with none, one too small and the planned one, on the current stream,
    and what is refused without one is refused with one."""
    import torch
    s = synth.uniform(5000, 9)
    dev = to_dev(s)
    cam = lib.Camera.ortho(96, 80)
    want = lib.splat(*dev, cam)
    ws = None
    if size is not None:
        ws = torch.empty(lib.splat_workspace_bytes(5000, cam) if size == "planned" else size, dtype=torch.uint8,
                         device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert lib._stream().value == side.cuda_stream
        got = lib.splat(*dev, cam, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(got, want)
    with pytest.raises(lib.LodError):
        lib.splat(*dev, lib.Camera.ortho(0, 80), workspace=ws, out=want)
    with pytest.raises(lib.LodError):
        lib.splat(*dev, cam, sigma=-1.0, workspace=ws)


@pytest.mark.parametrize("W,H", [(512, 512), (513, 512)])
@pytest.mark.parametrize("N", [30_000, 40_000, 520_000, 600_000])
def test_chunk_scans_beside_the_tile_plan(W, H, N):
    """1024 tiles (their chunk scans run in the plan's block) and 1056 (in a
    launch of their own); one chunk of units, two, sixteen and nineteen."""
    s = synth.uniform(N, 12)
    img = lib.splat(*to_dev(s), lib.Camera.ortho(W, H)).cpu().numpy()
    err, zeros_ok = image_rel_err(img, osplat.render(osplat.Camera(0, W, H), s.x, s.y, s.z, s.m))
    assert zeros_ok and err <= 1e-5, (W, H, N, err)
