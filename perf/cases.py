"""Work that programs using this framework have it do, as measurable cases.

Each case is a dict of plain values.  ``prepare`` makes on the GPU what a
program holds before the call (particles, a built tree, workspaces, cameras),
``run`` is one pass through the public entry points, ``work`` counts the bytes
and operations that the pass cannot do without, and ``exact`` evaluates the
same outputs with plain torch in float64 and integers.

Kinds of case:

* ``build``  -- LOD build of one snapshot or of a batch of snapshots
* ``step``   -- build, then cut and LOD render of the new tree
* ``frame``  -- cut and LOD render of a resident tree (optionally with
  highlighted ids, or at a frame time between two snapshots)
* ``full``   -- render of every particle of a snapshot, in its own order
* ``interp`` -- render of every particle at a time between two snapshots, with
  per-particle radii and colours
* ``grad``   -- differentiable render and its adjoint (refinement)

Sizes follow the repository's configurations: 262,144 particles with n = 4096
and depth 4; 16.7 M with n = 16000 and depth 8; 150 M; batches of uneven
snapshots of 0.5 M to 8 M; 16,000 points of one node in a 1024 x 1024 view.
"""
from __future__ import annotations

import math

import torch

from paper_0811_2055_amd import autograd, lib

DEV = "cuda"
NODE_KEYS = ("prefix", "depth", "parent", "first_child", "child_mask", "part_begin", "part_count",
             "pt_begin", "pt_count", "node_mass")
POINT_KEYS = ("pt_id", "qx", "qy", "qz", "pt_mass")
SIGNED = {torch.uint64: torch.int64, torch.uint32: torch.int32, torch.uint16: torch.int16}


def listed():
    return [
        # one view of one optimisation step over a node's stored points: hundreds of
        # thousands of these make up a refinement, so its latency is what counts
        dict(name="refine_16k", kind="grad", N=16000, source="node", W=1024, H=1024, view="persp", blob="gauss"),
        # the interactive end: a small tree rebuilt, and its frame at a small image
        dict(name="build_262k", kind="build", N=262144, n=4096, depth=4, alpha=1, snaps=1, source="plummer"),
        dict(name="frame_262k", kind="frame", N=262144, n=4096, depth=4, source="plummer", W=256, H=256,
             view="ortho", tau=1.0, blob="gauss", extra="none"),
        # gradients of a whole render, the larger end of refinement, with the radial blob
        dict(name="grad_1m_cubic", kind="grad", N=1000003, source="sp", W=1024, H=1024, view="ortho", blob="cubic",
             h=2.5),
        # a 256^3 simulation: its tree, its interactive frames and its full-data render
        dict(name="build_16m", kind="build", N=16777216, n=16000, depth=8, alpha=1, snaps=1, source="nfw"),
        dict(name="frame_16m_motion", kind="frame", N=16777216, n=16000, depth=8, source="nfw", W=1024, H=1024,
             view="persp", tau=1.0, blob="gauss", extra="motion"),
        dict(name="full_16m", kind="full", N=16777216, source="nfw", W=1024, H=1024, view="persp", blob="gauss"),
        dict(name="frame_16m_cubic", kind="frame", N=16777216, n=16000, depth=8, source="nfw", W=1920, H=1080,
             view="persp", tau=1.0, blob="cubic", h=1.5, extra="none"),
        dict(name="frame_16m_highlight", kind="frame", N=16777216, n=16000, depth=8, source="nfw", W=1024, H=1024,
             view="persp", tau=2.0, blob="gauss", extra="highlight", ids=1000000),
        # frames between two snapshots with sizes and colours of their own
        dict(name="interp_4m", kind="interp", N=4000037, source="nfw", W=1024, H=1024, view="persp", blob="cubic"),
        # many snapshots of uneven size in one call
        dict(name="build_batch", kind="build", N=60000000, n=16000, depth=8, alpha=1, snaps=32, source="sp"),
        # one snapshot at full scale: build, cut and frame
        dict(name="step_150m", kind="step", N=150000000, n=16000, depth=8, alpha=1, snaps=1, source="sp", W=1024,
             H=1024, view="ortho", tau=1.0, blob="gauss", extra="none"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randint(0, 1)

    kind = rng.choice(["build", "build", "frame", "frame", "full", "interp", "grad", "grad"])
    img = dict(W=rng.choice([256, 512, 640, 801, 1024, 1280]), H=rng.choice([192, 256, 480, 515, 768, 1024]),
               view=rng.choice(["ortho", "persp"]), blob=rng.choice(["gauss", "gauss", "cubic"]))
    if img["blob"] == "cubic":
        img["h"] = round(rng.uniform(1.0, 6.0), 2)
    if kind == "grad":
        return dict(kind=kind, N=size(1000, 2000000), source=rng.choice(["node", "sp", "plummer"]), **img)
    if kind == "full":
        return dict(kind=kind, N=size(1e5, 3e7), source=rng.choice(["nfw", "sp", "plummer"]), **img)
    if kind == "interp":
        return dict(kind=kind, N=size(1e5, 6e6), source=rng.choice(["nfw", "sp"]),
                    **dict(img, view="persp", blob="cubic"))
    tree = dict(N=size(2e5, 6e7), n=rng.choice([1000, 4096, 10001, 16000]), depth=rng.randint(4, 8),
                source=rng.choice(["nfw", "sp", "plummer"]))
    # lists of the selection hold n + 1 entries per node of each level, so a small n stays with the small sets
    if tree["N"] > 4e6:
        tree["n"] = rng.choice([8000, 16000, 16384])
    if kind == "build":
        snaps = rng.choice([1, 1, 1, 5, 16])
        return dict(kind=kind, alpha=rng.choice([1, 1, 0, -1]), snaps=snaps, **tree)
    extra = rng.choice(["none", "none", "motion", "highlight"])
    c = dict(kind=kind, extra=extra, tau=rng.choice([0.7, 1.0, 2.0, 4.0]), **tree, **img)
    if extra == "highlight":
        c["ids"] = size(1e3, 1e6)
    return c


# ---------------------------------------------------------------------------
# inputs, from the seed alone


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _directions(g, k):
    v = torch.randn(k, 3, generator=g, device=DEV, dtype=torch.float64)
    return v / v.norm(dim=1, keepdim=True).clamp_min_(1e-30)


def _plummer(g, N):
    """20 Plummer spheres holding 70% of the particles, the rest uniform."""
    k = int(N * 0.7)
    c = torch.randint(0, 20, (k,), generator=g, device=DEV)
    a = (0.01 + 0.04 * _rand(g, 20))[c]
    r = a / torch.sqrt(_rand(g, k).clamp_(1e-12, 1 - 1e-12).pow(-2.0 / 3.0) - 1.0)
    return torch.cat([_rand(g, 20, 3)[c] + r[:, None] * _directions(g, k), _rand(g, N - k, 3)])


def _nfw(g, N):
    """500 NFW haloes with power-law masses (slope -1.9), 20% uniform background."""
    k = N - int(N * 0.2)
    u = _rand(g, 500)
    lo = 1e-3 ** -0.9
    mh = (lo + u * (1.0 - lo)).pow(1.0 / -0.9)
    rvir = 0.05 * (mh / mh.max()).pow(1.0 / 3.0)
    conc = 5.0 + 10.0 * _rand(g, 500)
    centre = _rand(g, 500, 3)
    h = torch.searchsorted(torch.cumsum(mh, 0) / mh.sum(), _rand(g, k)).clamp_(max=499)
    c = conc[h]
    want = _rand(g, k) * (torch.log1p(c) - c / (1.0 + c))
    a, b = torch.zeros_like(c), c.clone()
    for _ in range(32):                       # enclosed mass ln(1+x) - x/(1+x) inverted by bisection
        x = 0.5 * (a + b)
        low = torch.log1p(x) - x / (1.0 + x) < want
        a, b = torch.where(low, x, a), torch.where(low, b, x)
    r = a * rvir[h] / c
    return torch.cat([centre[h] + r[:, None] * _directions(g, k), _rand(g, N - k, 3)])


def _sp(g, N):
    """Soneira-Peebles clustering: 8 levels, eta 4, lambda 1.9."""
    levels, eta, lam = 8, 4, 1.9
    tops = max(1, -(-N // eta ** levels))
    radius = (3.0 / (4.0 * math.pi * tops)) ** (1.0 / 3.0)
    pos = _rand(g, tops, 3)
    for _ in range(levels):
        pos = pos.repeat_interleave(eta, dim=0)
        pos += (radius * _rand(g, pos.shape[0]).pow_(1.0 / 3.0))[:, None] * _directions(g, pos.shape[0])
        radius /= lam
    return pos[:N]


def _node(g, N):
    """Points of one octree node of side 1/8, in Morton order, as a tree stores them."""
    p = torch.cat([0.05 * torch.randn(N // 2, 3, generator=g, device=DEV, dtype=torch.float64) + 0.5,
                   _rand(g, N - N // 2, 3)]).clamp_(0.0, 1.0 - 1e-6)
    key = _morton(*(torch.floor(p[:, i] * 1024).long() for i in range(3)), 10)
    return 0.375 + 0.125 * p[torch.argsort(key, stable=True)]


SOURCES = dict(plummer=_plummer, nfw=_nfw, sp=_sp, node=_node)


def _particles(case, seed):
    """x, y, z, m (float32): wrapped into the unit cube, in an order without
    spatial meaning (a node's points keep theirs)."""
    g = _gen(seed)
    N = case["N"]
    off = None
    if case.get("snaps", 1) > 1:
        cut = torch.exp(_rand(g, case["snaps"]) * math.log(16.0))      # log-uniform sizes, 1 : 16
        ends = torch.floor(torch.cumsum(cut, 0) / cut.sum() * N).long()
        ends[-1] = N
        off = [0] + ends.tolist()
        parts = [SOURCES[case["source"]](g, b - a)[torch.randperm(b - a, generator=g, device=DEV)]
                 for a, b in zip(off, off[1:])]
        pos = torch.cat(parts)
        off = torch.tensor(off, dtype=torch.int64, device=DEV)
    else:
        pos = SOURCES[case["source"]](g, N)
        if case["source"] != "node":
            pos = pos[torch.randperm(N, generator=g, device=DEV)]
    xyz = []
    for i in range(3):
        a = pos[:, i]
        xyz.append((a - torch.floor(a)).float().clamp_(0.0, 1.0 - 2.0 ** -24))
    m = ((0.5 + _rand(g, N)) / N).float()
    return (*xyz, m), off, g


def _next_snapshot(p, g):
    """The same particles a little later: a smooth flow and some noise."""
    x, y, z, m = (a.double() for a in p)
    ph = _rand(g, 3) * 6.28
    out = []
    for i, (a, b) in enumerate(((x, y), (y, z), (z, x))):
        d = 0.01 * torch.sin(2 * math.pi * b + ph[i]) + 0.0005 * torch.randn(
            a.shape, generator=g, device=DEV, dtype=torch.float64)
        out.append((a + d).float().clamp_(0.0, 1.0 - 2.0 ** -24))
    return (*out, p[3])


def _camera(case, seed):
    W, H = case["W"], case["H"]
    if case["view"] == "ortho":
        return lib.Camera.ortho(W, H)
    s = (int(seed) % 97) / 97.0 - 0.5
    if case.get("source") == "node":          # where the node's points are drawn: 0.5 to 1 pixel apart
        F = (W / 2.0) / math.tan(math.radians(30.0))
        dist = F * 0.125 / (max(case["N"], 1) ** (1.0 / 3.0) * (0.75 + 0.4 * s))
        dist = max(dist, 0.2)
        pos = (0.4375 + 0.3 * dist, 0.4375 + 0.2 * dist, 0.4375 - math.sqrt(0.87) * dist)
        return lib.Camera.look_at(pos, (0.4375,) * 3, W, H, 60.0, near=1e-4)
    return lib.Camera.look_at((0.5 + 0.1 * s, 0.5, -0.9 + 0.05 * s), (0.5, 0.5, 0.5), W, H, 60.0)


def _blob(case):
    if case["blob"] == "gauss":
        return None
    return lib.Blob.cubic(h_world=0.002) if case["kind"] == "interp" else lib.Blob.cubic(h_px=case["h"])


def _params(case):
    return lib.BuildParams(n=case["n"], max_depth=case["depth"], alpha=case.get("alpha", 1), seed=7)


def _builder(case, p, off):
    b = lib.Builder(case["N"], _params(case), DEV, case.get("snaps", 1))
    for a in b.tree.arrays.values():          # capacity-sized: what a build does not reach stays 0
        _plain(a).zero_()
    return b


def prepare(case, seed):
    kind = case["kind"]
    p, off, g = _particles(case, seed)
    s = dict(kind=kind, p=p)
    if kind in ("build", "step"):
        s["off"] = None if off is None else off.view(torch.uint64)
        s["builder"] = _builder(case, p, off)
    if kind == "build":
        return s
    s["cam"], s["blob"] = _camera(case, seed), _blob(case)
    s["image"] = torch.zeros(case["H"], case["W"], device=DEV)
    if kind in ("full", "grad", "interp"):
        s["ws"] = torch.empty(lib.splat_workspace_bytes(case["N"], s["cam"], blob=s["blob"]), dtype=torch.uint8,
                              device=DEV)
    if kind == "interp":
        s["q"] = _next_snapshot(p, g)
        s["h"] = [(0.002 * (1.0 + _rand(g, case["N"]))).float() for _ in range(2)]
        s["c"] = [_rand(g, case["N"]).float() for _ in range(2)]
    if kind == "grad":
        s["p"] = tuple(a.clone().requires_grad_(True) for a in p)
        s["g"] = torch.randn(case["H"], case["W"], generator=g, device=DEV)
    if kind in ("step", "frame"):
        s["n"], s["tau"], s["extra"] = case["n"], case["tau"], case["extra"]
        s["max"] = case["N"]                  # a cut draws a particle at most once
        if kind == "frame":
            b = _builder(case, p, off)
            s["tree"] = b.build(*p)
            torch.cuda.synchronize()
            del b
        if case["extra"] == "motion":
            q = _next_snapshot(p, g)
            s["motion"] = lib.encode_motion(s["tree"], *q[:3])[:3]
            del q
        if kind == "frame":
            s["p"] = None                     # a viewer holds the tree, not the particles
        cap = s["builder"].tree.node_capacity if kind == "step" else s["tree"].node_capacity
        s["cut_ws"] = torch.empty(16 * cap + 65536, dtype=torch.uint8, device=DEV)
        if case["extra"] == "highlight":
            ids = torch.randperm(case["N"], generator=g, device=DEV)[:min(case["ids"], case["N"] // 4)]
            s["hl_max"] = int(ids.numel())
            bits = lib.highlight_bits(ids.cpu().numpy(), case["N"], DEV)
            s["flags"] = lib.highlight_flags(s["tree"], bits, case["N"])
            s["image_hl"] = torch.zeros_like(s["image"])
            need = lib.splat_lod_highlight_workspace_bytes(cap, s["max"], s["hl_max"], s["cam"], blob=s["blob"])
        else:
            need = lib.splat_lod_workspace_bytes(cap, s["max"], s["cam"], blob=s["blob"])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


# ---------------------------------------------------------------------------
# one pass


def _plain(t):
    return t.view(SIGNED[t.dtype]) if t.dtype in SIGNED else t


def _tree_out(tree):
    out = {k: _plain(tree.arrays[k]) for k in NODE_KEYS + POINT_KEYS}
    out["counts"] = _plain(tree.counts)
    return out


def _frame(s, tree):
    ids, nsel = lib.select_nodes(tree, s["cam"], s["tau"], s["n"], workspace=s["cut_ws"])
    if s["extra"] == "highlight":
        img, hl = lib.splat_lod_highlight(tree, ids, nsel, s["max"], s["cam"], s["flags"], s["hl_max"],
                                          workspace=s["ws"], out=s["image"], out_hl=s["image_hl"], blob=s["blob"])
        return {"image": img, "highlight": hl, "selected": _plain(nsel)}
    if s["extra"] == "motion":
        img = lib.splat_lod_motion(tree, ids, nsel, s["max"], s["motion"], 0.4, s["cam"], workspace=s["ws"],
                                   out=s["image"], blob=s["blob"])
    else:
        img = lib.splat_lod(tree, ids, nsel, s["max"], s["cam"], workspace=s["ws"], out=s["image"], blob=s["blob"])
    return {"image": img, "selected": _plain(nsel)}


def run(state):
    s = state
    kind = s["kind"]
    if kind == "build":
        return _tree_out(s["builder"].build(*s["p"], snap_offsets=s["off"]))
    if kind == "step":
        tree = s["builder"].build(*s["p"])
        return {**_tree_out(tree), **_frame(s, tree)}
    if kind == "frame":
        return _frame(s, s["tree"])
    if kind == "full":
        return {"image": lib.splat(*s["p"], s["cam"], workspace=s["ws"], out=s["image"], blob=s["blob"])}
    if kind == "interp":
        img, col = lib.splat_interp(s["p"], s["q"], 0.37, s["cam"], blob=s["blob"], hA=s["h"][0], hB=s["h"][1],
                                    cA=s["c"][0], cB=s["c"][1], workspace=s["ws"])
        return {"image": img, "colour": col}
    img = autograd.splat_render(*s["p"], s["cam"], workspace=s["ws"], blob=s["blob"])
    gx, gy, gz, gm = torch.autograd.grad(img, s["p"], s["g"])
    return {"image": img.detach(), "x": gx, "y": gy, "z": gz, "m": gm}


def work(case):
    """Inputs read once, outputs written once; per point and covered pixel one
    weight evaluated (about 6 operations) and added."""
    N, kind = case["N"], case["kind"]
    bytes_, flops = 0.0, 0.0
    if kind in ("build", "step"):
        bytes_ += 16.0 * N + 14.0 * 1.5 * N + 59.0 * 8 * N / case["n"]
    if kind == "build":
        return dict(bytes=bytes_, flops=0.0)
    radius = 3.0 if case["blob"] == "gauss" else (4.0 if kind == "interp" else case["h"])
    pixels = 4.0 * radius * radius if case["blob"] == "gauss" else math.pi * radius * radius
    per_point = {"step": 10.0, "frame": 16.0 if case.get("extra") == "motion" else 10.0, "full": 16.0,
                 "interp": 48.0, "grad": 32.0}[kind]
    # a cut in perspective at a pixel or more of spacing draws about half of the particles
    drawn = N * (1.0 if kind != "frame" or case["view"] == "ortho" else 0.5)
    bytes_ += per_point * drawn + 4.0 * case["W"] * case["H"] * (2.0 if kind in ("interp", "grad") else 1.0)
    flops += drawn * pixels * 8.0 * (3.0 if kind == "grad" else 1.0)
    return dict(bytes=bytes_, flops=flops)


# ---------------------------------------------------------------------------
# the same outputs in float64 and integers, with torch alone


def _spread(v, bits):
    out = torch.zeros_like(v)
    for b in range(bits):
        out |= ((v >> b) & 1) << (3 * b)
    return out


def _morton(cx, cy, cz, bits):
    return _spread(cx, bits) | (_spread(cy, bits) << 1) | (_spread(cz, bits) << 2)


def _philox_u(ids, snap, seed):
    """Philox4x32-10 output word 0 plus 1 of counter (id, 0, snapshot, 0)."""
    M = 0xFFFFFFFF

    def mul(a, b):                            # 32 x 32 -> (high, low) in int64
        p, q = a * (b & 0xFFFF), a * (b >> 16)
        return ((q + (p >> 16)) >> 16) & M, ((q << 16) + p) & M

    c0, c1, c2, c3 = ids & M, ids >> 32, snap, torch.zeros_like(ids)
    k0, k1 = seed & M, (seed >> 32) & M
    for _ in range(10):
        h0, l0 = mul(c0, 0xD2511F53)
        h1, l1 = mul(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0 + 1


def _exact_tree(p, off, n, D, alpha, seed):
    """The tree of the particles: node table, stored points, float64 masses."""
    x, y, z, m = p
    N, dev = x.numel(), x.device
    gid = torch.arange(N, device=dev)
    snap = torch.zeros_like(gid) if off is None else torch.searchsorted(off, gid, right=True) - 1
    fix = [torch.floor(a.double() * 2.0 ** (D + 16)).long().clamp_(max=(1 << (D + 16)) - 1) for a in (x, y, z)]
    key = _morton(*(f >> 16 for f in fix), D) | (snap << (3 * D))
    skey, order = torch.sort(key, stable=True)
    del key
    _, inv, cnt = torch.unique_consecutive(skey, return_inverse=True, return_counts=True)
    w = cnt[inv]                              # particles in the depth-D cell
    del inv, cnt
    lid = order if off is None else order - off[snap[order]]
    U = _philox_u(lid, snap[order], seed)
    if alpha > 0:
        a, b = (1 << 31) // w, (1 << 31) % w
        K = torch.where((w == 1) & (U == 1 << 32), torch.full_like(U, (1 << 63) - 1), U * a + (U * b) // w)
        wp = w.double()
    elif alpha == 0:
        K = torch.where(U == 1 << 32, torch.full_like(U, (1 << 63) - 1), U << 31)
        wp = torch.ones_like(w, dtype=torch.float64)
    else:
        K, wp = U * w, 1.0 / w.double()
    by_id = torch.argsort(order)              # sorted positions in id order, then stably by K
    korder = by_id[torch.sort(K[by_id], stable=True)[1]]
    del by_id, K
    ms = m[order].double()
    csum = torch.cat([torch.zeros(1, dtype=torch.float64, device=dev), torch.cumsum(ms, 0)])
    levels, points = [], []
    start = count = None
    for d in range(D + 1):
        cell = skey >> (3 * (D - d))
        head = torch.cat([torch.ones(1, dtype=torch.bool, device=dev), cell[1:] != cell[:-1]])
        st = head.nonzero()[:, 0]
        del head
        ct = torch.diff(torch.cat([st, torch.tensor([N], device=dev)]))
        if d:                                 # children of splitting nodes only
            par = torch.searchsorted(start, st, right=True) - 1
            ok = (par >= 0) & (st < start[par.clamp_min(0)] + count[par.clamp_min(0)]) & (count[par.clamp_min(0)] > n)
            st, ct = st[ok], ct[ok]
        if not st.numel():
            break
        start, count = st, ct
        M = csum[st + ct] - csum[st]
        node = torch.full((N,), -1, dtype=torch.int32, device=dev)
        node[_ranges(st, ct)] = torch.repeat_interleave(
            torch.arange(st.numel(), dtype=torch.int32, device=dev), ct)
        big = ct > n
        take = node >= 0
        mass = ms
        if bool(big.any()):
            grp, o = torch.sort(node[korder], stable=True)
            first = torch.searchsorted(grp, torch.arange(st.numel(), dtype=torch.int32, device=dev))
            g = grp.long().clamp_min(0)
            rank = torch.arange(N, device=dev) - first[g]
            pos = korder[o]
            drop = (grp >= 0) & big[g] & (rank >= n)
            take[pos[drop]] = False
            wit = pos[(grp >= 0) & big[g] & (rank == n)]           # in node order
            del grp, o, g, rank, pos, drop
            tau = torch.ones(st.numel(), dtype=torch.float64, device=dev)
            tau[big] = wp[wit] * 2.0 ** 32 / U[wit].double()
            sel = take & big[node.long().clamp_min(0)] & (node >= 0)
            i = sel.nonzero()[:, 0]
            v = node[i].long()
            raw = ms[i] / torch.clamp(wp[i] / tau[v], max=1.0)
            tot = torch.zeros(st.numel(), dtype=torch.float64, device=dev).index_add_(0, v, raw)
            mass = ms.clone()
            mass[i] = raw * (M / tot.clamp_min(1e-300))[v]
            del sel, i, v, raw
        i = take.nonzero()[:, 0]
        cells = skey[st] >> (3 * (D - d))
        o = order[i]
        points.append(dict(node=node[i].long(), id=lid[i], mass=mass[i],
                           q=[((f[o] >> (D - d)) & 0xFFFF) for f in fix], orig=o))
        levels.append(dict(cell=cells, begin=st, count=ct, mass=M, split=big & (d < D),
                           stored=torch.clamp(ct, max=n)))
        del node, take, mass
    return levels, points


def _ranges(st, ct):
    first = torch.cumsum(ct, 0) - ct
    return torch.arange(int(ct.sum()), device=st.device) + torch.repeat_interleave(st - first, ct)


def _compact(v, bits):
    out = torch.zeros_like(v)
    for b in range(bits):
        out |= ((v >> (3 * b)) & 1) << b
    return out


def _exact_cut(levels, D, cam, tau, n):
    """Per level, which nodes are drawn."""
    drawn, live = [], None
    limit = tau * n ** (1.0 / 3.0)
    for d, L in enumerate(levels):
        side = 2.0 ** -d
        cell = L["cell"] & ((1 << (3 * d)) - 1)
        o = [_compact(cell >> k, d).double() * side for k in range(3)]
        if cam.projection == 0:
            want = torch.full_like(L["split"], cam.W * side > limit)
        else:
            pos = torch.tensor(cam.pos, dtype=torch.float32).double().tolist()
            F = float(torch.tensor(cam.F, dtype=torch.float32))
            inside = torch.ones_like(L["split"])
            for a, c in zip(o, pos):
                inside &= (a <= c) & (c <= a + side)
            dist = torch.sqrt(sum((a + side * 0.5 - c) ** 2 for a, c in zip(o, pos)))
            want = inside | (F * side > limit * dist)
        go = L["split"] & want
        if d:
            up = levels[d - 1]
            par = torch.searchsorted(up["begin"], L["begin"], right=True) - 1
            here = live[par]
        else:
            here = torch.ones_like(go)
        drawn.append(here & ~go)
        live = here & go
    return drawn


def _exact_lod_points(case, p, q, levels, points, drawn):
    """Decoded positions (float32) and masses of the drawn stored points, and their ids."""
    out = []
    t = torch.tensor(0.4, dtype=torch.float32).item()
    for d, (L, P, keep) in enumerate(zip(levels, points, drawn)):
        i = keep[P["node"]].nonzero()[:, 0]
        if not i.numel():
            continue
        v = P["node"][i]
        cell = L["cell"][v] & ((1 << (3 * d)) - 1)
        xyz = []
        for k in range(3):
            Q = (_compact(cell >> k, d) << 16) + P["q"][k][i]
            a = ((2 * Q + 1).double() * 2.0 ** -(d + 17)).float()
            if q is not None:
                Q1 = torch.floor(q[k][P["orig"][i]].double() * 2.0 ** (d + 16)).long()
                dq = ((Q1 - Q + 2) >> 2).clamp_(-32768, 32767)
                b = ((2 * (Q + 4 * dq) + 1).double() * 2.0 ** -(d + 17)).float()
                a = a + (b - a) * t
            xyz.append(a)
        out.append((*xyz, P["mass"][i].float().double(), P["id"][i]))
    return [torch.cat([o[k] for o in out]) for k in range(5)]


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def _project(cam, x, y, z):
    """Screen positions by the library's float32 sequence, visibility, depth."""
    if cam.projection == 0:
        return x * float(cam.W), y * float(cam.H), torch.ones_like(x, dtype=torch.bool), (None, None, None)
    d = [a - _f32(c) for a, c in zip((x, y, z), cam.pos)]
    dot = lambda e: (d[0] * _f32(e[0]) + d[1] * _f32(e[1])) + d[2] * _f32(e[2])  # noqa: E731
    xc, yc, zc = dot(cam.right), dot(cam.up), dot(cam.fwd)
    vis = zc > _f32(cam.near)
    zs = torch.where(vis, zc, torch.ones_like(zc))
    u = (xc.double() / zs.double()).float() * _f32(cam.F) + cam.W * 0.5
    v = (yc.double() / zs.double()).float() * _f32(cam.F) + cam.H * 0.5
    return u, v, vis, (xc, yc, zs)


def _cubic(qq):
    return torch.where(qq <= 0.5, 1.0 - 6.0 * qq * qq + 6.0 * qq ** 3, 2.0 * (1.0 - qq).clamp_min(0.0) ** 3)


CUBIC_NORM = 40.0 / (7.0 * math.pi)


def _footprint(cam, u, v, reach):
    """Every pixel offset pair within `reach` of the points: (flat index, ox, oy, inside the image)."""
    i0 = torch.floor(u.double() - 0.5 - reach).long()
    j0 = torch.floor(v.double() - 0.5 - reach).long()
    k = 2 * int(math.ceil(reach)) + 2
    for b in range(k):
        j = j0 + b
        oy = v - (j.float() + 0.5)
        for a in range(k):
            i = i0 + a
            ox = u - (i.float() + 0.5)
            ok = (i >= 0) & (i < cam.W) & (j >= 0) & (j < cam.H)
            yield j.clamp(0, cam.H - 1) * cam.W + i.clamp(0, cam.W - 1), ox, oy, ok


def _weight(ox, oy, h):
    """Blob value at float32 offsets, in float64 (h: cubic radius, or None for the Gaussian of sigma 1)."""
    if h is None:
        on = (ox.abs() <= 3.0) & (oy.abs() <= 3.0)
        return torch.where(on, torch.exp(-0.5 * (ox.double() ** 2 + oy.double() ** 2)) / (2 * math.pi), 0.0)
    r2 = ox.double() ** 2 + oy.double() ** 2
    return torch.where(r2 < h * h, CUBIC_NORM / (h * h) * _cubic(torch.sqrt(r2) / h), 0.0)


def _exact_image(cam, x, y, z, masses, blob, hw=None, step=1 << 21):
    imgs = [torch.zeros(cam.H * cam.W, dtype=torch.float64, device=x.device) for _ in masses]
    for c in range(0, x.numel(), step):
        s = slice(c, c + step)
        u, v, vis, cc = _project(cam, x[s], y[s], z[s])
        lim = 20.0
        vis = vis & (u > -lim) & (u < cam.W + lim) & (v > -lim) & (v < cam.H + lim)
        keep = vis.nonzero()[:, 0]
        u, v = u[keep], v[keep]
        ms = [m[s][keep] for m in masses]
        h, reach = None, 3.0
        if blob is not None and hw is None:
            h, reach = _f32(blob.h_px), _f32(blob.h_px)
        elif blob is not None:
            zc = cc[2][keep].double()
            h = ((hw[s][keep] * _f32(cam.F)).double() / zc).float().clamp(1.0, 16.0).double()
            reach = float(h.max()) if h.numel() else 1.0
        for idx, ox, oy, ok in _footprint(cam, u, v, reach):
            wt = torch.where(ok, _weight(ox, oy, h), 0.0)
            for img, m in zip(imgs, ms):
                img.index_add_(0, idx, wt * m)
    return [i.view(cam.H, cam.W) for i in imgs]


def _exact_grad(cam, p, g, blob):
    x, y, z, m = p
    u, v, vis, (xc, yc, zc) = _project(cam, x, y, z)
    h = None if blob is None else _f32(blob.h_px)
    gf = g.double().reshape(-1)
    am, au, av = (torch.zeros(x.numel(), dtype=torch.float64, device=x.device) for _ in range(3))
    for idx, ox, oy, ok in _footprint(cam, u.clamp(-1e4, 1e5), v.clamp(-1e4, 1e5), 3.0 if h is None else h):
        ok = ok & vis
        gp = torch.where(ok, gf[idx], 0.0)
        oxd, oyd = ox.double(), oy.double()
        if h is None:
            G = _weight(ox, oy, None) * gp
            am += G
            au -= G * oxd
            av -= G * oyd
        else:
            r2 = oxd ** 2 + oyd ** 2
            qq = torch.sqrt(r2) / h
            slope = torch.where(qq <= 0.5, -12.0 + 18.0 * qq, -6.0 * (1.0 - qq) ** 2 / qq.clamp_min(0.25))
            t = torch.where(r2 < h * h, CUBIC_NORM / h ** 4 * slope, 0.0) * gp
            am += _weight(ox, oy, h) * gp
            au += t * oxd
            av += t * oyd
    au, av = au * m.double(), av * m.double()
    if cam.projection == 0:
        gx, gy, gz = au * cam.W, av * cam.H, torch.zeros_like(au)
    else:
        F, zz = _f32(cam.F), zc.double()
        a, bu, bv = F / zz, F * xc.double() / zz ** 2, F * yc.double() / zz ** 2
        r, up, f = ([_f32(e) for e in t] for t in (cam.right, cam.up, cam.fwd))
        gx, gy, gz = (torch.where(vis, au * (a * r[k] - bu * f[k]) + av * (a * up[k] - bv * f[k]), 0.0)
                      for k in range(3))
    return gx, gy, gz, am


def exact(case, seed):
    kind = case["kind"]
    p, off, g = _particles(case, seed)
    if kind in ("build", "step", "frame"):
        n, D = case["n"], case["depth"]
        levels, points = _exact_tree(p, off, n, D, case.get("alpha", 1), 7)
    if kind in ("build", "step"):
        _, node_cap, point_cap = lib.build_plan(case["N"], _params(case), case.get("snaps", 1))
        mass = torch.zeros(max(node_cap, 1), dtype=torch.float64, device=DEV)
        a = torch.cat([L["mass"] for L in levels])
        mass[:a.numel()] = a
        pm = torch.zeros(max(point_cap, 1), dtype=torch.float64, device=DEV)
        a = torch.cat([P["mass"] for P in points])
        pm[:a.numel()] = a
        out = {k: None for k in NODE_KEYS + POINT_KEYS + ("counts",)}
        out.update(node_mass=mass, pt_mass=pm)
        if kind == "build":
            return out
    cam, blob = _camera(case, seed), _blob(case)
    if kind in ("step", "frame"):
        q = _next_snapshot(p, g) if case["extra"] == "motion" else None
        drawn = _exact_cut(levels, D, cam, case["tau"], n)
        x, y, z, m, ids = _exact_lod_points(case, p, q, levels, points, drawn)
        del levels, points
        masses = [m]
        if case["extra"] == "highlight":
            on = torch.zeros(case["N"], dtype=torch.float64, device=DEV)
            on[torch.randperm(case["N"], generator=g, device=DEV)[:min(case["ids"], case["N"] // 4)]] = 1.0
            masses.append(m * on[ids])
        imgs = _exact_image(cam, x, y, z, masses, blob)
        img = {"image": imgs[0], "selected": None}
        if case["extra"] == "highlight":
            img["highlight"] = imgs[1]
        return {**out, **img} if kind == "step" else img
    if kind == "full":
        return {"image": _exact_image(cam, *p[:3], [p[3].double()], blob)[0]}
    if kind == "interp":
        t = _f32(0.37)
        q = _next_snapshot(p, g)
        h = [(0.002 * (1.0 + _rand(g, case["N"]))).float() for _ in range(2)]
        c = [_rand(g, case["N"]).float() for _ in range(2)]
        mix = lambda a, b: a + (b - a) * t  # noqa: E731
        m = mix(p[3], q[3]).double()
        img, col = _exact_image(cam, *(mix(a, b) for a, b in zip(p[:3], q[:3])), [m, m * mix(*c).double()], blob,
                                mix(*h))
        return {"image": img, "colour": col}
    gi = torch.randn(case["H"], case["W"], generator=g, device=DEV)
    gx, gy, gz, gm = _exact_grad(cam, p, gi, blob)
    img = _exact_image(cam, *p[:3], [p[3].double()], blob)[0]
    return {"image": img, "x": gx, "y": gy, "z": gz, "m": gm}
