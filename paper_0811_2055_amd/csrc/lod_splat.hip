// Additive Gaussian point splat, its adjoint, and the LOD point decode for
// gfx950 (rendering paragraph of arXiv:0811.2055: every point drawn as a
// blob evaluated for each pixel it covers).
//
// Forward: points are binned to 16x16 pixel tiles by a stable counting sort
// (per-wave units, a count pass and a fill pass, ballot ranks inside the
// wave), so a tile's pair list depends on the input alone.  Each list is cut
// into slices; one 256-thread block per slice adds the separable blobs to its
// 16x16 tile as rank-64 products on the matrix cores (MFMA 16x16x4, float32).
// Each wave adds its products to float64 sums of its own, the four wave sums
// of a pixel are added in wave order at the end of the slice, and a final pass
// adds a tile's slice partials in slice order.  The cubic blob, which is not
// separable, is evaluated pixel by pixel (float64).  Every order of addition
// is fixed: the image is bit-reproducible.  The LOD render feeds the binning
// straight from the tree's 16-bit node-relative points, decoding them in
// registers.
//
// The screen position and pixel offsets follow a fixed float32 sequence with
// no contraction (this file is compiled with -ffp-contract=off) so that the
// set of pixels a point covers is decided exactly as written.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>
#include <cmath>

#include "lod.h"
#include "lod_device.hpp"
#include "lod_internal.hpp"
#include "lod_scan.hpp"

using namespace lodk;

namespace {

constexpr int TS = lodh::SPLAT_TS;
constexpr int PT = 256;            // threads per block

struct Cam {
  uint32_t proj, W, H;
  float px, py, pz, rx, ry, rz, ux, uy, uz, fx, fy, fz, F, near_z;
  float R;          // truncation half-width in pixels (float32)
  float inv2s2;     // 1 / (2 sigma^2)
  float norm;       // 1 / (2 pi sigma^2)
  float wscale;     // the power of two below it: multiplies masses without rounding
  double wnorm;     // the rest of the normalisation: multiplies a slice's float64 sums
  float inv_s2;     // 1 / sigma^2
  int nin, nmax;    // pixels at most nin from the one that holds the point are covered, none beyond nmax is
  float kexp2;      // -log2(e) / (2 sigma^2): Gaussian factor = exp2(o^2 kexp2)
  uint32_t tiles_x, tiles_y;
  uint32_t blob;    // LOD_BLOB_GAUSSIAN or LOD_BLOB_CUBIC
  float hpx;        // cubic: fixed pixel radius (when Fhw == 0)
  float Fhw;        // cubic, perspective world size: fl(F h_world), else 0
};

Cam make_cam(const lod_camera &c, const splat_params &sp, const lodh::SplatLayout *L) {
  Cam k{};
  k.proj = c.projection; k.W = c.W; k.H = c.H;
  k.px = c.pos[0]; k.py = c.pos[1]; k.pz = c.pos[2];
  k.rx = c.right[0]; k.ry = c.right[1]; k.rz = c.right[2];
  k.ux = c.up[0]; k.uy = c.up[1]; k.uz = c.up[2];
  k.fx = c.fwd[0]; k.fy = c.fwd[1]; k.fz = c.fwd[2];
  k.F = c.F; k.near_z = c.near_z;
  const float s = sp.sigma_px;
  k.R = sp.radius_sigmas * s;
  const double s64 = (double)s;
  k.inv2s2 = (float)(1.0 / (2.0 * s64 * s64));
  k.norm = (float)(1.0 / (2.0 * M_PI * s64 * s64));
  k.inv_s2 = (float)(1.0 / (s64 * s64));
  const double kexp2 = -1.4426950408889634 / (2.0 * s64 * s64);
  k.kexp2 = (float)kexp2;
  // the point lies within half a pixel of its pixel's centre; the binning admits
  // pixels 1/100 further out, and its float32 range and the
  // offsets are within 1/200 pixel of the exact ones
  k.nin = (int)std::floor((double)k.R - 0.52);
  k.nmax = (int)std::floor((double)k.R + 0.52);
  const double norm = 1.0 / (2.0 * M_PI * s64 * s64);
  const int e2 = std::min(std::ilogb(norm), 127);
  k.wscale = std::ldexp(1.0f, e2);
  // the Gaussian drawn is that of the rounded exponent constant: a blob keeps
  // its mass (a bias of up to 3.6e-8 of every dense pixel otherwise)
  k.wnorm = norm / std::ldexp(1.0, e2) * (std::isfinite(k.kexp2) ? (double)k.kexp2 / kexp2 : 1.0);
  if (L) { k.tiles_x = L->tiles_x; k.tiles_y = L->tiles_y; }
  k.blob = sp.blob;
  k.hpx = sp.h_px;
  k.Fhw = (sp.blob == LOD_BLOB_CUBIC && sp.h_world > 0.0f) ? c.F * sp.h_world : 0.0f;
  return k;
}

// Pinned float32 projection; returns false when culled.
__device__ __forceinline__ bool project(const Cam &c, float x, float y, float z, float &u, float &v,
                                        float &xc, float &yc, float &zc) {
  if (c.proj == 0) {
    u = x * (float)c.W;
    v = y * (float)c.H;
    xc = yc = zc = 0.0f;
    return true;
  }
  const float dx = x - c.px, dy = y - c.py, dz = z - c.pz;
  xc = ((dx * c.rx) + (dy * c.ry)) + (dz * c.rz);
  yc = ((dx * c.ux) + (dy * c.uy)) + (dz * c.uz);
  zc = ((dx * c.fx) + (dy * c.fy)) + (dz * c.fz);
  if (!(zc > c.near_z)) return false;
  u = (c.F * __fdiv_rn(xc, zc)) + (float)c.W * 0.5f;
  v = (c.F * __fdiv_rn(yc, zc)) + (float)c.H * 0.5f;
  return true;
}

// First and last index in [lo_clip, hi_clip] whose float32 offset
// fl(t - (i + 1/2)) lies in [-R, R].  The offset is non-increasing in i, so
// the set is an interval; a float estimate is corrected by exact tests.
__device__ __forceinline__ bool clip_range(float t, float R, int lo_clip, int hi_clip, int &lo, int &hi) {
  auto inside_hi = [&](int i) { return t - ((float)i + 0.5f) >= -R; };   // offset not below -R
  auto inside_lo = [&](int i) { return t - ((float)i + 0.5f) <= R; };    // offset not above R
  int a = (int)floorf(t - 0.5f - R);
  while (!inside_lo(a)) ++a;
  while (inside_lo(a - 1)) --a;
  int b = (int)floorf(t - 0.5f + R);
  while (!inside_hi(b)) --b;
  while (inside_hi(b + 1)) ++b;
  lo = max(a, lo_clip);
  hi = min(b, hi_clip);
  return lo <= hi;
}

// Inclusive range [lo, hi] of pixel indices along one axis whose float32
// offset fl(t - (i + 1/2)) lies within [-R, R], clipped to [0, size).
__device__ __forceinline__ bool axis_range(const Cam &c, float t, uint32_t size, int &lo, int &hi) {
  const float lim = c.R + 4.0f;
  if (!(t > -lim && t < (float)size + lim)) return false;
  return clip_range(t, c.R, 0, (int)size - 1, lo, hi);
}

// --- binning -----------------------------------------------------------------
//
// Points are binned to 16x16 pixel tiles by a stable counting sort, so that
// every tile's pair list -- and with it the image -- is a function of the
// input alone.  The points are cut into rounds of 64 consecutive ones and the
// rounds into U = 64 C contiguous ranges ("units"), one wave each.  Pass 1
// counts each unit's pairs per tile into row u of a [U][tiles] table; two
// column scans (within chunks of 64 units, then over the C chunks) and a scan
// over tiles give every (tile, unit) its slot range.  Pass 2 re-derives the
// pairs in the same order, so a tile's list is ordered by round and, inside
// a round, by lane (rounds that spread too far: by the tile's index within
// the point, then by lane).  Rounds start at multiples of 64, so the lists do
// not depend on how many units there are.
//
// What bounds both passes is instruction issue, and the chain from one round's
// counters to the next one's.  A wave therefore keeps the counters of an 8x8
// tile window in its 64 lanes (lane l: tile column l % 8, row l / 8).  A round
// whose points all fall in the window (nearly all rounds of points in Morton
// order) turns every point's tile rectangle into a 64-bit cell mask, ORs the
// masks over the wave, and visits each set cell once: one ballot gives the
// cell's points, their number and their ranks, with no table access.

constexpr int BW = 64;              // binning block: one wave, one unit
constexpr int BR = 8;               // rounds of 64 points loaded together by the count pass
constexpr int BR_FILL = 8;          // and by the fill pass
constexpr int WINT = 8;             // window edge in tiles: WINT * WINT == WAVE

// decoded float32 coordinate of a stored point (cell coordinate c at depth d,
// 16-bit offset q): centre of the quantisation cell, exact in float32
__device__ __forceinline__ float decode_coord(uint32_t c, uint32_t q, int d) {
  return (float)(2u * ((c << 16) + q) + 1u) * ldexpf(1.0f, -(d + 17));
}

// float32 nearest (2 (c 2^16 + q + 4 dq) + 1) 2^-(d+17): the position a motion
// code dq moves a stored point to (signed: a point may leave its cell)
__device__ __forceinline__ float decode_motion(uint32_t c, uint32_t q, int dq, int d) {
  const int64_t Q = ((int64_t)c << 16) + (int64_t)q + 4 * (int64_t)dq;
  return (float)(2 * Q + 1) * ldexpf(1.0f, -(d + 17));
}

// fl(a + fl(t fl(b - a))): the value at frame time t in [0, 1] between a and b
__device__ __forceinline__ float lerp_t(float a, float b, float t) { return a + t * (b - a); }

// offset of listed node k (k_lod_offsets)
constexpr int LOFF = 1024;
__device__ __forceinline__ uint64_t lod_off(const uint64_t *offs, const uint64_t *bsum, uint64_t k) {
  return offs[k] + bsum[k / LOFF];
}

// Point sources.  A wave first resolves the addresses of its next BR rounds of
// points (resolve + end_round, in round order), then issues all their loads
// at once (fetch), so one memory latency covers BR rounds.

// raw float32 arrays
struct RawSrc {
  const float *x, *y, *z, *m;
  uint64_t n;
  struct Addr {
    uint64_t k;
  };
  struct Cursor {
    uint64_t last;      // a valid index: loads are unconditional (a predicated
                        // load would be waited for on its own)
    __device__ void begin(const RawSrc &, uint64_t b, uint64_t e) { last = e - 1; }
    __device__ __forceinline__ Addr resolve(const RawSrc &, uint64_t k, bool valid) {
      return Addr{valid ? k : last};
    }
    __device__ void end_round(const RawSrc &) {}
    __device__ __forceinline__ void fetch(const RawSrc &s, const Addr &a, bool, float &px, float &py,
                                          float &pz, float &pm) const {
      px = s.x[a.k]; py = s.y[a.k]; pz = s.z[a.k]; pm = s.m[a.k];
    }
    // the point's attribute (second image channel)
    __device__ __forceinline__ float attr(const RawSrc &s, const Addr &a) const { return s.aux[a.k]; }
    __device__ __forceinline__ float wradius(const RawSrc &, const Addr &) const { return 0.0f; }
  };
  __device__ uint64_t count() const { return n_dev ? min(*n_dev, n) : n; }
  const float *aux = nullptr;
  const uint64_t *n_dev = nullptr;   // device count (at most n), when set
};

// Two snapshots of the same particles and a frame time t: every quantity is
// fl(a + fl(t fl(b - a))); per-point world radii (cubic blob) and colours
// are optional.
struct InterpSrc {
  const float *xa, *ya, *za, *ma, *xb, *yb, *zb, *mb;
  const float *ha, *hb, *ca, *cb;   // may be null
  uint64_t n;
  float t;
  struct Addr {
    uint64_t k;
  };
  struct Cursor {
    uint64_t last;
    __device__ void begin(const InterpSrc &, uint64_t b, uint64_t e) { last = e - 1; }
    __device__ __forceinline__ Addr resolve(const InterpSrc &, uint64_t k, bool valid) {
      return Addr{valid ? k : last};
    }
    __device__ void end_round(const InterpSrc &) {}
    __device__ __forceinline__ void fetch(const InterpSrc &s, const Addr &a, bool, float &px, float &py,
                                          float &pz, float &pm) const {
      const float x0 = s.xa[a.k], y0 = s.ya[a.k], z0 = s.za[a.k], m0 = s.ma[a.k];
      const float x1 = s.xb[a.k], y1 = s.yb[a.k], z1 = s.zb[a.k], m1 = s.mb[a.k];
      px = lerp_t(x0, x1, s.t); py = lerp_t(y0, y1, s.t); pz = lerp_t(z0, z1, s.t); pm = lerp_t(m0, m1, s.t);
    }
    __device__ __forceinline__ float attr(const InterpSrc &s, const Addr &a) const {
      return lerp_t(s.ca[a.k], s.cb[a.k], s.t);
    }
    __device__ __forceinline__ float wradius(const InterpSrc &s, const Addr &a) const {
      return s.ha ? lerp_t(s.ha[a.k], s.hb[a.k], s.t) : 0.0f;
    }
  };
  __device__ uint64_t count() const { return n; }
};

// The stored points of a list of tree nodes, decoded on the fly.  offs is the
// exclusive scan of the nodes' point counts; the wave keeps the node holding
// its current point in registers and walks offs per lane when a round crosses
// into later nodes.
template <bool MOTION>
struct TreeSrcT {
  lod_tree t;
  const uint32_t *ids;
  const uint64_t *offs, *bsum;   // offset of node k: lod_off
  const uint64_t *n_ids;
  uint64_t max_ids;
  const uint64_t *total;     // points to draw (device)
  __device__ __forceinline__ uint64_t off(uint64_t k) const { return lod_off(offs, bsum, k); }
  struct Addr {
    uint64_t sidx;
    uint32_t cx, cy, cz;
    int d;
  };
  struct Cursor {
    uint64_t c, ob, oe, pb, far_c;
    uint32_t cx, cy, cz;
    int d;
    __device__ __forceinline__ void set(const TreeSrcT &s, uint64_t cc) {
      c = cc;
      const uint32_t v = s.ids[cc];
      ob = s.off(cc); oe = s.off(cc + 1);
      d = s.t.depth[v];
      const uint64_t pfx = s.t.prefix[v];
      const uint32_t cell = d ? (uint32_t)(pfx & ((1ull << (3 * d)) - 1)) : 0u;
      cx = compact3(cell); cy = compact3(cell >> 1); cz = compact3(cell >> 2);
      pb = s.t.pt_begin[v];
      far_c = cc;
    }
    __device__ void begin(const TreeSrcT &s, uint64_t b, uint64_t) {
      // the last node whose offset is <= b; it holds point b (b < total).  The
      // wave's 64 lanes probe the range together: three dependent reads for
      // 33 thousand nodes instead of fifteen, which every unit waits for
      // before its first point.
      const uint32_t lane = threadIdx.x & (WAVE - 1);
      uint64_t lo = 0, hi = min(*s.n_ids, s.max_ids);
      while (hi - lo > 1) {
        const uint64_t step = (hi - lo + WAVE - 1) / WAVE, p = lo + step * (lane + 1);
        const uint64_t c = (uint64_t)__popcll(__ballot(p < hi && s.off(min(p, hi - 1)) <= b));
        hi = min(hi, lo + step * (c + 1));
        lo += step * c;
      }
      set(s, lo);
    }
    __device__ __forceinline__ Addr resolve(const TreeSrcT &s, uint64_t k, bool valid) {
      // invalid lanes load the cached node's first point (in bounds, unused)
      Addr a{pb, cx, cy, cz, d};
      if (!valid) return a;
      if (k < oe) {
        a.sidx = pb + (k - ob);
        return a;
      }
      uint64_t cl = c + 1;
      while (s.off(cl + 1) <= k) ++cl;
      far_c = max(far_c, cl);
      const uint32_t v = s.ids[cl];
      a.d = s.t.depth[v];
      const uint64_t pfx = s.t.prefix[v];
      const uint32_t cell = a.d ? (uint32_t)(pfx & ((1ull << (3 * a.d)) - 1)) : 0u;
      a.cx = compact3(cell); a.cy = compact3(cell >> 1); a.cz = compact3(cell >> 2);
      a.sidx = s.t.pt_begin[v] + (k - s.off(cl));
      return a;
    }
    // Whether points [k0, k1) all lie in the cached node: then the addresses
    // and the cell are the same for every lane (scalar registers, one vector
    // offset) and fetch_run reads the whole batch with fetch's results.
    __device__ __forceinline__ bool run_inside(uint64_t k0, uint64_t k1) const {
      const uint64_t end = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(oe >> 32)) << 32) |
                           __builtin_amdgcn_readfirstlane((uint32_t)oe);
      return k1 <= end;
    }
    template <int R>
    __device__ __forceinline__ void fetch_run(const TreeSrcT &s, uint64_t k0, float (&px)[R], float (&py)[R],
                                              float (&pz)[R], float (&pm)[R]) const {
      const uint32_t lane = threadIdx.x & (WAVE - 1);
      const uint64_t first = pb + (k0 - ob);
      const uint64_t base = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(first >> 32)) << 32) |
                            __builtin_amdgcn_readfirstlane((uint32_t)first);
      const int du = __builtin_amdgcn_readfirstlane(d);
      const uint32_t ux = __builtin_amdgcn_readfirstlane(cx), uy = __builtin_amdgcn_readfirstlane(cy),
                     uz = __builtin_amdgcn_readfirstlane(cz);
      const uint16_t *ax = s.t.qx + base, *ay = s.t.qy + base, *az = s.t.qz + base;
      const float *am = s.t.pt_mass + base;
      uint32_t qx[R], qy[R], qz[R];
      int dx[R], dy[R], dz[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t o = (uint32_t)r * WAVE + lane;
        qx[r] = ax[o]; qy[r] = ay[o]; qz[r] = az[o]; pm[r] = am[o];
        if constexpr (MOTION) {
          dx[r] = (s.dqx + base)[o]; dy[r] = (s.dqy + base)[o]; dz[r] = (s.dqz + base)[o];
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        px[r] = decode_coord(ux, qx[r], du);
        py[r] = decode_coord(uy, qy[r], du);
        pz[r] = decode_coord(uz, qz[r], du);
        if constexpr (MOTION) {
          px[r] = lerp_t(px[r], decode_motion(ux, qx[r], dx[r], du), s.t_frame);
          py[r] = lerp_t(py[r], decode_motion(uy, qy[r], dy[r], du), s.t_frame);
          pz[r] = lerp_t(pz[r], decode_motion(uz, qz[r], dz[r], du), s.t_frame);
        }
      }
    }
    // move the cached node to the furthest node any lane reached
    __device__ void end_round(const TreeSrcT &s) {
      if (!__ballot(far_c != c)) return;      // every lane stayed in the cached node
      uint64_t f = far_c;
#pragma unroll
      for (int o = 1; o < WAVE; o <<= 1) f = max(f, (uint64_t)__shfl_xor(f, o, WAVE));
      if (f != c) set(s, f);
    }
    __device__ __forceinline__ void fetch(const TreeSrcT &s, const Addr &a, bool, float &px, float &py,
                                          float &pz, float &pm) const {
      const uint32_t qx = s.t.qx[a.sidx], qy = s.t.qy[a.sidx], qz = s.t.qz[a.sidx];
      pm = s.t.pt_mass[a.sidx];
      if constexpr (MOTION) {
        // the point at frame time t between its decoded position and the
        // position its motion code decodes to
        const int dx = s.dqx[a.sidx], dy = s.dqy[a.sidx], dz = s.dqz[a.sidx];
        px = lerp_t(decode_coord(a.cx, qx, a.d), decode_motion(a.cx, qx, dx, a.d), s.t_frame);
        py = lerp_t(decode_coord(a.cy, qy, a.d), decode_motion(a.cy, qy, dy, a.d), s.t_frame);
        pz = lerp_t(decode_coord(a.cz, qz, a.d), decode_motion(a.cz, qz, dz, a.d), s.t_frame);
      } else {
        px = decode_coord(a.cx, qx, a.d);
        py = decode_coord(a.cy, qy, a.d);
        pz = decode_coord(a.cz, qz, a.d);
      }
    }
    __device__ __forceinline__ float wradius(const TreeSrcT &, const Addr &) const { return 0.0f; }
    // 1 when the stored point's highlight flag is set, else 0
    __device__ __forceinline__ float attr(const TreeSrcT &s, const Addr &a) const {
      return s.hl_test(a.sidx, s.hl_word(a.sidx)) ? 1.0f : 0.0f;
    }
    __device__ __forceinline__ uint64_t point_index(const TreeSrcT &, const Addr &a) const { return a.sidx; }
  };
  __device__ uint64_t count() const { return *total; }
  const uint32_t *hl_flags = nullptr;  // highlight flags, one bit per stored point
  uint64_t hl_words = 1;
  const int16_t *dqx = nullptr, *dqy = nullptr, *dqz = nullptr;   // motion codes (MOTION)
  float t_frame = 0.0f;
  // the flag word of stored point s (in bounds for any s) and its flag
  __device__ __forceinline__ uint32_t hl_word(uint64_t sidx) const {
    return hl_flags[min(sidx >> 5, hl_words - 1)];
  }
  __device__ __forceinline__ bool hl_test(uint64_t sidx, uint32_t word) const {
    return (word >> (uint32_t)(sidx & 31u)) & 1u;
  }
};
using TreeSrc = TreeSrcT<false>;
using TreeMotionSrc = TreeSrcT<true>;
template <class S> struct IsTree { static constexpr bool value = false; };
template <bool M> struct IsTree<TreeSrcT<M>> { static constexpr bool value = true; };

// One point's screen position, pixel radius (cubic blob), attribute and tile
// rectangle (ntx = nty = 0: not drawn).
struct Blob {
  float u, v, m, h, a;
  int tx0, ty0, ntx, nty;
};

// Pair records of the binned (point, tile) pairs, one type per render form:
// Gaussian (u, v, m) is float3; the others carry the attribute and / or the
// cubic blob's pixel radius.
struct RecGA { float u, v, m, a; };        // Gaussian + attribute
struct RecC { float u, v, m, h; };         // cubic
struct RecCA { float u, v, m, h, a; };     // cubic + attribute
__device__ __forceinline__ void rec_put(float3 *r, uint64_t i, const Blob &b) { r[i] = make_float3(b.u, b.v, b.m); }
__device__ __forceinline__ void rec_put(RecGA *r, uint64_t i, const Blob &b) { r[i] = RecGA{b.u, b.v, b.m, b.a}; }
__device__ __forceinline__ void rec_put(RecC *r, uint64_t i, const Blob &b) { r[i] = RecC{b.u, b.v, b.m, b.h}; }
__device__ __forceinline__ void rec_put(RecCA *r, uint64_t i, const Blob &b) { r[i] = RecCA{b.u, b.v, b.m, b.h, b.a}; }
template <class R> struct RecInfo { static constexpr bool aux = false; static constexpr bool cubic = false; };
template <> struct RecInfo<RecGA> { static constexpr bool aux = true; static constexpr bool cubic = false; };
template <> struct RecInfo<RecC> { static constexpr bool aux = false; static constexpr bool cubic = true; };
template <> struct RecInfo<RecCA> { static constexpr bool aux = true; static constexpr bool cubic = true; };

// Pixels [lo, hi] (clipped to [0, size)) that contain every pixel a blob at
// screen coordinate t can cover: the float32 offset test |t - (i + 1/2)| <= R
// is decided to within 2^-8 for |t| < 2^15 (the camera limits), so a margin
// of 1/100 pixel makes the range conservative.  A tile this admits without a
// covered pixel only adds a pair whose rows are zero in the accumulation.
__device__ __forceinline__ bool cover_range(float R, float t, uint32_t size, int &lo, int &hi) {
  const float reach = R + 0.01f;
  const float a = fmaxf(ceilf(t - 0.5f - reach), 0.0f);
  const float b = fminf(floorf(t - 0.5f + reach), (float)(int)(size - 1));
  // clamped first: a coordinate far outside gives a > b (a NaN fails t == t)
  if (!(a <= b && t == t)) return false;
  lo = (int)a;
  hi = (int)b;
  return true;
}

// Pixel radius of a cubic blob at camera depth zc: the fixed radius, or the
// projected world radius fl(fl(F h_world) / zc) clamped to [1, 16] pixels.
// A per-point world radius hw > 0 replaces the camera's.
__device__ __forceinline__ float cubic_radius(const Cam &c, float zc, float hw = 0.0f) {
  const float Fhw = hw > 0.0f ? c.F * hw : c.Fhw;
  if (Fhw > 0.0f) return fminf(fmaxf(__fdiv_rn(Fhw, zc), lodh::BLOB_H_MIN), lodh::BLOB_H_MAX);
  return c.hpx;
}

__device__ __forceinline__ Blob make_blob(const Cam &c, bool valid, float px, float py, float pz, float pm,
                                          float pa = 0.0f, float hw = 0.0f) {
  Blob b{0.0f, 0.0f, pm, 0.0f, pa, 0, 0, 0, 0};
  if (!valid) return b;
  float xc, yc, zc;
  if (!project(c, px, py, pz, b.u, b.v, xc, yc, zc)) return b;
  const float R = c.blob == LOD_BLOB_CUBIC ? cubic_radius(c, zc, hw) : c.R;
  b.h = R;
  int i0, i1, j0, j1;
  if (!cover_range(R, b.u, c.W, i0, i1) || !cover_range(R, b.v, c.H, j0, j1)) return b;
  b.tx0 = i0 / TS; b.ty0 = j0 / TS;
  b.ntx = i1 / TS - b.tx0 + 1;
  b.nty = j1 / TS - b.ty0 + 1;
  return b;
}

// OR of a value over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast 15, 31
  v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, WAVE - 1);
}

// Largest value over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, WAVE - 1);
}

__device__ __forceinline__ uint32_t rank_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// One lane's writes to a table that another lane of the same wave reads.
__device__ __forceinline__ void wave_sync_mem() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A unit's per-tile counters (pass 1) or list cursors (pass 2), private to its
// wave.  LdsTab: in LDS, for rounds that touch tiles all over the image (every
// round of points in random order).  RowTab: the unit's own row of the count
// table in global memory, touched when a window is opened or closed; no LDS,
// so as many waves run as registers allow, and no row-sized initialisation of
// LDS.  get / put are a lane's own element.
template <class CT>
struct LdsTab {
  static constexpr bool adds = true;
  CT *lc;
  __device__ __forceinline__ uint32_t get(uint32_t t) const { return (uint32_t)lc[t]; }
  __device__ __forceinline__ void put(uint32_t t, uint32_t v) const { lc[t] = (CT)v; }
  // counts only: lanes may add to one tile at a time (16-bit counters are
  // added in their 32-bit word; a unit's counts stay below 2^16, so no carry
  // crosses the halves)
  __device__ __forceinline__ void add(uint32_t t) const {
    if constexpr (sizeof(CT) == 2) atomicAdd(reinterpret_cast<uint32_t *>(lc) + (t >> 1), 1u << (16 * (t & 1u)));
    else atomicAdd(&lc[t], 1u);
  }
};
struct RowTab {
  static constexpr bool adds = false;
  uint32_t *row;
  const uint32_t *off, *pre;     // added to what is read (list starts of the tile and the chunk), or null
  __device__ __forceinline__ uint32_t base(uint32_t t) const { return (off ? off[t] : 0u) + (pre ? pre[t] : 0u); }
  __device__ __forceinline__ uint32_t get(uint32_t t) const { return row[t] + base(t); }
  __device__ __forceinline__ void put(uint32_t t, uint32_t v) const { row[t] = v - base(t); }
};

// The counters of an 8x8 tile window, one per lane.
template <class Tab>
struct TileWin {
  int wx = -(1 << 20), wy = 0;   // closed: no point lies in it
  uint32_t cur = 0, tile = 0;
  bool inside = false;           // this lane's tile lies in the image
  __device__ __forceinline__ bool open() const { return wx >= 0; }
  __device__ __forceinline__ void load(const Tab &tab, const Cam &c, int x, int y) {
    const int lane = threadIdx.x & (WAVE - 1);
    wx = x; wy = y;
    const int tx = wx + lane % WINT, ty = wy + lane / WINT;
    inside = tx < (int)c.tiles_x && ty < (int)c.tiles_y;
    tile = inside ? (uint32_t)(ty * (int)c.tiles_x + tx) : 0u;
    cur = inside ? tab.get(tile) : 0u;
  }
  __device__ __forceinline__ void close(const Tab &tab) {
    if (!open()) return;
    if (inside) tab.put(tile, cur);
    wx = -(1 << 20);
    wave_sync_mem();
  }
};

// The pairs of one round whose points do not fit one window, tile index by
// tile index within the point.  Counting in LDS adds lane by lane.  Otherwise
// a ballot per tile bit groups and ranks the lanes of one tile, and the
// lowest of them moves the tile's counter.
template <bool FILL, class Tab, class RecT>
__device__ __forceinline__ void emit_spread(const Blob &bl, const Cam &c, int nbits, const Tab &tab,
                                            RecT *__restrict__ rec) {
  const int lane = threadIdx.x & (WAVE - 1);
  for (int dy = 0; __ballot(dy < bl.nty); ++dy) {
    for (int dx = 0; __ballot(dy < bl.nty && dx < bl.ntx); ++dx) {
      const bool has = dy < bl.nty && dx < bl.ntx;
      const uint32_t t = has ? (uint32_t)((bl.ty0 + dy) * (int)c.tiles_x + bl.tx0 + dx) : 0u;
      if constexpr (!FILL && Tab::adds) {
        if (has) tab.add(t);
      } else {
        uint64_t peers = __ballot(has);
        for (int b = 0; b < nbits; ++b) {
          const uint64_t bal = __ballot((t >> b) & 1u);
          peers &= ((t >> b) & 1u) ? bal : ~bal;
        }
        const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (WAVE - lane));
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        const uint32_t old = has ? tab.get(t) : 0u;
        wave_sync_mem();
        if (has && below == 0) tab.put(t, old + (uint32_t)__popcll(peers));
        wave_sync_mem();
        if (FILL && has) rec_put(rec, old + below, bl);
      }
    }
  }
  wave_sync_mem();
}

// The pairs of one round of 64 points (each at most 8 tiles wide and high).
template <bool FILL, class Tab, class RecT>
__device__ __forceinline__ void emit_round(const Blob &bl, const Cam &c, int nbits, const Tab &tab,
                                           TileWin<Tab> &win, RecT *__restrict__ rec) {
  const int lane = threadIdx.x & (WAVE - 1);
  const bool drawn = bl.ntx > 0;
  const uint64_t live = __ballot(drawn);
  if (!live) return;
  auto fits = [&]() {
    return drawn && (uint32_t)(bl.tx0 - win.wx) <= (uint32_t)(WINT - bl.ntx) &&
           (uint32_t)(bl.ty0 - win.wy) <= (uint32_t)(WINT - bl.nty);
  };
  if (__ballot(fits()) != live) {
    // a new window around the round's tiles, if one holds them all (a
    // property of the round alone, and with it the order of its pairs)
    win.close(tab);
    const uint32_t big = 1u << 20;
    const int x1 = (int)wave_max(drawn ? (uint32_t)(bl.tx0 + bl.ntx) : 0u);
    const int y1 = (int)wave_max(drawn ? (uint32_t)(bl.ty0 + bl.nty) : 0u);
    const int x0 = (int)(big - wave_max(drawn ? big - (uint32_t)bl.tx0 : 0u));
    const int y0 = (int)(big - wave_max(drawn ? big - (uint32_t)bl.ty0 : 0u));
    if (x1 - x0 > WINT || y1 - y0 > WINT) {
      emit_spread<FILL, Tab, RecT>(bl, c, nbits, tab, rec);
      return;
    }
    // the round's tiles in the middle of it
    const int x = max(x0 - (WINT - (x1 - x0)) / 2, 0), y = max(y0 - (WINT - (y1 - y0)) / 2, 0);
    win.load(tab, c, x, y);
  }
  // the point's cells: its columns in every row, its rows
  uint32_t mlo = 0, mhi = 0;
  if (drawn) {
    const uint32_t cols = ((1u << bl.ntx) - 1u) << (bl.tx0 - win.wx);
    const uint32_t cols4 = __builtin_amdgcn_perm(cols, cols, 0u);   // byte 0 in all four bytes
    const uint64_t rows = (~0ull >> (64 - 8 * bl.nty)) << (8 * (bl.ty0 - win.wy));
    mlo = cols4 & (uint32_t)rows;
    mhi = cols4 & (uint32_t)(rows >> 32);
  }
  auto cells_of = [&](uint32_t word, uint32_t m, int first) {
    while (word) {
      const int b = __builtin_ctz(word);
      word &= word - 1u;
      const bool mine = (m & (1u << b)) != 0u;
      const uint64_t grp = __ballot(mine);
      const int cell = first + b;
      if constexpr (FILL) {
        const uint32_t old = (uint32_t)__builtin_amdgcn_readlane((int)win.cur, cell);
        if (mine) rec_put(rec, old + rank_below(grp), bl);
      }
      if (lane == cell) win.cur += (uint32_t)__popcll(grp);
    }
  };
  cells_of(wave_or(mlo), mlo, 0);
  cells_of(wave_or(mhi), mhi, 32);
}

// Highlight staging: the count pass writes the decoded points whose id is
// selected to x, y, z, m at [b, b + k) of its unit's point range [b, e)
// (sequence order), and k to count[unit].
struct HlStage {
  float *x, *y, *z, *m;
  uint64_t *count, *scan;   // per unit (scan: a copy, scanned afterwards)
};

// Points per unit of a partition of n points: whole rounds.
__device__ __forceinline__ uint64_t unit_points(uint64_t n, uint32_t units) {
  const uint64_t rounds = (n + WAVE - 1) / WAVE;
  return (rounds + units - 1) / units * WAVE;
}

// The pairs of points [u0 per, min(n, (u0 + g) per)): g consecutive units.
// Returns the points staged (HL).
template <class Src, bool FILL, class Tab, class RecT, bool HL = false>
__device__ __forceinline__ uint32_t bin_unit(const Src &src, const Cam &c, uint32_t units, uint32_t u0, uint32_t g,
                                             int nbits, const Tab &tab, RecT *__restrict__ rec,
                                             HlStage hs = HlStage{}) {
  const int lane = threadIdx.x;
  const uint64_t n = src.count();
  const uint64_t per = unit_points(n, units);
  const uint64_t b = (uint64_t)u0 * per, e = min(n, b + (uint64_t)g * per);
  uint32_t staged = 0;
  if (b >= e) return 0;
  typename Src::Cursor cur;
  cur.begin(src, b, e);
  TileWin<Tab> win;
  constexpr int R = FILL ? BR_FILL : BR;
  for (uint64_t k0 = b; k0 < e; k0 += (uint64_t)R * WAVE) {
    float px[R], py[R], pz[R], pm[R], pa[R], ph[R];
    uint64_t pid[HL ? R : 1];
    bool whole = false;
    if constexpr (IsTree<Src>::value) {
      whole = k0 + (uint64_t)R * WAVE <= e && cur.run_inside(k0, k0 + (uint64_t)R * WAVE);
      if (whole) {
        cur.template fetch_run<R>(src, k0, px, py, pz, pm);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          pa[r] = ph[r] = 0.0f;
          if (HL) pid[r] = cur.pb + (k0 + (uint64_t)r * WAVE + lane - cur.ob);
        }
      }
    }
    if (!whole) {
      typename Src::Addr ad[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint64_t k = k0 + (uint64_t)r * WAVE + lane;
        ad[r] = cur.resolve(src, k, k < e);
        cur.end_round(src);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint64_t k = k0 + (uint64_t)r * WAVE + lane;
        cur.fetch(src, ad[r], k < e, px[r], py[r], pz[r], pm[r]);
        pa[r] = (FILL && RecInfo<RecT>::aux) ? cur.attr(src, ad[r]) : 0.0f;
        ph[r] = c.blob == LOD_BLOB_CUBIC ? cur.wradius(src, ad[r]) : 0.0f;
        if constexpr (HL) pid[r] = cur.point_index(src, ad[r]);
      }
    }
    if constexpr (HL) {
      // ID highlighting: the flag test of every drawn point, and the
      // flagged ones staged in sequence order (wave ballot ranks).  A wave's
      // points are mostly consecutive stored points, so its flag loads fall
      // on one or two words.
      uint32_t word[R];
#pragma unroll
      for (int r = 0; r < R; ++r) word[r] = src.hl_word(pid[r]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool in = k0 + (uint64_t)r * WAVE + lane < e && src.hl_test(pid[r], word[r]);
        const uint64_t mask = __ballot(in);
        if (in) {
          const uint64_t o = b + staged + rank_below(mask);
          hs.x[o] = px[r]; hs.y[o] = py[r]; hs.z[o] = pz[r]; hs.m[o] = pm[r];
        }
        staged += (uint32_t)__popcll(mask);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const Blob bl = make_blob(c, k0 + (uint64_t)r * WAVE + lane < e, px[r], py[r], pz[r], pm[r], pa[r], ph[r]);
      emit_round<FILL, Tab, RecT>(bl, c, nbits, tab, win, rec);
    }
  }
  win.close(tab);
  return staged;
}

// Pass 1: row u of the [U][tiles] count table.  CT = uint16_t when a unit
// holds at most 65535 points (a point adds at most one pair per tile), which
// halves the LDS per wave and doubles the resident waves; CT = void: counted
// in the row itself.
template <class Src, class CT, bool HL = false>
__global__ __launch_bounds__(BW) void k_bin_count(Src src, Cam c, uint32_t units, int nbits, uint32_t *ucount,
                                                  HlStage hs = HlStage{}) {
  extern __shared__ uint32_t lds_raw[];
  const uint32_t nt = c.tiles_x * c.tiles_y;
  uint32_t *row = ucount + (uint64_t)blockIdx.x * nt;
  uint32_t staged;
  if constexpr (std::is_void<CT>::value) {
    for (uint32_t i = threadIdx.x; i < nt; i += BW) row[i] = 0u;
    wave_sync_mem();
    staged = bin_unit<Src, false, RowTab, float3, HL>(src, c, units, blockIdx.x, 1, nbits,
                                                      RowTab{row, nullptr, nullptr}, (float3 *)nullptr, hs);
  } else {
    CT *lc = reinterpret_cast<CT *>(lds_raw);
    for (uint32_t i = threadIdx.x; i < nt; i += BW) lc[i] = 0;
    __syncthreads();
    staged = bin_unit<Src, false, LdsTab<CT>, float3, HL>(src, c, units, blockIdx.x, 1, nbits, LdsTab<CT>{lc},
                                                          (float3 *)nullptr, hs);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nt; i += BW) row[i] = lc[i];
  }
  if (HL && threadIdx.x == 0) { hs.count[blockIdx.x] = staged; hs.scan[blockIdx.x] = staged; }
}

// Gather the staged highlighted points into one array in unit order: unit u
// holds count[u] points at [u per, ...) of the staging arrays and goes to
// [off[u], ...) (off = exclusive scan of the counts, off[units] = total).
// At most cap points are kept; more sets the capacity status bit.
__global__ void k_hl_gather(HlStage hs, const uint64_t *__restrict__ off, const uint64_t *__restrict__ n_points,
                            uint64_t max_points, uint32_t units, float *__restrict__ x, float *__restrict__ y,
                            float *__restrict__ z, float *__restrict__ m, uint64_t cap,
                            uint64_t *__restrict__ total, uint64_t *status) {
  const uint64_t n = min(*n_points, max_points);
  const uint64_t per = unit_points(n, units);
  const uint32_t u = blockIdx.x;
  const uint64_t b = (uint64_t)u * per, o = off[u], k = hs.count[u];
  for (uint64_t j = threadIdx.x; j < k && o + j < cap; j += blockDim.x) {
    x[o + j] = hs.x[b + j]; y[o + j] = hs.y[b + j]; z[o + j] = hs.z[b + j]; m[o + j] = hs.m[b + j];
  }
  if (u == 0 && threadIdx.x == 0) {
    const uint64_t tot = off[units];
    *total = min(tot, cap);
    if (tot > cap) atomicOr((unsigned long long *)status, (unsigned long long)LOD_STATUS_CAPACITY);
  }
}

// Highlight flags of the stored points: bit s of flags (uint32 words) is set
// when the id of stored point s has its bit in the id bitset (ids >= n_bits
// are not selected).  One wave codes 64 consecutive points, two words.
__global__ void k_hl_flags(const lod_tree t, const uint32_t *__restrict__ bits, uint64_t n_bits,
                           uint64_t cap_points, uint32_t *__restrict__ flags) {
  const uint64_t np = min(t.counts[1], cap_points);
  const uint64_t nwords = (n_bits + 31) >> 5;
  const uint64_t nw = (cap_points + 63) >> 6;     // wave groups of 64 points
  const int lane = threadIdx.x & (WAVE - 1);
  for (uint64_t g = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; g < nw;
       g += ((uint64_t)gridDim.x * blockDim.x) >> 6) {
    const uint64_t sidx = g * 64 + lane;
    bool on = false;
    if (sidx < np) {
      const uint32_t id = t.pt_id[sidx];
      const uint32_t w = bits[min((uint64_t)(id >> 5), nwords - 1)];
      on = (uint64_t)id < n_bits && ((w >> (id & 31u)) & 1u);
    }
    const uint64_t mask = __ballot(on);
    if (lane == 0) reinterpret_cast<uint2 *>(flags)[g] = make_uint2((uint32_t)mask, (uint32_t)(mask >> 32));
  }
}

// Column scans of the count table: exclusive prefix over the 64 units of each
// chunk (in place) and the chunk totals.  A column is a chain of dependent
// adds but not of loads: sixteen rows are loaded together.
__global__ void k_bin_colscan(uint32_t *__restrict__ ucount, uint32_t nt, uint32_t *__restrict__ pchunk) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t ch = blockIdx.y;
  if (t >= nt) return;
  uint32_t run = 0;
  for (uint32_t u = ch * 64; u < ch * 64 + 64; u += 16) {
    uint32_t v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = ucount[(uint64_t)(u + k) * nt + t];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      ucount[(uint64_t)(u + k) * nt + t] = run;
      run += v[k];
    }
  }
  pchunk[(uint64_t)ch * nt + t] = run;
}

// Exclusive prefix of one tile's counts over the chunks (in place); returns the
// tile's total.
__device__ __forceinline__ uint32_t scan_chunks(uint32_t *__restrict__ pchunk, uint32_t nt, uint32_t chunks,
                                                uint32_t t) {
  uint32_t run = 0;
  for (uint32_t c0 = 0; c0 < chunks; c0 += 16) {
    uint32_t v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = pchunk[(uint64_t)min(c0 + k, chunks - 1) * nt + t];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (c0 + k < chunks) {
        pchunk[(uint64_t)(c0 + k) * nt + t] = run;
        run += v[k];
      }
  }
  return run;
}

__global__ void k_bin_chunkscan(uint32_t *__restrict__ pchunk, uint32_t nt, uint32_t chunks,
                                uint32_t *__restrict__ tile_count) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nt) tile_count[t] = scan_chunks(pchunk, nt, chunks, t);
}

// log2 of the pairs of a slice (a block's share of a tile's list) when `pairs`
// pairs are drawn: a function of the image's input alone, not of the sizes that
// the workspace was planned for, because the order of the float64 sums depends
// on it.
// Long slices of dense tiles end last and leave CUs idle; short ones add
// partial tiles and sums, and a cubic slice takes longer.  Accumulation and
// final sums in us at slices of 512, 1024, 2048 and 4096:
//   Gaussian, 256^2, clumps    2^19 pairs 17.5 19.2 22.2 25.9
//             (1024^2)         2^20  23.5 22.4 26.6 32.6   (41.6 39.7 42.7 49.4)
//                              2^22  56.3 49.0 49.2 56.0   (75.4 68.6 67.8 76.2)
//                              2^23  100 86 80 83          (117 103 101 107)
//                              2^25  346 291 278 265       (336 299 289 289)
//                              2^27  1379 1190 1081 1048   (1262 1128 1060 1024)
//   cubic, h = 2.5, 1024^2,    2^19  73 96 118 168         (68 66 67 66)
//          clumps (uniform)    2^21  156 175 220 266       (144 138 138 139)
//                              2^22  267 275 313 381       (263 248 245 245)
//                              2^23  473 474 496 561       (493 476 457 458)
//                              2^26  3409 3379 3360 3338   (3544 3455 3665 3668)
__host__ __device__ inline uint32_t slice_bits(uint32_t pairs, bool cubic) {
  if (cubic) return pairs <= 1u << 21 ? 9 : pairs <= 1u << 26 ? 10 : 12;
  return pairs <= 1u << 19 ? 9 : pairs <= 1u << 22 ? 10 : pairs <= 1u << 25 ? 11 : 12;
}

__device__ __forceinline__ uint32_t slices_of(uint32_t pairs, uint32_t bits) {
  return (pairs + (1u << bits) - 1u) >> bits;
}

// Offsets of the tiles' pair lists and of their slices (exclusive, with the
// totals at [nt]), and a cleared status word: one block, since there are at
// most 8192 tiles.  tile_count null: no points.  pchunk not null: at most PLAN_T
// tiles, whose chunk scans this block does, a thread each (its reads take as
// long as the launch that they replace only at 64 chunks).
constexpr int PLAN_T = 1024;
constexpr int PLAN_ITEMS = lodh::SPLAT_MAX_TILES / PLAN_T;
__global__ __launch_bounds__(PLAN_T) void k_tile_plan(const uint32_t *__restrict__ tile_count,
                                                      uint32_t *__restrict__ pchunk, uint32_t chunks, uint32_t nt,
                                                      int cubic,
                                                      uint32_t *__restrict__ tile_off,
                                                      uint32_t *__restrict__ slice_off, uint64_t *clear_status) {
  __shared__ uint32_t tmp[PLAN_T / WAVE + 1];
  const uint32_t per = (nt + PLAN_T - 1) / PLAN_T;   // tiles per thread (at most PLAN_ITEMS)
  const uint32_t t0 = threadIdx.x * per;
  uint32_t cnt[PLAN_ITEMS], pairs = 0, slices = 0;
  const uint32_t scanned = pchunk && threadIdx.x < nt ? scan_chunks(pchunk, nt, chunks, threadIdx.x) : 0u;
#pragma unroll
  for (int k = 0; k < PLAN_ITEMS; ++k)
    cnt[k] = pchunk ? (k ? 0u : scanned)
                    : (tile_count && (uint32_t)k < per && t0 + k < nt) ? tile_count[t0 + k] : 0u;
#pragma unroll
  for (int k = 0; k < PLAN_ITEMS; ++k) pairs += cnt[k];
  uint32_t tp, ts;
  uint32_t p = block_excl_scan<uint32_t>(pairs, tmp, tp);
  const uint32_t bits = slice_bits(tp, cubic);
#pragma unroll
  for (int k = 0; k < PLAN_ITEMS; ++k) slices += slices_of(cnt[k], bits);
  uint32_t q = block_excl_scan<uint32_t>(slices, tmp, ts);
#pragma unroll
  for (int k = 0; k < PLAN_ITEMS; ++k) {
    if ((uint32_t)k < per && t0 + k < nt) { tile_off[t0 + k] = p; slice_off[t0 + k] = q; }
    p += cnt[k];
    q += slices_of(cnt[k], bits);
  }
  if (threadIdx.x == 0) {
    tile_off[nt] = tp;
    slice_off[nt] = ts;
    if (clear_status) *clear_status = 0;
  }
}

// Pass 2: write the records.  Block f covers the g consecutive units f g ..
// f g + g - 1 (a tile's list holds their pairs in unit order, so one cursor per
// tile carries over from one unit to the next); its cursor for tile t starts
// at tile_off[t] + (pairs of earlier chunks) + (pairs of earlier units in its
// chunk).  LDS: the cursors are kept in LDS, else in the unit's row of the
// count table (g = 1).  The pair count (tile_off[nt]) is checked against the
// record capacity once: past it nothing is written and the status word says
// so.  The blocks also write the slice descriptors, (first pair,
// tile | pairs << 16), one per slice, a lane per tile.
template <class Src, class RecT, bool LDS>
__global__ __launch_bounds__(BW) void k_bin_fill(Src src, Cam c, uint32_t units, uint32_t g, int nbits,
                                                 uint32_t *ucount, const uint32_t *__restrict__ pchunk,
                                                 const uint32_t *__restrict__ tile_off,
                                                 const uint32_t *__restrict__ slice_off,
                                                 uint2 *__restrict__ table, uint64_t max_slices, RecT *__restrict__ rec, uint64_t max_pairs,
                                                 uint64_t *status) {
  extern __shared__ uint32_t lc[];
  const uint32_t nt = c.tiles_x * c.tiles_y;
  const uint32_t slice = 1u << slice_bits(tile_off[nt], RecInfo<RecT>::cubic);
  for (uint32_t t = blockIdx.x * BW + threadIdx.x; t < nt; t += gridDim.x * BW) {
    const uint32_t b = slice_off[t], e = slice_off[t + 1];
    const uint32_t p = tile_off[t], cnt = tile_off[t + 1] - p;
    for (uint32_t k = 0; b + k < e && b + k < max_slices; ++k)
      table[b + k] = make_uint2(p + k * slice, t | (min(cnt - k * slice, slice) << 16));
  }
  if (tile_off[nt] > max_pairs) {
    if (threadIdx.x == 0) atomicOr((unsigned long long *)status, (unsigned long long)LOD_STATUS_CAPACITY);
    return;
  }
  const uint32_t u0 = blockIdx.x * g;
  const uint32_t *pre = pchunk ? pchunk + (uint64_t)(u0 / 64) * nt : nullptr;   // null: one chunk
  uint32_t *row = ucount + (uint64_t)u0 * nt;
  if constexpr (LDS) {
    for (uint32_t i = threadIdx.x; i < nt; i += BW) lc[i] = tile_off[i] + (pre ? pre[i] : 0u) + row[i];
    __syncthreads();
    bin_unit<Src, true, LdsTab<uint32_t>, RecT>(src, c, units, u0, g, nbits, LdsTab<uint32_t>{lc}, rec);
  } else {
    bin_unit<Src, true, RowTab, RecT>(src, c, units, u0, g, nbits, RowTab{row, tile_off, pre}, rec);
  }
}

// --- accumulation --------------------------------------------------------------

// One block per slice.  The blob is separable, so a chunk of 64 points adds
// Gy^T Gx to the 16x16 tile, with Gx[k][i] = exp(-ox^2/2s^2) and Gy[k][j] =
// m norm exp(-oy^2/2s^2) inside point k's truncation square and 0 outside.
// A wave forms its points' rows in LDS, one point per lane, reads them back as
// the operands of 16 MFMA steps (16x16x4, float32) and adds the products (64
// per pixel) to float64 sums, four pixels per lane; at the end of the slice the
// four wave sums of each pixel are added in wave order.  A wave reads only rows
// that its own lanes wrote, and the LDS operations of one wave complete in
// order, so the waves of a block run their chunks without block barriers.  No
// atomics: the image is bit-reproducible.
//
// Narrow blobs (k_accumulate_narrow) cover at most nine pixels per axis; wider
// ones fill whole rows (k_accumulate_wide).
// Pair record loads (the attribute of records that carry none is 0).
__device__ __forceinline__ void load_rec(const float3 *r, uint64_t q, float &u, float &v, float &m, float &a) {
  const float3 t = r[q];
  u = t.x; v = t.y; m = t.z; a = 0.0f;
}
__device__ __forceinline__ void load_rec(const RecGA *r, uint64_t q, float &u, float &v, float &m, float &a) {
  const float4 t = reinterpret_cast<const float4 *>(r)[q];
  u = t.x; v = t.y; m = t.z; a = t.w;
}

typedef float float4v __attribute__((ext_vector_type(4)));

// The slices of a block and their records, loaded one chunk ahead across slice
// boundaries (clamped indices: every load is issued unconditionally).  Pair
// indices are 32-bit.
template <class RecT>
struct SliceWalk {
  const uint2 *table;
  const RecT *rec;
  uint32_t last, total, sl;
  uint2 sd, nsd;
  float nu, nv, nm, na = 0.0f;
  __device__ __forceinline__ void begin(const uint2 *tb, const RecT *r, uint32_t n, uint64_t max_pairs) {
    table = tb; rec = r; total = n; last = (uint32_t)(max_pairs - 1);
    sl = blockIdx.x;
    sd = table[sl];
    load_rec(rec, min(sd.x + threadIdx.x, last), nu, nv, nm, na);
    peek();
  }
  __device__ __forceinline__ void peek() { nsd = table[min(sl + gridDim.x, total - 1)]; }
  // records of the slice (all inside the record array)
  __device__ __forceinline__ uint32_t count() const { return min(sd.y >> 16, last - sd.x + 1u); }
  // this thread's record of the chunk at offset o (0 past the slice's n), and the next load
  __device__ __forceinline__ void take(uint32_t o, uint32_t n, float &u, float &v, float &m, float &a) {
    const bool have = o + threadIdx.x < n;
    u = have ? nu : 0.0f; v = have ? nv : 0.0f; m = have ? nm : 0.0f; a = have ? na : 0.0f;
    const uint32_t next = o + PT < n ? sd.x + o + PT : nsd.x;
    load_rec(rec, min(next + threadIdx.x, last), nu, nv, nm, na);
  }
  __device__ __forceinline__ void next() {
    sl += gridDim.x;
    sd = nsd;
    peek();
  }
};

// Value of lane `from` of each row of 16 lanes, in all lanes of the row.
template <int FROM>
__device__ __forceinline__ uint32_t row_bcast(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + FROM, 0xF, 0xF, true);
}

// A row value times its point's attribute; 0 where the blob does not reach the
// row, also for an attribute that is infinite or NaN.
__device__ __forceinline__ float times_attr(float row, float at) { return row != 0.0f ? row * at : 0.0f; }

// Calls f(integral_constant<int, 0>) .. f(integral_constant<int, 15>).
template <class F, int... T>
__device__ __forceinline__ void for_16(F f, std::integer_sequence<int, T...>) {
  (f(std::integral_constant<int, T>{}), ...);
}

// Narrow blobs: radius below 3.98 pixels.  A pixel's Gaussian is one hardware
// exponential of its own offset; only the pixels between nin and nmax steps
// away from the one that holds the point need the truncation test.  (A chain
// of products from pixel to pixel, three exponentials per axis, draws 150 M
// points in 1.89 ms where this takes 2.03, but carries a rounding of the
// exponential per step: 1.2 to 1.4 times the error of an axis at sigma 0.5 to
// 1, 2.1 times at 2 and 4.4 times at 8.)  The mass takes only the power of two
// in the normalisation; the rest multiplies the float64 sums.
//
// A point's window of up to nine values goes to the same columns of its row,
// 0 .. 2 nmax, with 16 zeros on either side that nothing overwrites, so
// that the writes have no bank conflicts and nothing is cleared between
// chunks; the reader of pixel p of point k starts p - (window origin) further
// on, an address that one lane-broadcast add gives (lane l holds point l; the
// points 16 r .. 16 r + 15 are the r-th operands of the 16 steps).  x rows are
// read before y rows overwrite them, which halves the LDS per wave.
//
// Bound by vector issue beside the matrix steps (a chunk of 64 points: about
// 170 vector instructions, 14 of them exponentials, and 16 matrix steps of 32
// cycles).  150 M points drawn at 1024^2, 285 M pairs: 2.31 -> 2.03 ms against a
// form that cleared and wrote 8-wide windows at varying columns (LDS bank
// conflicts half of the LDS time, 16 exponentials per point, four waves per
// SIMD; now six).  Error against float64 at sigma 1, radius 3, 16 points to a
// pixel: 5.1e-8 -> 3.0e-8.
constexpr int NPAD = TS;
constexpr int NROW = 9 + TS;                  // odd: lane i's window starts on its own bank
constexpr int NWAVE = TS + WAVE * NROW;       // a wave's rows: the zeros after one row precede the next
static_assert(NWAVE % 2 == 0, "the wave sums use the rows as float64");
template <class RecT>
__global__ __launch_bounds__(PT) void k_accumulate_narrow(const uint2 *__restrict__ table,
                                                          const uint32_t *__restrict__ slice_off, uint32_t nt,
                                                          const RecT *__restrict__ rec, Cam c,
                                                          double *__restrict__ partial, double *__restrict__ partial_aux, uint64_t max_slices,
                                                          uint64_t max_pairs) {
  constexpr bool AUX = RecInfo<RecT>::aux;
  constexpr int NW = PT / WAVE, NCH = AUX ? 2 : 1;
  __shared__ __align__(8) float rows[NW][NWAVE];
  const uint32_t total_slices = (uint32_t)min((uint64_t)slice_off[nt], max_slices);
  if (blockIdx.x >= total_slices) return;
  const int w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int px = lane % TS;                         // operand pixel; column of the sums
  for (int i = lane; i < NWAVE; i += WAVE) rows[w][i] = 0.0f;
  float *mine = &rows[w][NPAD + lane * NROW];       // this lane's window
  const uint32_t pxb = 4u * (uint32_t)(w * NWAVE + px);
  auto at_byte = [&](uint32_t o) { return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(rows) + o); };
  const int nmax = c.nmax, nin = c.nin;
  SliceWalk<RecT> sw;
  sw.begin(table, rec, total_slices, max_pairs);
  for (; sw.sl < total_slices; sw.next()) {
    const uint32_t t = sw.sd.y & 0xFFFFu;
    const uint32_t pn = sw.count();
    const int tx0 = (int)(t % c.tiles_x) * TS, ty0 = (int)(t / c.tiles_x) * TS;
    double sum[NCH][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[0][i] = sum[NCH - 1][i] = 0.0;
    for (uint32_t c0 = 0; c0 < pn; c0 += PT) {
      float u, v, m, at;
      sw.take(c0, pn, u, v, m, at);
      // the window of one axis, scaled by w0; returns where its row's pixel 0
      // lies (in bytes from the wave's rows)
      auto window = [&](float x, int t0, float w0) -> uint32_t {
        const float fc = floorf(x);
        const float d = x - (fc + 0.5f);
        const float R = c.R;
        auto gauss = [&](float o) { return w0 * __builtin_amdgcn_exp2f((o * o) * c.kexp2); };
        const float e0 = gauss(d);
        mine[nmax] = (nin >= 0 || fabsf(d) <= R) ? e0 : 0.0f;
#pragma unroll
        for (int n = 1; n <= 4; ++n) {
          if (n > nmax) break;                                  // uniform
          float vp = gauss(d - (float)n), vm = gauss(d + (float)n);
          if (n > nin) {
            vp = fabsf(x - ((fc + (float)n) + 0.5f)) <= R ? vp : 0.0f;
            vm = fabsf(x - ((fc - (float)n) + 0.5f)) <= R ? vm : 0.0f;
          }
          mine[nmax + n] = vp;
          mine[nmax - n] = vm;
        }
        // a pair's window meets the tile: its origin lies in [-2 nmax, 15]
        // (lanes past the slice: any place inside the row)
        const int wx = min(max((int)fc - nmax - t0, -2 * nmax), TS - 1);
        return 4u * (uint32_t)(lane * NROW + NPAD - wx);
      };
      float av[16], bv[16];
      const uint32_t rx = window(u, tx0, 1.0f);
      wave_sync_mem();
      for_16([&](auto st) { bv[st] = at_byte(row_bcast<st>(rx) + pxb); }, std::make_integer_sequence<int, 16>{});
      wave_sync_mem();
      const uint32_t ry = window(v, ty0, m * c.wscale);
      wave_sync_mem();
      for_16([&](auto st) { av[st] = at_byte(row_bcast<st>(ry) + pxb); }, std::make_integer_sequence<int, 16>{});
      wave_sync_mem();
      float4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int st = 0; st < 16; ++st) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[st], bv[st], acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[0][i] += (double)acc[i];
      if constexpr (AUX) {
        // the second channel's rows are the first's times the point's attribute
        for_16([&](auto st) { av[st] = times_attr(av[st], __uint_as_float(row_bcast<st>(__float_as_uint(at)))); },
               std::make_integer_sequence<int, 16>{});
        float4v acc2 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int st = 0; st < 16; ++st) acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[st], bv[st], acc2, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[NCH - 1][i] += (double)acc2[i];
      }
    }
    // the wave sums of each pixel, through the start of the rows (lane l holds
    // rows 4 (l / 16) .. + 3 of column l % 16)
    double *part = reinterpret_cast<double *>(rows[w]);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      wave_sync_mem();
#pragma unroll
      for (int i = 0; i < 4; ++i) part[((lane / TS) * 4 + i) * TS + px] = sum[ch][i];
      __syncthreads();
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < NW; ++g) s += reinterpret_cast<const double *>(rows[g])[threadIdx.x];
      (ch ? partial_aux : partial)[(uint64_t)sw.sl * (TS * TS) + threadIdx.x] = s * c.wnorm;
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[i * WAVE + lane] = 0.0;
    wave_sync_mem();
  }
}

// Wider blobs: whole rows of 16 values, every pixel with its own exponential
// (relative error ~3e-7) and truncation test.
constexpr int GXS = TS + 1;          // padded row: conflict-free writes
template <class RecT>
__global__ __launch_bounds__(PT) void k_accumulate_wide(const uint2 *__restrict__ table,
                                                        const uint32_t *__restrict__ slice_off, uint32_t nt,
                                                        const RecT *__restrict__ rec, Cam c,
                                                        double *__restrict__ partial, double *__restrict__ partial_aux,
                                                        uint64_t max_slices, uint64_t max_pairs) {
  constexpr bool AUX = RecInfo<RecT>::aux;
  constexpr int NW = PT / WAVE, NCH = AUX ? 2 : 1;
  __shared__ float gx[PT][GXS];
  __shared__ float gy[PT][GXS];
  __shared__ double part[NW][TS * TS];  // the waves' slice sums
  const uint32_t total_slices = (uint32_t)min((uint64_t)slice_off[nt], max_slices);
  if (blockIdx.x >= total_slices) return;
  const int w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  SliceWalk<RecT> sw;
  sw.begin(table, rec, total_slices, max_pairs);
  for (; sw.sl < total_slices; sw.next()) {
    const uint32_t t = sw.sd.y & 0xFFFFu;
    const uint32_t pn = sw.count();
    const int tx0 = (int)(t % c.tiles_x) * TS, ty0 = (int)(t / c.tiles_x) * TS;
    double sum[NCH][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[0][i] = sum[NCH - 1][i] = 0.0;
    for (uint32_t c0 = 0; c0 < pn; c0 += PT) {
      float u, v, m, at;
      sw.take(c0, pn, u, v, m, at);
      // A pixel is covered when its float32 offset fl(t - (i + 1/2)) lies in
      // [-R, R].  Pixels past the image edge are computed and dropped by the
      // final sum; lanes past the slice carry mass 0.
      const float R = c.R, w0 = m * c.wscale;
      const float cx0 = (float)tx0 + 0.5f, cy0 = (float)ty0 + 0.5f;
#pragma unroll
      for (int e = 0; e < TS; ++e) {
        const float ox = u - (cx0 + (float)e), oy = v - (cy0 + (float)e);
        const float ex = __builtin_amdgcn_exp2f((ox * ox) * c.kexp2);
        const float ey = __builtin_amdgcn_exp2f((oy * oy) * c.kexp2);
        gx[threadIdx.x][e] = fabsf(ox) <= R ? ex : 0.0f;
        gy[threadIdx.x][e] = fabsf(oy) <= R ? w0 * ey : 0.0f;
      }
      wave_sync_mem();
      float av[16], bv[16];   // all LDS operands first: one wait, not sixteen
#pragma unroll
      for (int st = 0; st < 16; ++st) {
        const int kk = w * WAVE + (lane / TS) * 16 + st;
        av[st] = gy[kk][lane % TS];
        bv[st] = gx[kk][lane % TS];
      }
      wave_sync_mem();        // the next chunk rewrites this wave's rows after its reads
      float4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int st = 0; st < 16; ++st) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[st], bv[st], acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[0][i] += (double)acc[i];
      if constexpr (AUX) {
        for_16([&](auto st) { av[st] = times_attr(av[st], __uint_as_float(row_bcast<st>(__float_as_uint(at)))); },
               std::make_integer_sequence<int, 16>{});
        float4v acc2 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int st = 0; st < 16; ++st) acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[st], bv[st], acc2, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[NCH - 1][i] += (double)acc2[i];
      }
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
      for (int i = 0; i < 4; ++i) part[w][((lane / TS) * 4 + i) * TS + lane % TS] = sum[ch][i];
      __syncthreads();
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < NW; ++g) s += part[g][threadIdx.x];
      (ch ? partial_aux : partial)[(uint64_t)sw.sl * (TS * TS) + threadIdx.x] = s * c.wnorm;
      __syncthreads();
    }
  }
}

// Sum each tile's slice partials and write the image: FIN_G groups of 256
// threads (a thread per pixel) add a contiguous share of the slices each, in
// slice order in float64, sixteen loaded together (a tile in front of a dense
// clump has thousands of slices), and the shares are added in order.
constexpr int FIN_G = 4;
__global__ __launch_bounds__(FIN_G * PT) void k_finalize(const uint32_t *__restrict__ slice_off, uint32_t nt,
                                                         const double *__restrict__ partial, Cam c,
                                                         float *__restrict__ image, uint64_t max_slices) {
  __shared__ double share[FIN_G - 1][PT];
  const uint32_t g = threadIdx.x / PT, p = threadIdx.x % PT;
  for (uint32_t t = blockIdx.x; t < nt; t += gridDim.x) {
    const uint32_t b = slice_off[t], e = (uint32_t)min((uint64_t)slice_off[t + 1], max_slices);
    const uint32_t per = e > b ? (e - b + FIN_G - 1) / FIN_G : 0u;
    const uint32_t b1 = min(e, b + g * per), e1 = min(e, b1 + per);
    double s = 0.0;
    for (uint32_t sl = b1; sl < e1; sl += 16) {
      double v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = partial[(uint64_t)min(sl + k, e1 - 1) * (TS * TS) + p];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (sl + k < e1) s += v[k];
    }
    if (e > b + 1) {   // uniform: a single slice is its own sum
      if (g) share[g - 1][p] = s;
      __syncthreads();
      if (g == 0)
        for (int k = 0; k < FIN_G - 1; ++k) s += share[k][p];
      __syncthreads();
    }
    if (g) continue;
    const int i = (int)(t % c.tiles_x) * TS + (int)(p % TS);
    const int j = (int)(t / c.tiles_x) * TS + (int)(p / TS);
    if (i < (int)c.W && j < (int)c.H) image[(uint64_t)j * c.W + i] = (float)s;
  }
}

// --- radial cubic blob -------------------------------------------------------------
//
// The compact cubic spline of smoothed-particle hydrodynamics, normalised in
// two dimensions: W(r; h) = 40 / (7 pi h^2) w(r / h), w(q) = 1 - 6 q^2 + 6 q^3
// (q <= 1/2), 2 (1 - q)^3 (1/2 < q < 1), 0 beyond.  A pixel takes a point iff
// fl64(ox^2) + fl64(oy^2) < h^2 in float64 (both squares of the float32
// offsets are exact there).  The value is evaluated in float64: near the rim
// w ~ 2 (1 - q)^3 needs 1 - q to far better than float32's relative 6e-8 for
// the pixel's 1e-5 bound, so q = sqrt(r^2) / h is formed in float64, and so
// are the sums.
constexpr double kCubicNorm = 40.0 / (7.0 * 3.14159265358979323846);

__device__ __forceinline__ void load_rec(const RecC *r, uint64_t q, float &u, float &v, float &m, float &h,
                                         float &a) {
  const float4 t = reinterpret_cast<const float4 *>(r)[q];
  u = t.x; v = t.y; m = t.z; h = t.w; a = 0.0f;
}
__device__ __forceinline__ void load_rec(const RecCA *r, uint64_t q, float &u, float &v, float &m, float &h,
                                         float &a) {
  const RecCA t = r[q];
  u = t.u; v = t.v; m = t.m; h = t.h; a = t.a;
}

// One block per slice (as the Gaussian accumulation).  The spline is not
// separable, so every covered pixel of every record is evaluated: a blob of
// pixel radius h covers only pixels of the W x W window that starts at its
// first admitted pixel, W = floor(2 h + 0.05) + 1 (the binning's conservative
// range starts 1/100 pixel early, and the float32 rounding of the range stays
// below the rest of the margin).  The lanes of a wave take (record, window
// pixel) items:
//   W <= 4   four records of 16 pixels each per step
//   W == 5   two records of 32 lanes
//   W == 6   the records' pixels end to end, 64 per step
//   W <= 8   one record of 8 x 8 pixels per step
//   larger   one record over all pixels of the tile, four rows per step
// so that the lanes do the same work wherever the records lie.  A wave sorts
// its 64 records by these classes in LDS (stable), each with the float64
// factors every one of its pixels needs, and adds the contributions to tile
// sums of its own in LDS (float64, one LDS add instruction per step).  Two
// records that may cover one pixel in the same step go to different sums, or
// are added by different instructions, and a wave's LDS instructions complete
// in order: every sum is formed in an order fixed by the records, so the image
// is bit-reproducible.  What bounds it is the issue of the float64 evaluation,
// 54 vector instructions per step of 64 items (vector issue busy 68% of the
// time, LDS 44%).
//
// Before, thread p owned pixel p and walked the records of a chunk that cover
// it (narrow blobs), or all of them (radii that differ or exceed 3.9 pixels):
// where a dense clump puts a whole chunk on a few pixels (an NFW core, all of
// a Morton run), a few lanes walked while the block waited.  Accumulation of
// 16.7 M NFW particles' cut at 1920x1080, h = 1.5 px: 856 -> 388 us; of 4 M
// particles with world radii (1.3 to 2.5 px) and a colour channel: 2537 -> 447
// us; of 1 M at h = 2.5 px: 175 -> 148 us.
constexpr int CSUM = 2;              // tile sums per wave
constexpr int CRS = TS + 2;          // their row stride in float64 (36 banks: a window's rows stay apart)
constexpr int CTILE = TS * CRS;
constexpr int NCLS = 5;

__device__ __forceinline__ void lds_add_f64(double *p, double v) { unsafeAtomicAdd(p, v); }

template <class RecT>
__global__ __launch_bounds__(PT) void k_accumulate_cubic(const uint2 *__restrict__ table,
                                                         const uint32_t *__restrict__ slice_off, uint32_t nt,
                                                         const RecT *__restrict__ rec, Cam c,
                                                         double *__restrict__ partial, double *__restrict__ partial_aux, uint64_t max_slices,
                                                         uint64_t max_pairs) {
  constexpr bool AUX = RecInfo<RecT>::aux;
  constexpr int NW = PT / WAVE;
  constexpr int CH = AUX ? 2 : 1;                        // image channels
  constexpr int U = AUX ? 2 : 1;                         // two channels leave room for half the waves
  __shared__ double sum[NW][CSUM][CH][CTILE];
  // a record: u, v, and either the centre of its window's first pixel or (a
  // blob over the whole tile) of the tile's; 1 / h^2, m 40 / (7 pi h^2); h^2;
  // that first pixel within the tile (int16 x, y)
  __shared__ float4 sgeo[NW][WAVE];
  __shared__ double2 sfac[NW][WAVE];
  __shared__ double shh[NW][WAVE];
  __shared__ uint32_t sorg[NW][WAVE];
  __shared__ double sfaca[AUX ? NW : 1][AUX ? WAVE : 1]; // the same times the attribute
  const uint32_t total_slices = (uint32_t)min((uint64_t)slice_off[nt], max_slices);
  if (blockIdx.x >= total_slices) return;
  const int w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  for (uint32_t sl = blockIdx.x; sl < total_slices; sl += gridDim.x) {
    const uint2 sd = table[sl];
    const uint32_t t = sd.y & 0xFFFFu;
    const uint64_t pb = sd.x;
    const uint64_t pe = min(pb + (sd.y >> 16), max_pairs);
    const int tx0 = (int)(t % c.tiles_x) * TS, ty0 = (int)(t / c.tiles_x) * TS;
    for (int i = threadIdx.x; i < NW * CSUM * CH * CTILE; i += PT) (&sum[0][0][0][0])[i] = 0.0;
    __syncthreads();
    // U steps together: item u of this lane is pixel (dx, dy) from the first one
    // of record slot[u] of this wave; its value is added to sum g by the
    // instruction of its phase.  The U chains of LDS reads and float64
    // operations run side by side, without branches.
    auto items = [&](const bool (&live)[2], const uint32_t (&slot)[2], const int (&dx)[2], const int (&dy)[2],
                     const int (&g)[2], const int (&phase)[2], int phases) {
      float4 r[U];
      double2 f[U];
      double hh[U], fa[U];
      uint32_t org[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        r[u] = sgeo[w][slot[u]];
        f[u] = sfac[w][slot[u]];
        hh[u] = shh[w][slot[u]];
        org[u] = sorg[w][slot[u]];
        fa[u] = AUX ? sfaca[AUX ? w : 0][AUX ? slot[u] : 0] : 0.0;
      }
      bool ok[U];
      int o[U];
      double wq[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int px = (int)(int16_t)(org[u] & 0xFFFFu) + dx[u], py = (int)(int16_t)(org[u] >> 16) + dy[u];
        // pixel centres are half-integers below 2^15: the sums are exact
        const float ox = r[u].x - (r[u].z + (float)dx[u]), oy = r[u].y - (r[u].w + (float)dy[u]);
        const double ox64 = (double)ox, oy64 = (double)oy;
        const double r2 = __builtin_fma(ox64, ox64, oy64 * oy64);   // exact squares, one rounding
        ok[u] = live[u] && r2 < hh[u] && (unsigned)px < (unsigned)TS && (unsigned)py < (unsigned)TS;
        // q = sqrt(r2) / h from the hardware reciprocal square root and one
        // Newton step (relative error far below 1e-12)
        const double q2 = fmax(r2 * f[u].x, 1e-280);
        const double y = __builtin_amdgcn_rsq(q2);
        const double gq = q2 * y;
        const double q = __builtin_fma(gq, __builtin_fma(-gq, 0.5 * y, 0.5), gq);
        const double p = 1.0 - q;
        const double wi = __builtin_fma(-6.0 * q2, p, 1.0), wo = (p * p) * (p + p);
        wq[u] = q <= 0.5 ? wi : wo;
        o[u] = py * CRS + px;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        for (int ph = 0; ph < phases; ++ph)
          if (ok[u] && (phases == 1 || phase[u] == ph)) {
            lds_add_f64(&sum[w][g[u]][0][o[u]], f[u].y * wq[u]);
            if constexpr (AUX) lds_add_f64(&sum[w][g[u]][CH - 1][o[u]], fa[u] * wq[u]);
          }
    };
    for (uint64_t c0 = pb + (uint64_t)w * WAVE; c0 < pe; c0 += PT) {
      // the wave's records, sorted by class
      const bool have = c0 + lane < pe;
      float u, v, m, h, at;
      load_rec(rec, have ? c0 + lane : pb, u, v, m, h, at);
      const int win = (int)floorf(2.0f * h + 0.05f) + 1;
      const int cls = win <= 4 ? 0 : win <= 6 ? win - 4 : win <= 8 ? 3 : 4;
      uint32_t slot = 0, first[NCLS + 1];
      first[0] = 0;
#pragma unroll
      for (int k = 0; k < NCLS; ++k) {
        const uint64_t mask = __ballot(have && cls == k);
        if (have && cls == k) slot = first[k] + rank_below(mask);
        first[k + 1] = first[k] + (uint32_t)__popcll(mask);
      }
      if (have) {
        const int x0 = (int)ceilf(u - 0.5f - h - 0.01f) - tx0, y0 = (int)ceilf(v - 0.5f - h - 0.01f) - ty0;
        const double h2 = (double)h * (double)h, ih2 = 1.0 / h2;
        const double fm = (double)m * (kCubicNorm * ih2);
        const int fx = cls == 4 ? 0 : x0, fy = cls == 4 ? 0 : y0;
        sgeo[w][slot] = make_float4(u, v, (float)(tx0 + fx) + 0.5f, (float)(ty0 + fy) + 0.5f);
        sfac[w][slot] = make_double2(ih2, fm);
        shh[w][slot] = h2;
        sorg[w][slot] = ((uint32_t)fx & 0xFFFFu) | ((uint32_t)fy << 16);
        if constexpr (AUX) sfaca[w][slot] = fm * (double)at;
      }
      wave_sync_mem();
      const int l16 = lane & 15, l32 = lane & 31;
      for (uint32_t k = first[0]; k < first[1]; k += 4 * U) {
        const uint32_t a0 = k + lane / 16, a1 = a0 + 4, last = first[1] - 1;
        items({a0 <= last, a1 <= last}, {min(a0, last), min(a1, last)}, {l16 & 3, l16 & 3}, {l16 >> 2, l16 >> 2},
              {(lane >> 4) & 1, (lane >> 4) & 1}, {lane >> 5, lane >> 5}, 2);
      }
      for (uint32_t k = first[1]; k < first[2]; k += 2 * U) {
        const uint32_t a0 = k + lane / 32, a1 = a0 + 2, last = first[2] - 1;
        items({l32 < 25 && a0 <= last, l32 < 25 && a1 <= last}, {min(a0, last), min(a1, last)}, {l32 % 5, l32 % 5},
              {l32 / 5, l32 / 5}, {lane >> 5, lane >> 5}, {0, 0}, 1);
      }
      const uint32_t n6 = 36 * (first[3] - first[2]);
      for (uint32_t k = 0; k < n6; k += U * WAVE) {
        const uint32_t i0 = k + lane, i1 = i0 + WAVE, j0 = min(i0, n6 - 1), j1 = min(i1, n6 - 1);
        const uint32_t r0 = j0 / 36, r1 = j1 / 36, e0 = j0 % 36, e1 = j1 % 36;
        items({i0 < n6, i1 < n6}, {first[2] + r0, first[2] + r1}, {(int)(e0 % 6), (int)(e1 % 6)},
              {(int)(e0 / 6), (int)(e1 / 6)}, {(int)(r0 & 1), (int)(r1 & 1)},
              {(int)((r0 >> 1) & 1), (int)((r1 >> 1) & 1)}, 2);
      }
      for (uint32_t k = first[3]; k < first[4]; k += U) {
        const uint32_t k1 = min(k + 1, first[4] - 1);
        items({true, k + 1 < first[4]}, {k, k1}, {lane & 7, lane & 7}, {lane >> 3, lane >> 3}, {0, 0}, {0, 0}, 1);
      }
      for (uint32_t k = first[4]; k < first[5]; ++k)
        for (int y = 0; y < TS; y += U * (WAVE / TS))
          items({true, true}, {k, k}, {lane % TS, lane % TS}, {y + lane / TS, y + WAVE / TS + lane / TS}, {0, 0},
                {0, 0}, 1);
      wave_sync_mem();                                   // the records are rewritten
    }
    __syncthreads();
    const int o = (threadIdx.x / TS) * CRS + threadIdx.x % TS;
    double s[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      s[ch] = 0.0;
#pragma unroll
      for (int g = 0; g < NW * CSUM; ++g) s[ch] += sum[g / CSUM][g % CSUM][ch][o];
    }
    partial[(uint64_t)sl * (TS * TS) + threadIdx.x] = s[0];
    if constexpr (AUX) partial_aux[(uint64_t)sl * (TS * TS) + threadIdx.x] = s[CH - 1];
    __syncthreads();
  }
}

// Sum over the four lanes of a quad, in every lane.
__device__ __forceinline__ double quad_sum(double v) {
  auto swapped = [](double a, auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    const uint64_t b = (uint64_t)__double_as_longlong(a);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, C, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), C, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
  };
  v += swapped(v, std::integral_constant<int, 0xB1>{});   // quad_perm 1 0 3 2
  v += swapped(v, std::integral_constant<int, 0x4E>{});   // quad_perm 2 3 0 1
  return v;
}

// One pixel's terms of the cubic blob's adjoint: (ox, oy) its offset, gf the
// image's gradient there, rad = (h^2, 1 / h^2), fac the factors of the
// position's and the radius' sums; s = sums of the mass, u, v and radius.
__device__ __forceinline__ void adjoint_pixel(float ox, float oy, float gf, double2 rad, double2 fac, bool radius,
                                              double (&s)[4]) {
  const double ox64 = (double)ox, oy64 = (double)oy;
  const double r2 = __builtin_fma(ox64, ox64, oy64 * oy64);   // exact squares, one rounding
  const double q2 = fmax(r2 * rad.y, 1e-280);
  const double yq = __builtin_amdgcn_rsq(q2), gq = q2 * yq;
  const double nt = __builtin_fma(-gq, 0.5 * yq, 0.5);
  const double q = __builtin_fma(gq, nt, gq), qi = __builtin_fma(yq, nt, yq);   // q and 1 / q
  const double pq = 1.0 - q, pp = pq * pq;
  const bool inner = q <= 0.5;
  const double wq = inner ? __builtin_fma(-6.0 * q2, pq, 1.0) : pp * (pq + pq);
  const double dwq = inner ? __builtin_fma(18.0, q, -12.0) : -6.0 * pp * qi;    // w'(q) / q
  const double gp = (double)gf;
  if (r2 < rad.x) {
    const double t = fac.x * (dwq * gp);
    s[0] += wq * gp;
    s[1] += t * ox64;
    s[2] += t * oy64;
    if (radius) s[3] += fac.y * (__builtin_fma(-q2, dwq, -2.0 * wq) * gp);
  }
}

// The gradients of a point from its four sums.
__device__ __forceinline__ void adjoint_point(const Cam &c, bool vis, float xc, float yc, float zc, float h,
                                              bool dh_live, double ih2, double am, double au, double av, double ah,
                                              uint64_t k, float *gm, float *gx, float *gy, float *gz) {
  double dx = 0.0, dy = 0.0, dz = 0.0;
  if (vis) {
    if (c.proj == 0) {
      dx = au * (double)c.W;
      dy = av * (double)c.H;
    } else {
      const double zz = (double)zc;
      const double a = (double)c.F / zz;
      const double bu = (double)c.F * (double)xc / (zz * zz);
      const double bv = (double)c.F * (double)yc / (zz * zz);
      const double dh = dh_live ? -(double)h / zz : 0.0;
      dx = au * (a * c.rx - bu * c.fx) + av * (a * c.ux - bv * c.fx) + ah * dh * c.fx;
      dy = au * (a * c.ry - bu * c.fy) + av * (a * c.uy - bv * c.fy) + ah * dh * c.fy;
      dz = au * (a * c.rz - bu * c.fz) + av * (a * c.uz - bv * c.fz) + ah * dh * c.fz;
    }
  }
  gm[k] = (float)(am * (kCubicNorm * ih2));
  if (gx) gx[k] = (float)dx;
  if (gy) gy[k] = (float)dy;
  if (gz) gz[k] = (float)dz;
}

// Adjoint of the cubic blob over each point's own footprint (float64 sums):
// dI/dm = W, dI/dox = m 40/(7 pi h^4) (w'(q)/q) ox, and with a world-space size
// (radius not clamped) dI/dh = m 40/(7 pi h^3) (-2 w - q w'(q)) with
// dh/dp = -(h / zc) f.  A wave projects 64 points, a lane each, then takes the
// pixels of 16 points at a time, four lanes a point: four lanes read four
// neighbouring pixels of the gradient, where a thread per point reads 64
// scattered ones with every load.  Points of equally many pixels are taken
// together, so that no lane waits for a longer one's window.  Bound by the
// float64 operations of a pixel (vector issue 75 % busy); q, its reciprocal and
// w'(q)/q come from one hardware reciprocal square root and one Newton step
// instead of a square root and two divisions (of 9.6 M gradients with radii
// from 0.6 to 16 one differs, by an ulp of float32).  A million points of 25
// pixels: 66 us, against 101 with a thread per point; reading the gradient a
// pixel ahead changed nothing.
__global__ __launch_bounds__(PT) void k_backward_cubic(const float *__restrict__ x, const float *__restrict__ y,
                                                       const float *__restrict__ z, const float *__restrict__ m,
                                                       uint64_t count, Cam c, const float *__restrict__ g,
                                                       float *__restrict__ gm, float *__restrict__ gx,
                                                       float *__restrict__ gy, float *__restrict__ gz) {
  constexpr int NW = PT / WAVE;
  constexpr int Q = 4;                       // lanes per point
  __shared__ float4 sgeo[NW][WAVE];          // u, v, centre of the window's first pixel
  __shared__ int4 swin[NW][WAVE];            // its index, columns, pixels, step of four pixels (rows << 16 | columns)
  __shared__ double2 srad[NW][WAVE];         // h^2, 1 / h^2
  __shared__ double2 sfac[NW][WAVE];         // factors of the position's and the radius' sums
  __shared__ double ssum[NW][4][WAVE];       // mass, u, v, radius
  const int w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const bool radius = c.Fhw > 0.0f;
  for (uint64_t k0 = (uint64_t)blockIdx.x * PT + (uint64_t)w * WAVE; k0 < count; k0 += (uint64_t)gridDim.x * PT) {
    const uint64_t k = k0 + lane;
    const bool have = k < count;
    float u = 0.0f, v = 0.0f, xc = 0.0f, yc = 0.0f, zc = 0.0f;
    const bool vis = have && project(c, x[k], y[k], z[k], u, v, xc, yc, zc);
    // a culled point's pixel count is 0 and its sums stay 0: any finite radius
    // (the camera's fixed one may be 0 beside a world radius)
    const float h = vis ? cubic_radius(c, zc) : lodh::BLOB_H_MIN;
    bool dh_live = false;
    if (vis && radius) {
      const float hp = __fdiv_rn(c.Fhw, zc);
      dh_live = hp >= lodh::BLOB_H_MIN && hp <= lodh::BLOB_H_MAX;
    }
    int i0 = 0, i1 = -1, j0 = 0, j1 = -1;
    if (!(vis && cover_range(h, u, c.W, i0, i1) && cover_range(h, v, c.H, j0, j1))) i1 = i0 - 1;
    const int nx = i1 - i0 + 1, pixels = nx * (j1 - j0 + 1);
    const int cls = pixels <= 4 * Q ? 0 : pixels <= 5 * Q ? 1 : pixels <= 7 * Q ? 2 : 3;
    int slot = 0, first = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t mask = __ballot(cls == q);
      if (cls == q) slot = first + (int)rank_below(mask);
      first += __popcll(mask);
    }
    {
      const double h64 = (double)h, hh = h64 * h64, ih2 = 1.0 / hh;
      const double f = (have ? (double)m[k] : 0.0) * kCubicNorm * (ih2 * ih2);
      const int step = nx > Q ? Q : nx < 1 ? 0 : Q % nx, rows = nx > Q || nx < 1 ? 0 : Q / nx;
      sgeo[w][slot] = make_float4(u, v, (float)i0 + 0.5f, (float)j0 + 0.5f);
      swin[w][slot] = make_int4(j0 * (int)c.W + i0, nx, pixels, rows << 16 | step);
      srad[w][slot] = make_double2(hh, ih2);
      sfac[w][slot] = make_double2(f, dh_live ? f * h64 : 0.0);
    }
    wave_sync_mem();
#pragma unroll 1
    for (int r = 0; r < Q; ++r) {
      const int p = r * (WAVE / Q) + lane / Q;
      const float4 geo = sgeo[w][p];
      const int4 win = swin[w][p];
      const double2 rad = srad[w][p], fac = sfac[w][p];
      const int step = win.w & 0xFFFF, rows = win.w >> 16;
      double t[4] = {0.0, 0.0, 0.0, 0.0};
      int i = lane % Q, j = 0;
      while (i >= win.y && win.y > 0) { i -= win.y; ++j; }
      for (int e = lane % Q; e < win.z; e += Q) {
        const float gf = g[win.x + j * (int)c.W + i];
        // pixel centres are half-integers below 2^15: the sums are exact
        adjoint_pixel(geo.x - (geo.z + (float)i), geo.y - (geo.w + (float)j), gf, rad, fac, radius, t);
        i += step;
        j += rows;
        if (i >= win.y) { i -= win.y; ++j; }
      }
      t[0] = quad_sum(t[0]);
      t[1] = quad_sum(t[1]);
      t[2] = quad_sum(t[2]);
      if (radius) t[3] = quad_sum(t[3]);
      const int which = lane % Q;
      ssum[w][which][p] = which == 0 ? t[0] : which == 1 ? t[1] : which == 2 ? t[2] : t[3];
    }
    wave_sync_mem();
    if (have)
      adjoint_point(c, vis, xc, yc, zc, h, dh_live, srad[w][slot].y, ssum[w][0][slot], ssum[w][1][slot],
                    ssum[w][2][slot], ssum[w][3][slot], k, gm, gx, gy, gz);
    wave_sync_mem();                         // the next points rewrite the rows
  }
}

// The same with a thread per point: blobs of a fixed radius of a few pixels, for
// which the exchange between the lanes costs more than it saves (see the launch).
__global__ __launch_bounds__(PT) void k_backward_cubic_small(const float *__restrict__ x, const float *__restrict__ y,
                                                             const float *__restrict__ z, const float *__restrict__ m,
                                                             uint64_t count, Cam c, const float *__restrict__ g,
                                                             float *__restrict__ gm, float *__restrict__ gx,
                                                             float *__restrict__ gy, float *__restrict__ gz) {
  for (uint64_t k = (uint64_t)blockIdx.x * PT + threadIdx.x; k < count; k += (uint64_t)gridDim.x * PT) {
    float u, v, xc, yc, zc;
    const bool vis = project(c, x[k], y[k], z[k], u, v, xc, yc, zc);
    const double hh = (double)c.hpx * (double)c.hpx, ih2 = 1.0 / hh;
    const double2 rad = make_double2(hh, ih2), fac = make_double2((double)m[k] * kCubicNorm * (ih2 * ih2), 0.0);
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    int i0, i1, j0, j1;
    if (vis && cover_range(c.hpx, u, c.W, i0, i1) && cover_range(c.hpx, v, c.H, j0, j1))
      for (int j = j0; j <= j1; ++j)
        for (int i = i0; i <= i1; ++i)
          adjoint_pixel(u - ((float)i + 0.5f), v - ((float)j + 0.5f), g[(uint64_t)j * c.W + i], rad, fac, false, t);
    adjoint_point(c, vis, xc, yc, zc, c.hpx, false, ih2, t[0], t[1], t[2], 0.0, k, gm, gx, gy, gz);
  }
}

// --- adjoint -------------------------------------------------------------------

__global__ __launch_bounds__(PT) void k_backward(const float *__restrict__ x, const float *__restrict__ y,
                                                 const float *__restrict__ z, const float *__restrict__ m,
                                                 uint64_t count, Cam c, const float *__restrict__ g,
                                                 float *__restrict__ gm, float *__restrict__ gx,
                                                 float *__restrict__ gy, float *__restrict__ gz) {
  for (uint64_t k = (uint64_t)blockIdx.x * PT + threadIdx.x; k < count; k += (uint64_t)gridDim.x * PT) {
    float u, v, xc, yc, zc;
    float am = 0.0f, au = 0.0f, av = 0.0f;
    const bool vis = project(c, x[k], y[k], z[k], u, v, xc, yc, zc);
    int i0, i1, j0, j1;
    if (vis && axis_range(c, u, c.W, i0, i1) && axis_range(c, v, c.H, j0, j1)) {
      for (int j = j0; j <= j1; ++j) {
        const float oy = v - ((float)j + 0.5f);
        const float ey = c.norm * expf(-(oy * oy) * c.inv2s2);
        float rm = 0.0f, ru = 0.0f, rv = 0.0f;
        for (int i = i0; i <= i1; ++i) {
          const float ox = u - ((float)i + 0.5f);
          const float G = ey * expf(-(ox * ox) * c.inv2s2);
          const float gg = G * g[(uint64_t)j * c.W + i];
          rm += gg;
          ru -= gg * ox;
          rv -= gg * oy;
        }
        am += rm; au += ru; av += rv;
      }
    }
    const float mk = m[k];
    const float du = mk * au * c.inv_s2, dv = mk * av * c.inv_s2;
    float dx = 0.0f, dy = 0.0f, dz = 0.0f;
    if (vis) {
      if (c.proj == 0) {
        dx = du * (float)c.W;
        dy = dv * (float)c.H;
      } else {
        const float a = c.F / zc;
        const float bu = c.F * xc / (zc * zc);
        const float bv = c.F * yc / (zc * zc);
        dx = du * (a * c.rx - bu * c.fx) + dv * (a * c.ux - bv * c.fx);
        dy = du * (a * c.ry - bu * c.fy) + dv * (a * c.uy - bv * c.fy);
        dz = du * (a * c.rz - bu * c.fz) + dv * (a * c.uz - bv * c.fz);
      }
    }
    gm[k] = am;
    if (gx) gx[k] = dx;
    if (gy) gy[k] = dy;
    if (gz) gz[k] = dz;
  }
}

// --- motion codes ----------------------------------------------------------------

// Motion code of one coordinate: the particle's position a in the next
// snapshot against the stored code Q0 = (c << 16) + q at depth d,
// dq = floor((floor(a 2^(d+16)) - Q0 + 2) / 4) clamped to int16 (true when clamped).
__device__ __forceinline__ int16_t motion_code(float a, uint32_t c, uint32_t q, int d, bool &sat) {
  const int64_t Q1 = (int64_t)floorf(a * ldexpf(1.0f, d + 16));
  const int64_t Q0 = ((int64_t)c << 16) + (int64_t)q;
  const int64_t dq = (Q1 - Q0 + 2) >> 2;          // arithmetic shift: floor division by 4
  sat = dq < -32768 || dq > 32767;
  return (int16_t)max((int64_t)-32768, min((int64_t)32767, dq));
}

// One block per node (grid-stride over the node table); thread j codes the
// node's stored points j, j + blockDim, ...  The next snapshot's positions
// are indexed like the build input: snapshot offset + particle id.
__global__ void k_encode_motion(const lod_tree t, const float *__restrict__ xb, const float *__restrict__ yb,
                                const float *__restrict__ zb, const uint64_t *__restrict__ snap_off,
                                uint64_t cap_nodes, int16_t *__restrict__ dqx, int16_t *__restrict__ dqy,
                                int16_t *__restrict__ dqz, uint64_t *__restrict__ saturated) {
  const uint64_t nn = min(t.counts[0], cap_nodes);
  uint32_t sat_count = 0;
  for (uint64_t v = blockIdx.x; v < nn; v += gridDim.x) {
    const int d = t.depth[v];
    const uint64_t pfx = t.prefix[v];
    const uint32_t cell = d ? (uint32_t)(pfx & ((1ull << (3 * d)) - 1)) : 0u;
    const uint32_t cx = compact3(cell), cy = compact3(cell >> 1), cz = compact3(cell >> 2);
    const uint64_t base = snap_off ? snap_off[pfx >> (3 * d)] : 0ull;
    const uint64_t pb = t.pt_begin[v];
    const uint32_t pc = t.pt_count[v];
    for (uint32_t j = threadIdx.x; j < pc; j += blockDim.x) {
      const uint64_t sidx = pb + j;
      const uint64_t g = base + t.pt_id[sidx];
      bool s0, s1, s2;
      dqx[sidx] = motion_code(xb[g], cx, t.qx[sidx], d, s0);
      dqy[sidx] = motion_code(yb[g], cy, t.qy[sidx], d, s1);
      dqz[sidx] = motion_code(zb[g], cz, t.qz[sidx], d, s2);
      sat_count += (uint32_t)s0 + (uint32_t)s1 + (uint32_t)s2;
    }
  }
  if (sat_count) atomicAdd((unsigned long long *)saturated, (unsigned long long)sat_count);
}

// --- writing a node's points back (refinement) ---------------------------------

// Stored points of node v replaced by count positions and masses (count <=
// the node's pt_count): codes q = min(floor(a 2^(d+16)) - (c << 16), 65535)
// relative to the node's cell (positions outside the cell set the domain
// status bit and are clamped), masses as given.
__global__ void k_set_points(const lod_tree t, uint32_t v, const float *__restrict__ x, const float *__restrict__ y,
                             const float *__restrict__ z, const float *__restrict__ m, uint32_t count) {
  if ((uint64_t)v >= t.counts[0]) return;
  const int d = t.depth[v];
  const uint64_t pfx = t.prefix[v];
  const uint32_t cell = d ? (uint32_t)(pfx & ((1ull << (3 * d)) - 1)) : 0u;
  const uint32_t c3[3] = {compact3(cell), compact3(cell >> 1), compact3(cell >> 2)};
  const uint64_t pb = t.pt_begin[v];
  const uint32_t k = min(count, t.pt_count[v]);
  const float scale = ldexpf(1.0f, d + 16);
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < k; j += gridDim.x * blockDim.x) {
    const float a[3] = {x[j], y[j], z[j]};
    uint16_t q[3];
    bool out = false;
    for (int ax = 0; ax < 3; ++ax) {
      const int64_t Q = (int64_t)floorf(a[ax] * scale) - ((int64_t)c3[ax] << 16);
      out |= !(Q >= 0 && Q <= 65535 + 1) || !(a[ax] >= 0.0f);
      q[ax] = (uint16_t)max((int64_t)0, min((int64_t)65535, Q));
    }
    if (out) atomicOr((unsigned long long *)&t.counts[2], (unsigned long long)LOD_STATUS_DOMAIN);
    t.qx[pb + j] = q[0]; t.qy[pb + j] = q[1]; t.qz[pb + j] = q[2];
    t.pt_mass[pb + j] = m[j];
  }
}

// --- LOD decode ----------------------------------------------------------------

// Exclusive offsets of the listed nodes' points: block b scans ids
// [LOFF b, LOFF (b + 1)), one id past the last one included, and the scan of
// the blocks' totals (k_lod_total) is added where an offset is read (lod_off).
// Ids past the node count hold no points; blocks past the list write nothing.
// (One block walking the whole list took 56 us for the 33 k nodes of a 150 M
// particle cut; these two launches take 9.)
__global__ __launch_bounds__(LOFF) void k_lod_offsets(const lod_tree t, const uint32_t *__restrict__ ids,
                                                      const uint64_t *__restrict__ n_ids, uint64_t max_ids,
                                                      uint64_t *__restrict__ offs, uint64_t *__restrict__ bsum) {
  __shared__ uint64_t tmp[LOFF / WAVE + 1];
  const uint64_t ni = min(*n_ids, max_ids);
  const uint64_t k = (uint64_t)blockIdx.x * LOFF + threadIdx.x;
  if ((uint64_t)blockIdx.x * LOFF > ni) return;
  uint64_t c = 0;
  if (k < ni) {
    const uint32_t v = ids[k];
    if (v < t.counts[0]) c = t.pt_count[v];
  }
  uint64_t total;
  const uint64_t o = block_excl_scan<uint64_t>(c, tmp, total);
  if (k <= ni) offs[k] = o;
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// scan of the block totals (in place) and the number of points drawn (one block)
__global__ __launch_bounds__(LOFF) void k_lod_total(const lod_tree t, const uint64_t *__restrict__ n_ids,
                                                    uint64_t max_ids, uint64_t *__restrict__ bsum,
                                                    uint64_t max_points, uint64_t *__restrict__ total) {
  __shared__ uint64_t tmp[LOFF / WAVE + 1];
  const uint64_t nb = min(*n_ids, max_ids) / LOFF + 1;
  uint64_t run = 0;
  for (uint64_t b0 = 0; b0 < nb; b0 += LOFF) {
    const uint64_t b = b0 + threadIdx.x;
    uint64_t step;
    const uint64_t o = block_excl_scan<uint64_t>(b < nb ? bsum[b] : 0ull, tmp, step);
    if (b < nb) bsum[b] = run + o;
    run += step;
  }
  if (threadIdx.x == 0) {
    *total = min(run, max_points);
    if (run > max_points)
      atomicOr((unsigned long long *)&t.counts[2], (unsigned long long)LOD_STATUS_CAPACITY);
  }
}

__global__ __launch_bounds__(PT) void k_lod_decode(const lod_tree t, const uint32_t *__restrict__ ids,
                                                   const uint64_t *__restrict__ n_ids, uint64_t max_ids,
                                                   const uint64_t *__restrict__ offs,
                                                   const uint64_t *__restrict__ bsum, uint64_t max_points,
                                                   float *__restrict__ x, float *__restrict__ y,
                                                   float *__restrict__ z, float *__restrict__ m) {
  const uint64_t nn = t.counts[0];
  const uint64_t ni = min(*n_ids, max_ids);
  for (uint64_t k = blockIdx.x; k < ni; k += gridDim.x) {
    const uint32_t v = ids[k];
    if (v >= nn) continue;
    const int d = t.depth[v];
    const uint64_t pfx = t.prefix[v];
    const uint32_t cell = d ? (uint32_t)(pfx & ((1ull << (3 * d)) - 1)) : 0u;
    const uint32_t cx = compact3(cell), cy = compact3(cell >> 1), cz = compact3(cell >> 2);
    const uint64_t pb = t.pt_begin[v];
    const uint32_t pc = t.pt_count[v];
    const uint64_t ob = lod_off(offs, bsum, k);
    for (uint32_t j = threadIdx.x; j < pc; j += PT) {
      const uint64_t o = ob + j;
      if (o >= max_points) break;
      const uint64_t s = pb + j;
      x[o] = decode_coord(cx, t.qx[s], d);
      y[o] = decode_coord(cy, t.qy[s], d);
      z[o] = decode_coord(cz, t.qz[s], d);
      m[o] = t.pt_mass[s];
    }
  }
}

// --- view-dependent cut ----------------------------------------------------------

struct CutArgs {
  uint32_t proj, W;
  double px, py, pz;
  double F, tau_cbrt;   // tau * n^(1/3)
};

__device__ __forceinline__ bool descends(const lod_tree &t, uint32_t v, const CutArgs &c) {
  if (t.first_child[v] == NONE) return false;
  const int d = t.depth[v];
  const double side = ldexp(1.0, -d);
  if (c.proj == 0) return (double)c.W * side > c.tau_cbrt;
  const uint32_t cell = d ? (uint32_t)(t.prefix[v] & ((1ull << (3 * d)) - 1)) : 0u;
  const double ox = (double)compact3(cell) * side;
  const double oy = (double)compact3(cell >> 1) * side;
  const double oz = (double)compact3(cell >> 2) * side;
  const bool inside = (ox <= c.px && c.px <= ox + side) && (oy <= c.py && c.py <= oy + side) &&
                      (oz <= c.pz && c.pz <= oz + side);
  if (inside) return true;
  const double h = side * 0.5;
  const double dx = (ox + h) - c.px;
  const double dy = (oy + h) - c.py;
  const double dz = (oz + h) - c.pz;
  const double dist = __dsqrt_rn((dx * dx + dy * dy) + dz * dz);
  return c.F * side > c.tau_cbrt * dist;
}

// Drawn nodes of one block of CUT_T nodes: keep[v] = 1 + rank among the block's
// drawn nodes, or 0, and the block's number of drawn nodes.
constexpr int CUT_T = 1024;
__global__ __launch_bounds__(CUT_T) void k_cut_flags(const lod_tree t, CutArgs c, uint64_t cap_nodes,
                                                     uint32_t *__restrict__ keep, uint32_t *__restrict__ sums) {
  __shared__ uint32_t tmp[CUT_T / WAVE + 1];
  const uint64_t nn = min(t.counts[0], cap_nodes);
  const uint64_t v = (uint64_t)blockIdx.x * CUT_T + threadIdx.x;
  if ((uint64_t)blockIdx.x * CUT_T >= nn) return;   // uniform; k_cut_write reads no further than nn
  uint32_t f = 0;
  if (v < nn && !descends(t, (uint32_t)v, c)) {
    f = 1;
    uint32_t u = t.parent[v];
    while (u != NONE) {
      if (!descends(t, u, c)) { f = 0; break; }
      u = t.parent[u];
    }
  }
  uint32_t total;
  const uint32_t rank = block_excl_scan<uint32_t>(f, tmp, total);
  if (v < nn) keep[v] = f ? rank + 1u : 0u;
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// The drawn nodes in node order: a block adds up the blocks before it itself
// (at most some hundreds), which saves the launches of a scan.
__global__ __launch_bounds__(CUT_T) void k_cut_write(const lod_tree t, uint64_t cap_nodes,
                                                     const uint32_t *__restrict__ keep,
                                                     const uint32_t *__restrict__ sums, uint32_t *__restrict__ ids,
                                                     uint64_t cap, uint64_t *__restrict__ n_sel) {
  __shared__ uint64_t tmp[CUT_T / WAVE + 1];
  const uint64_t nn = min(t.counts[0], cap_nodes);
  const uint32_t nb = (uint32_t)((nn + CUT_T - 1) / CUT_T);   // blocks that hold nodes
  if (blockIdx.x >= max(nb, 1u)) return;
  uint64_t before = 0, all = 0;
  for (uint32_t b = threadIdx.x; b < nb; b += CUT_T) {
    const uint32_t s = sums[b];
    if (b < blockIdx.x) before += s;
    all += s;
  }
  before = block_reduce_sum<uint64_t>(before, tmp);
  const uint64_t v = (uint64_t)blockIdx.x * CUT_T + threadIdx.x;
  const uint32_t k = v < nn ? keep[v] : 0u;
  if (k) {
    const uint64_t o = before + k - 1u;
    if (o < cap) ids[o] = (uint32_t)v;
  }
  if (blockIdx.x == 0) {
    all = block_reduce_sum<uint64_t>(all, tmp);
    if (threadIdx.x == 0) {
      *n_sel = min(all, cap);
      if (all > cap) atomicOr((unsigned long long *)&t.counts[2], (unsigned long long)LOD_STATUS_CAPACITY);
    }
  }
}

}  // namespace

// -----------------------------------------------------------------------------
// host side

namespace lodh {

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Bytes of one binned (point, tile) record for a render form.
static size_t rec_bytes(const splat_params &sp, bool aux) {
  if (sp.blob == LOD_BLOB_CUBIC) return aux ? sizeof(RecCA) : sizeof(RecC);
  return aux ? sizeof(RecGA) : sizeof(float3);
}

lod_status splat_layout(uint64_t max_points, const lod_camera &cam, const splat_params &sp, SplatLayout &L,
                        bool aux, bool few_units) {
  L = SplatLayout{};
  L.tiles_x = (cam.W + TS - 1) / TS;
  L.tiles_y = (cam.H + TS - 1) / TS;
  const uint64_t nt = (uint64_t)L.tiles_x * L.tiles_y;
  if (nt == 0 || nt > SPLAT_MAX_TILES) return LOD_EUNSUPPORTED;
  L.n_tiles = (uint32_t)nt;
  const double R = (double)blob_max_radius(sp);
  const uint64_t width = 2 * (uint64_t)std::ceil(R) + 3;         // pixels a blob's tile range can span
  const uint64_t tpa = std::min<uint64_t>((width + TS - 1) / TS + 1, std::max(L.tiles_x, L.tiles_y));
  L.max_points = max_points;
  // pair counts are 32-bit, and a point adds at least one pair
  if (max_points >= (1ull << 32)) return LOD_EUNSUPPORTED;
  L.max_pairs = std::max<uint64_t>(1, max_points * tpa * tpa);
  if (L.max_pairs >= (1ull << 32)) return LOD_EUNSUPPORTED;
  L.aux = aux;
  // Units: 64 per chunk.  A unit's row of the count table is written, scanned
  // and read, so a unit is not much shorter than an eighth of the tiles (32
  // bytes of table per point), and no longer than 512 points while there are
  // fewer than 4096 units (a 256x256 image of 262 k points: 2048 units of 128,
  // where units of 2048 left 128 waves on the chip; 1 M points at 1024^2: see
  // the rows rule at the launches).  few_units (a workspace of fixed size):
  // 2048; the image does not depend on it.
  const uint64_t unit = few_units ? 2048 : std::min<uint64_t>(512, std::max<uint64_t>(128, nt / 2));
  L.chunks = (uint32_t)std::min<uint64_t>(SPLAT_MAX_CHUNKS,
                                          std::max<uint64_t>(1, (max_points + 64 * unit - 1) / (64 * unit)));
  L.units = 64 * L.chunks;
  // at most a slice per tile besides the full ones, of which the largest count
  // over all numbers of pairs up to max_pairs: a plan covers fewer points
  const bool cubic = sp.blob == LOD_BLOB_CUBIC;
  uint64_t full = 0;
  for (int top = 19; top <= 32; ++top) {   // slice_bits steps at powers of two
    const uint64_t pairs = std::min<uint64_t>(L.max_pairs, 1ull << top);
    full = std::max(full, pairs >> slice_bits((uint32_t)std::min<uint64_t>(pairs, ~0u), cubic));
  }
  L.max_slices = nt + full + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  L.tile_count = take(4 * (nt + 1));
  L.tile_off = take(4 * (nt + 1));
  L.ucount = take(4 * (size_t)L.units * nt);
  L.pchunk = take(4 * (size_t)L.chunks * nt);
  L.slice_off = take(4 * (nt + 1));
  L.counters = take(64);
  L.rec = take(rec_bytes(sp, aux) * L.max_pairs);
  L.partial = take(8 * (size_t)TS * TS * L.max_slices);
  L.partial_aux = aux ? take(8 * (size_t)TS * TS * L.max_slices) : L.partial;
  L.slice_table = take(8 * (size_t)L.max_slices);
  L.total = off;
  return LOD_OK;
}

// The size by which the allocation-free render accepts a call: binning units of
// 2048 points, the records, and a float32 tile per 4096 pairs and per tile.
size_t noalloc_size(uint64_t count, const splat_params &sp, const SplatLayout &L) {
  const uint64_t nt = L.n_tiles, slices = nt + L.max_pairs / 4096 + 1;
  const uint64_t chunks = std::min<uint64_t>(SPLAT_MAX_CHUNKS, std::max<uint64_t>(1, (count + (1u << 17) - 1) >> 17));
  return 3 * align256(4 * (nt + 1)) + align256(4 * 64 * chunks * nt) + align256(4 * chunks * nt) + align256(64) +
         align256(rec_bytes(sp, false) * L.max_pairs) + align256(4 * TS * TS * slices) + align256(8 * slices);
}

// Binning, accumulation and the final slice sums for any point source and
// record form.  image_aux receives the attribute channel (RecT carrying one).
template <class Src, class RecT>
static lod_status launch_splat_src(const Src &src, bool any, const lod_camera &cam, const splat_params &sp,
                                   void *ws, const SplatLayout &L, float *image, float *image_aux,
                                   uint64_t *status_word, hipStream_t st, const HlStage *hs = nullptr) {
  char *W = (char *)ws;
  Cam c = make_cam(cam, sp, &L);
  const uint32_t nt = L.n_tiles;
  uint32_t *tcount = (uint32_t *)(W + L.tile_count);
  uint32_t *toff = (uint32_t *)(W + L.tile_off);
  uint32_t *ucount = (uint32_t *)(W + L.ucount);
  uint32_t *pchunk = (uint32_t *)(W + L.pchunk);
  uint32_t *soff = (uint32_t *)(W + L.slice_off);
  uint64_t *ctr = (uint64_t *)(W + L.counters);
  uint64_t *status = status_word ? status_word : ctr;
  RecT *rec = (RecT *)(W + L.rec);
  double *partial = (double *)(W + L.partial), *partial_aux = (double *)(W + L.partial_aux);
  uint2 *stab = (uint2 *)(W + L.slice_table);
  int nbits = 0;
  while ((1u << nbits) < nt) ++nbits;
  const size_t lds = 4 * (size_t)nt;
  // Counters and cursors in the rows of the count table for points in Morton
  // order (a tree's): their rounds stay in one window for long, and the waves
  // per CU are not limited by LDS.  In LDS for arrays in the caller's order,
  // which may be random, unless a unit's points are too few to pay for the
  // initialisation of its LDS row and for the waves that its LDS keeps away
  // (random points, fill + count: 1 M in units of 512, rows 111 us, of 2048 in
  // LDS 168; 4 M in units of 977, LDS 264, rows 486; 16.7 M 745 and 1890).
  const uint64_t per = (L.max_points + L.units - 1) / L.units;
  const bool rows = IsTree<Src>::value || per <= nt / 8;
  const uint32_t *pre = L.chunks > 1 ? pchunk : nullptr;
  const bool plan_scans = any && L.chunks > 1 && nt <= PLAN_T;
  if (any) {
    const bool narrow_counts = per + WAVE <= 65535;
    auto count = [&](auto kernel, size_t bytes, const HlStage &h) {
      LOD_LAUNCH_NAMED("k_bin_count", kernel, dim3(L.units), dim3(BW), bytes, st, src, c, L.units, nbits, ucount, h);
    };
    if constexpr (IsTree<Src>::value) {
      if (hs) count(k_bin_count<Src, void, true>, 0, *hs);
      else count(k_bin_count<Src, void>, 0, HlStage{});
    } else {
      if (rows) count(k_bin_count<Src, void>, 0, HlStage{});
      else if (narrow_counts) count(k_bin_count<Src, uint16_t>, 2 * (size_t)(nt + 1), HlStage{});
      else count(k_bin_count<Src, uint32_t>, lds, HlStage{});
    }
    LOD_LAUNCH(k_bin_colscan, dim3((nt + 255) / 256, L.chunks), dim3(256), 0, st, ucount, nt,
               L.chunks > 1 ? pchunk : tcount);
    if (L.chunks > 1 && !plan_scans)
      LOD_LAUNCH(k_bin_chunkscan, dim3((nt + 255) / 256), dim3(256), 0, st, pchunk, nt, L.chunks, tcount);
  }
  LOD_LAUNCH(k_tile_plan, dim3(1), dim3(PLAN_T), 0, st, any ? tcount : (uint32_t *)nullptr,
             plan_scans ? pchunk : (uint32_t *)nullptr, L.chunks, nt, (int)RecInfo<RecT>::cubic, toff, soff,
             status_word ? (uint64_t *)nullptr : ctr);
  if (any) {
    auto fill = [&](auto kernel, uint32_t g, size_t bytes) {
      LOD_LAUNCH_NAMED("k_bin_fill", kernel, dim3(L.units / g), dim3(BW), bytes, st, src, c, L.units, g, nbits,
                       ucount, pre, toff, soff, stab, L.max_slices, rec, L.max_pairs, status);
    };
    // with cursors in LDS, blocks of two units when there are many (32-bit
    // cursors take twice the LDS of the 16-bit counts: fewer resident waves)
    if constexpr (IsTree<Src>::value) {
      fill(k_bin_fill<Src, RecT, false>, 1u, 0);
    } else {
      if (rows) fill(k_bin_fill<Src, RecT, false>, 1u, 0);
      else fill(k_bin_fill<Src, RecT, true>, L.units >= 4096 ? 2u : 1u, lds);
    }
  }
  const unsigned agrid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(16384, L.max_slices));
  if (any) {
    if constexpr (RecInfo<RecT>::cubic) {
      LOD_LAUNCH(k_accumulate_cubic<RecT>, dim3(agrid), dim3(PT), 0, st, stab, soff, nt, rec, c, partial,
                 partial_aux, L.max_slices, L.max_pairs);
    } else {
      const bool narrow = c.R < 3.98f;   // windows of nine pixels
      auto acc = [&](auto kernel) {
        LOD_LAUNCH_NAMED("k_accumulate", kernel, dim3(agrid), dim3(PT), 0, st, stab, soff, nt, rec, c, partial,
                         partial_aux, L.max_slices, L.max_pairs);
      };
      if (narrow) acc(k_accumulate_narrow<RecT>);
      else acc(k_accumulate_wide<RecT>);
    }
  }
  LOD_LAUNCH(k_finalize, dim3(std::min<uint32_t>(nt, 4096)), dim3(FIN_G * PT), 0, st, soff, nt, partial, c, image,
             L.max_slices);
  if constexpr (RecInfo<RecT>::aux)
    LOD_LAUNCH(k_finalize, dim3(std::min<uint32_t>(nt, 4096)), dim3(FIN_G * PT), 0, st, soff, nt, partial_aux, c,
               image_aux, L.max_slices);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

// Dispatch on the blob kind and on whether an attribute channel is drawn.
template <class Src>
static lod_status splat_any(const Src &src, bool any, const lod_camera &cam, const splat_params &sp, void *ws,
                            const SplatLayout &L, float *image, float *image_aux, uint64_t *status_word,
                            hipStream_t st, const HlStage *hs = nullptr) {
  const bool cubic = sp.blob == LOD_BLOB_CUBIC;
  if constexpr (!IsTree<Src>::value) {   // the LOD render draws no attribute channel
    if (L.aux) {
      if (cubic) return launch_splat_src<Src, RecCA>(src, any, cam, sp, ws, L, image, image_aux, status_word, st, hs);
      return launch_splat_src<Src, RecGA>(src, any, cam, sp, ws, L, image, image_aux, status_word, st, hs);
    }
  }
  if (cubic) return launch_splat_src<Src, RecC>(src, any, cam, sp, ws, L, image, nullptr, status_word, st, hs);
  return launch_splat_src<Src, float3>(src, any, cam, sp, ws, L, image, nullptr, status_word, st, hs);
}

lod_status launch_splat(const float *x, const float *y, const float *z, const float *m, const float *aux,
                        uint64_t count, const lod_camera &cam, const splat_params &sp, void *ws, const SplatLayout &L,
                        float *image, float *image_aux, hipStream_t st) {
  RawSrc src{x, y, z, m, count};
  src.aux = aux;
  return splat_any(src, count > 0, cam, sp, ws, L, image, image_aux, nullptr, st);
}

lod_status launch_splat_interp(const InterpArgs &a, const lod_camera &cam, const splat_params &sp, void *ws,
                               const SplatLayout &L, float *image, float *image_color, hipStream_t st) {
  const InterpSrc src{a.xa, a.ya, a.za, a.ma, a.xb, a.yb, a.zb, a.mb, a.ha, a.hb, a.ca, a.cb, a.count, a.t};
  return splat_any(src, a.count > 0, cam, sp, ws, L, image, image_color, nullptr, st);
}

// Offsets of the listed nodes' points and the number of points drawn.
static void lod_offsets(const lod_tree &tree, const uint32_t *node_ids, const uint64_t *n_ids, uint64_t max_ids,
                        uint64_t *offs, uint64_t *bsum, uint64_t max_points, uint64_t *total, hipStream_t st) {
  LOD_LAUNCH(k_lod_offsets, dim3((unsigned)(max_ids / LOFF + 1)), dim3(LOFF), 0, st, tree, node_ids, n_ids, max_ids,
             offs, bsum);
  LOD_LAUNCH(k_lod_total, dim3(1), dim3(LOFF), 0, st, tree, n_ids, max_ids, bsum, max_points, total);
}

lod_status launch_encode_motion(const lod_tree &tree, const float *xb, const float *yb, const float *zb,
                                const uint64_t *snap_off, int16_t *dqx, int16_t *dqy, int16_t *dqz,
                                uint64_t *saturated, hipStream_t st) {
  fill_u64(saturated, 1, 0, st);
  const unsigned g = (unsigned)std::min<uint64_t>(16384, std::max<uint64_t>(1, tree.node_capacity));
  LOD_LAUNCH(k_encode_motion, dim3(g), dim3(256), 0, st, tree, xb, yb, zb, snap_off, tree.node_capacity, dqx, dqy,
             dqz, saturated);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

lod_status launch_splat_lod_motion(const lod_tree &tree, const uint32_t *node_ids, const uint64_t *n_ids, void *ws,
                                   const LodDrawLayout &D, const int16_t *dqx, const int16_t *dqy,
                                   const int16_t *dqz, float t, const lod_camera &cam, const splat_params &sp,
                                   const SplatLayout &L, float *image, hipStream_t st) {
  char *W = (char *)ws;
  uint64_t *offs = (uint64_t *)(W + D.offs);
  uint64_t *cnt = (uint64_t *)(W + D.count);
  uint64_t *bsum = (uint64_t *)(W + D.bsum);
  lod_offsets(tree, node_ids, n_ids, D.max_ids, offs, bsum, D.max_points, cnt, st);
  TreeMotionSrc src{tree, node_ids, offs, bsum, n_ids, D.max_ids, cnt};
  src.dqx = dqx; src.dqy = dqy; src.dqz = dqz;
  src.t_frame = t;
  return splat_any(src, true, cam, sp, W + D.total, L, image, nullptr, tree.counts + 2, st);
}

lod_status launch_set_points(const lod_tree &tree, uint32_t node, const float *x, const float *y, const float *z,
                             const float *m, uint32_t count, hipStream_t st) {
  if (!count) return LOD_OK;
  const unsigned g = (unsigned)std::min<uint64_t>(1024, (count + 255) / 256);
  LOD_LAUNCH(k_set_points, dim3(g), dim3(256), 0, st, tree, node, x, y, z, m, count);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

lod_status launch_splat_backward(const float *x, const float *y, const float *z, const float *m, uint64_t count,
                                 const lod_camera &cam, const splat_params &sp, const float *grad, float *gm,
                                 float *gx, float *gy, float *gz, hipStream_t st) {
  if (!count) return LOD_OK;
  Cam c = make_cam(cam, sp, nullptr);
  const unsigned grid = (unsigned)std::min<uint64_t>(65535, (count + PT - 1) / PT);
  // up to nine pixels: a thread a point (1 M and 3 M points, four lanes a point ->
  // a thread: h = 0.6 25 -> 17 and 56 -> 38 us, 1 28 -> 24 and 63 -> 56, 1.25 36
  // -> 33 and 84 -> 81; but 1.5 40 -> 42 and 93 -> 103, 2.5 67 -> 99)
  if (sp.blob == LOD_BLOB_CUBIC && c.Fhw == 0.0f && c.hpx <= 1.25f)
    LOD_LAUNCH(k_backward_cubic_small, dim3(grid), dim3(PT), 0, st, x, y, z, m, count, c, grad, gm, gx, gy, gz);
  else if (sp.blob == LOD_BLOB_CUBIC)
    LOD_LAUNCH(k_backward_cubic, dim3(grid), dim3(PT), 0, st, x, y, z, m, count, c, grad, gm, gx, gy, gz);
  else
    LOD_LAUNCH(k_backward, dim3(grid), dim3(PT), 0, st, x, y, z, m, count, c, grad, gm, gx, gy, gz);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

LodDrawLayout lod_draw_layout(uint64_t node_capacity, uint64_t max_points) {
  LodDrawLayout L{};
  L.max_ids = std::max<uint64_t>(1, node_capacity);
  L.max_points = std::max<uint64_t>(1, max_points);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  L.offs = take(8 * (L.max_ids + 1));
  L.bsum = take(8 * (L.max_ids / LOFF + 1));
  L.count = take(64);
  L.total = off;
  return L;
}

HlLayout hl_layout(const SplatLayout &L, uint64_t max_highlighted, const lod_camera &cam, const splat_params &sp,
                   lod_status &s) {
  HlLayout H{};
  H.cap = std::max<uint64_t>(1, max_highlighted);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  for (int a = 0; a < 4; ++a) H.stage[a] = take(4 * L.max_points);
  H.count = take(8 * (size_t)L.units);
  H.scan = take(8 * ((size_t)L.units + 1));
  H.scan_tmp = take(8 * scan_tmp_elems<uint64_t>((uint64_t)L.units + 1));
  H.total_ctr = take(64);
  for (int a = 0; a < 4; ++a) H.pts[a] = take(4 * H.cap);
  s = splat_layout(H.cap, cam, sp, H.L2, false);
  H.splat = off;
  H.total = off + H.L2.total;
  return H;
}

lod_status launch_hl_flags(const lod_tree &tree, const uint32_t *bits, uint64_t n_bits, uint32_t *flags,
                           hipStream_t st) {
  const uint64_t groups = (tree.point_capacity + 63) / 64;
  const unsigned g = (unsigned)std::min<uint64_t>(65535, std::max<uint64_t>(1, (groups + 3) / 4));
  LOD_LAUNCH(k_hl_flags, dim3(g), dim3(256), 0, st, tree, bits, n_bits, tree.point_capacity, flags);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

lod_status launch_splat_lod(const lod_tree &tree, const uint32_t *node_ids, const uint64_t *n_ids, void *ws,
                            const LodDrawLayout &D, const lod_camera &cam, const splat_params &sp,
                            const SplatLayout &L, const uint32_t *hl_flags, const HlLayout *H,
                            float *image, float *image_hl, hipStream_t st) {
  char *W = (char *)ws;
  uint64_t *offs = (uint64_t *)(W + D.offs);
  uint64_t *cnt = (uint64_t *)(W + D.count);
  uint64_t *bsum = (uint64_t *)(W + D.bsum);
  lod_offsets(tree, node_ids, n_ids, D.max_ids, offs, bsum, D.max_points, cnt, st);
  TreeSrc src{tree, node_ids, offs, bsum, n_ids, D.max_ids, cnt};
  if (!H) return splat_any(src, true, cam, sp, W + D.total, L, image, nullptr, tree.counts + 2, st);
  // ID highlighting: the count pass of the main render tests every drawn
  // point's flag and stages the flagged ones; they are gathered in unit
  // order and drawn by a second, small render
  src.hl_flags = hl_flags;
  src.hl_words = (tree.point_capacity + 63) / 64 * 2;
  char *HW = W + D.total + L.total;
  HlStage hs{(float *)(HW + H->stage[0]), (float *)(HW + H->stage[1]), (float *)(HW + H->stage[2]),
             (float *)(HW + H->stage[3]), (uint64_t *)(HW + H->count), (uint64_t *)(HW + H->scan)};
  fill_u64(hs.scan + L.units, 1, 0, st);
  lod_status s = splat_any(src, true, cam, sp, W + D.total, L, image, nullptr, tree.counts + 2, st, &hs);
  if (s != LOD_OK) return s;
  device_scan<uint64_t>(hs.scan, (uint64_t)L.units + 1, (uint64_t *)(HW + H->scan_tmp), st);
  float *px = (float *)(HW + H->pts[0]), *py = (float *)(HW + H->pts[1]);
  float *pz = (float *)(HW + H->pts[2]), *pm = (float *)(HW + H->pts[3]);
  uint64_t *hl_total = (uint64_t *)(HW + H->total_ctr);
  LOD_LAUNCH(k_hl_gather, dim3(L.units), dim3(256), 0, st, hs, (const uint64_t *)hs.scan, (const uint64_t *)cnt,
             D.max_points, L.units, px, py, pz, pm, H->cap, hl_total, tree.counts + 2);
  RawSrc hsrc{px, py, pz, pm, H->cap};
  hsrc.n_dev = hl_total;
  return splat_any(hsrc, true, cam, sp, HW + H->splat, H->L2, image_hl, nullptr, tree.counts + 2, st);
}

size_t decode_workspace(uint64_t node_capacity) {
  const uint64_t n = std::max<uint64_t>(1, node_capacity);
  return align256(8 * (n + 1)) + align256(8 * (n / LOFF + 1));
}

lod_status launch_decode(const lod_tree &tree, const uint32_t *node_ids, const uint64_t *n_ids, uint64_t max_points,
                         float *x, float *y, float *z, float *m, uint64_t *n_points, void *ws, hipStream_t st) {
  const uint64_t max_ids = std::max<uint64_t>(1, tree.node_capacity);
  char *W = (char *)ws;
  uint64_t *offs = (uint64_t *)W;
  uint64_t *bsum = (uint64_t *)(W + align256(8 * (max_ids + 1)));
  lod_offsets(tree, node_ids, n_ids, max_ids, offs, bsum, max_points, n_points, st);
  const unsigned dg = (unsigned)std::min<uint64_t>(16384, max_ids);
  LOD_LAUNCH(k_lod_decode, dim3(dg), dim3(PT), 0, st, tree, node_ids, n_ids, max_ids, offs, bsum, max_points, x, y, z, m);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

size_t cut_workspace(uint64_t node_capacity) {
  const uint64_t n = std::max<uint64_t>(1, node_capacity) + 1;
  return align256(4 * n) + align256(4 * ((n + CUT_T - 1) / CUT_T));
}

lod_status launch_cut(const lod_tree &tree, const lod_camera &cam, float tau_px, uint32_t n, uint32_t *node_ids,
                      uint64_t cap, uint64_t *n_selected, void *ws, hipStream_t st) {
  const uint64_t nc = std::max<uint64_t>(1, tree.node_capacity);
  char *W = (char *)ws;
  uint32_t *keep = (uint32_t *)W;
  uint32_t *sums = (uint32_t *)(W + align256(4 * (nc + 1)));
  CutArgs c{};
  c.proj = cam.projection; c.W = cam.W;
  c.px = (double)cam.pos[0]; c.py = (double)cam.pos[1]; c.pz = (double)cam.pos[2];
  c.F = (double)cam.F;
  c.tau_cbrt = (double)tau_px * std::cbrt((double)n);
  const unsigned g = (unsigned)((nc + CUT_T - 1) / CUT_T);
  LOD_LAUNCH(k_cut_flags, dim3(g), dim3(CUT_T), 0, st, tree, c, nc, keep, sums);
  LOD_LAUNCH(k_cut_write, dim3(g), dim3(CUT_T), 0, st, tree, nc, keep, sums, node_ids, cap, n_selected);
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

}  // namespace lodh
