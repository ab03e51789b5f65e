// Octree level-of-detail build for gfx950 (octree and quantisation
// paragraphs of arXiv:0811.2055; readings fixed in the oracle's docstrings).
//
// Data path (all device-resident, one stream, no host synchronisation):
//   keygen     domain check and digit-0 tile histograms of the sort key
//              (snapshot | 3D-bit Morton); the first scatter pass recomputes
//              the key and the 48-bit fraction from x, y, z
//   radix sort stable LSD, 8-bit digits, reduce-then-scan: per-tile digit
//              histograms, one device scan, scatter with wave-ballot ranks and
//              LDS-staged coalesced writes; payload (id, fraction, mass) rides
//              along so nothing is gathered at random afterwards
//   density    run lengths of equal depth-L cells (block max/min scans), then
//              Philox U and the 12-bit bin of the integer selection key K per
//              sorted position (on a second stream, beside the tree)
//   tree       the first levels by one block; then level by level: octant
//              boundaries by a nine-way search of eight lanes per octant, and
//              the next level written with one thread per (node, octant)
//   leaves     float64 leaf masses; the per-level schedule copies the leaves'
//              particles inside its selection launches
//   selection  bottom up, per node holding > n: the node's float64 mass from
//              its children, the (n+1)-th smallest (K, id) over the children's
//              top lists or own range (key-bin histogram, exact keys only in
//              the threshold bin), then an order-preserving compaction;
//              float64 renormalisation, 16-bit quantisation and output
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "lod.h"
#include "lod_device.hpp"
#include "lod_internal.hpp"
#include "lod_scan.hpp"

using namespace lodk;

namespace {

constexpr int TB = 256;          // threads per block for streaming kernels
constexpr int ITEMS = 16;        // elements per thread
constexpr int TILE = TB * ITEMS; // elements per density tile (4096)

// radix sort tiles: scatter blocks of STB threads x SITEMS elements; the
// histogram kernels (TB threads) cover the same STILE elements per block.
// 512-thread scatter blocks take 43 KB of LDS, so two run on a CU and one's
// ranking overlaps the other's stores (1024 threads and 84 KB: one block per
// CU, 2.5% slower build).
constexpr int STB = 512;                     // scatter threads per block
constexpr int SITEMS = 8;                    // elements per scatter thread
constexpr int STILE = STB * SITEMS;          // elements per sort tile
constexpr int HITEMS = STILE / TB;           // elements per histogram thread
constexpr int HCHUNK = 8;                    // loads issued together in keygen (twice that in upsweep)
static_assert(HITEMS % (2 * HCHUNK) == 0, "histogram chunks must divide the tile");
constexpr int RADIX = 256;
constexpr uint32_t STATUS_INTERNAL = 8u;

// ---------------------------------------------------------------------------
// parameters passed by value to kernels

struct BuildArgs {
  uint64_t N;
  uint32_t n;
  int D;
  int shift_rho;       // 3 (D - L)
  int alpha;
  uint64_t seed;
  uint32_t n_snap;
  const uint64_t *snap_off;   // device [n_snap+1] or null
  uint64_t node_cap, point_cap;
  uint64_t *counts;           // device [3]
};

__device__ __forceinline__ uint32_t snapshot_of(const BuildArgs &a, uint64_t e) {
  if (a.n_snap <= 1 || !a.snap_off) return 0;
  // largest s with snap_off[s] <= e
  uint32_t lo = 0, hi = a.n_snap;   // answer in [0, n_snap)
  while (hi - lo > 1) {
    uint32_t mid = (lo + hi) >> 1;
    if (a.snap_off[mid] <= e) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint64_t local_id(const BuildArgs &a, uint32_t snap, uint32_t gidx) {
  return (a.n_snap <= 1 || !a.snap_off) ? (uint64_t)gidx : (uint64_t)gidx - a.snap_off[snap];
}

// ---------------------------------------------------------------------------
// Start of a build, one launch: the status and counts cleared (before any kernel
// that sets a bit), the snapshot offsets checked by the block that cleared
// them, and the zeroed part of the workspace (levels, leaf-copy cursors,
// totals of the tree's levels).

__global__ __launch_bounds__(256) void k_build_init(BuildArgs a, uint32_t *__restrict__ zero, uint64_t n_zero) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_zero;
       i += (uint64_t)gridDim.x * blockDim.x)
    zero[i] = 0u;
  if (blockIdx.x) return;
  if (threadIdx.x < 3) a.counts[threadIdx.x] = 0;
  if (!a.snap_off || a.n_snap <= 1 || a.N == 0) return;   // no particles: no offsets are read
  __syncthreads();
  bool bad = false;
  for (uint32_t s = threadIdx.x; s < a.n_snap; s += blockDim.x) {
    uint64_t lo = a.snap_off[s], hi = a.snap_off[s + 1];
    if (hi < lo || hi - lo >= (1ull << 31)) bad = true;
  }
  if (threadIdx.x == 0 && (a.snap_off[0] != 0 || a.snap_off[a.n_snap] != a.N)) bad = true;
  if (__syncthreads_or(bad) && threadIdx.x == 0) a.counts[2] = LOD_STATUS_OFFSETS;
}

// ---------------------------------------------------------------------------
// sort key and 48-bit fraction of particle e.  Both the keygen histogram and
// the first scatter pass call this, so their digits agree bit for bit (NaN and
// out-of-range coordinates map to 0 and are reported by keygen's check).

struct PKey {
  uint32_t key;
  uint64_t lo;
  bool ok;
};

__device__ __forceinline__ PKey particle_key(const BuildArgs &a, float xe, float ye, float ze, float me,
                                             uint64_t e) {
  uint32_t X, Y, Z;
  bool ok = fixed_coord(xe, a.D, X);
  ok &= fixed_coord(ye, a.D, Y);
  ok &= fixed_coord(ze, a.D, Z);
  ok &= (me >= 0.0f) && (me <= 3.4028235e38f);
  const uint32_t cmask = (1u << a.D) - 1u;
  const uint32_t cx = (X >> 16) & cmask, cy = (Y >> 16) & cmask, cz = (Z >> 16) & cmask;
  uint32_t k = spread3(cx) | (spread3(cy) << 1) | (spread3(cz) << 2);
  if (a.n_snap > 1) k |= (uint32_t)(((uint64_t)snapshot_of(a, e) << (3 * a.D)) & 0xFFFFFFFFull);
  const uint64_t lo = (uint64_t)(X & 0xFFFFu) | ((uint64_t)(Y & 0xFFFFu) << 16) | ((uint64_t)(Z & 0xFFFFu) << 32);
  return PKey{k, lo, ok};
}

// keygen: domain check and digit-0 tile histograms (reads the input only; the
// first scatter pass recomputes the keys instead of reading them back)
__global__ __launch_bounds__(TB) void k_keygen(const float *__restrict__ x, const float *__restrict__ y,
                                               const float *__restrict__ z, BuildArgs a, uint32_t *__restrict__ thist,
                                               uint64_t n_tiles) {
  __shared__ uint32_t hist[RADIX];
  __shared__ int bad;
  for (int i = threadIdx.x; i < RADIX; i += TB) hist[i] = 0;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  const uint64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  bool my_bad = false;
  // all loads first (clamped indices: a predicated load is waited for alone)
  for (int c = 0; c < HITEMS; c += HCHUNK) {
    float xs[HCHUNK], ys[HCHUNK], zs[HCHUNK];
#pragma unroll
    for (int i = 0; i < HCHUNK; ++i) {
      const uint64_t e = min(tile * STILE + (uint64_t)(c + i) * TB + threadIdx.x, a.N - 1);
      xs[i] = x[e]; ys[i] = y[e]; zs[i] = z[e];
    }
#pragma unroll
    for (int i = 0; i < HCHUNK; ++i) {
      const uint64_t e = tile * STILE + (uint64_t)(c + i) * TB + threadIdx.x;
      if (e < a.N) {
        // positions only: the masses are checked by the first scatter pass
        const PKey pk = particle_key(a, xs[i], ys[i], zs[i], 0.0f, e);
        my_bad |= !pk.ok;
        atomicAdd(&hist[pk.key & 0xFFu], 1u);
      }
    }
  }
  if (my_bad) bad = 1;
  __syncthreads();
  for (int i = threadIdx.x; i < RADIX; i += TB) thist[(uint64_t)i * n_tiles + tile] = hist[i];
  if (threadIdx.x == 0 && bad)
    atomicOr((unsigned long long *)&a.counts[2], (unsigned long long)LOD_STATUS_DOMAIN);
}

// per-tile digit histogram for passes after the first
__global__ __launch_bounds__(TB) void k_upsweep(const uint32_t *__restrict__ key, uint64_t N, int shift,
                                                uint32_t *__restrict__ thist, uint64_t n_tiles) {
  __shared__ uint32_t hist[RADIX];
  for (int i = threadIdx.x; i < RADIX; i += TB) hist[i] = 0;
  __syncthreads();
  const uint64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  for (int c = 0; c < HITEMS; c += 2 * HCHUNK) {
    uint32_t ks[2 * HCHUNK];
#pragma unroll
    for (int i = 0; i < 2 * HCHUNK; ++i)
      ks[i] = key[min(tile * STILE + (uint64_t)(c + i) * TB + threadIdx.x, N - 1)];
#pragma unroll
    for (int i = 0; i < 2 * HCHUNK; ++i)
      if (tile * STILE + (uint64_t)(c + i) * TB + threadIdx.x < N) atomicAdd(&hist[(ks[i] >> shift) & 0xFFu], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < RADIX; i += TB) thist[(uint64_t)i * n_tiles + tile] = hist[i];
}

// Stable scatter of one LSD pass over STILE-element tiles, STB threads.  Wave
// w of the block owns tile elements [w*P, (w+1)*P) with P = STILE / waves; in
// round r lane l holds element w*P + r*64 + l, so element order is (w, r, l).
// All loads of a thread's SITEMS elements are issued first, so their latency
// overlaps the ranking.
// Ranks within a wave come from 8 ballots (the lanes sharing the digit) and a
// wave-private LDS counter per digit; the tile is staged in LDS in digit order
// so that the global writes of each digit run are contiguous.

// FIRST: the input is the particles themselves (x, y, z, m with ids implicit);
// keys and fractions come from particle_key.  Otherwise (key, id, fraction,
// mass) arrays of the previous pass.
// The fractions ride the sort as 6 bytes per particle: x and y's 16 bits in
// a 32-bit array, z's in a 16-bit one (18-byte records instead of 20).
struct ScatterIn {
  const uint32_t *key, *idx;
  const uint32_t *lo;
  const uint16_t *lz;
  const float *x, *y, *z, *m;
};

template <bool FIRST>
__global__ __launch_bounds__(STB) void k_scatter(BuildArgs a, int shift, const uint32_t *__restrict__ thist,
                                                 const uint32_t *__restrict__ tsum, uint64_t n_tiles, ScatterIn in,
                                                 uint32_t *__restrict__ key_out, uint32_t *__restrict__ idx_out,
                                                 uint32_t *__restrict__ lo_out, uint16_t *__restrict__ lz_out,
                                                 float *__restrict__ m_out) {
  const uint64_t N = a.N;
  constexpr int NW = STB / WAVE;              // waves per block
  constexpr int PER_WAVE = STILE / NW;
  constexpr int ROUNDS = PER_WAVE / WAVE;     // 8
  __shared__ uint32_t wcnt[NW][RADIX];
  __shared__ uint32_t bin_start[RADIX];       // tile-local start of each digit
  __shared__ uint32_t gofs[RADIX];            // global start of this tile's digit run
  __shared__ uint64_t stage[STILE];
  __shared__ uint32_t tmp[STB / WAVE + 1];

  const int lane = threadIdx.x & (WAVE - 1);
  const int w = threadIdx.x / WAVE;
  const uint64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t tbase = tile * STILE;
  const uint64_t ebase = tbase + (uint64_t)w * PER_WAVE + lane;
  // this tile's global digit offsets (the scan of the digit-major counts: a
  // 4096-count block's own scan plus the scanned block totals), loaded first
  // (every thread, clamped index) so that waiting for them does not wait for
  // the element loads
  const uint64_t hi = (uint64_t)min((int)threadIdx.x, RADIX - 1) * n_tiles + tile;
  const uint32_t g0 = thist[hi] + tsum[hi / SCAN_TILE];
  uint32_t kk[ROUNDS], ii[ROUNDS];
  uint64_t ll[ROUNDS];
  float mm[ROUNDS];
  if (FIRST) {
    // every load of the thread first (the key computation branches on the
    // snapshot count, and a load issued after a branch waits for it)
    float xs[ROUNDS], ys[ROUNDS], zs[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      // clamped, unconditional loads; lanes past N are masked out below
      const uint64_t e = min(ebase + (uint64_t)r * WAVE, N - 1);
      xs[r] = in.x[e]; ys[r] = in.y[e]; zs[r] = in.z[e]; mm[r] = in.m[e];
    }
    bool bad_mass = false;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint64_t e = min(ebase + (uint64_t)r * WAVE, N - 1);
      const PKey pk = particle_key(a, xs[r], ys[r], zs[r], mm[r], e);
      kk[r] = pk.key;
      ll[r] = pk.lo;
      ii[r] = (uint32_t)(ebase + (uint64_t)r * WAVE);
      // keygen checked the positions; the masses are checked here
      bad_mass |= ebase + (uint64_t)r * WAVE < N && !(mm[r] >= 0.0f && mm[r] <= 3.4028235e38f);
    }
    if (bad_mass) atomicOr((unsigned long long *)&a.counts[2], (unsigned long long)LOD_STATUS_DOMAIN);
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint64_t e = min(ebase + (uint64_t)r * WAVE, N - 1);
      kk[r] = in.key[e];
      ii[r] = in.idx[e];
      ll[r] = (uint64_t)in.lo[e] | ((uint64_t)in.lz[e] << 32);
      mm[r] = in.m[e];
    }
  }
  for (int i = threadIdx.x; i < NW * RADIX; i += STB) (&wcnt[0][0])[i] = 0;
  if (threadIdx.x < RADIX) gofs[threadIdx.x] = g0;
  __syncthreads();

  const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (WAVE - lane));
  uint32_t dig[ROUNDS];
  uint32_t rnk[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool valid = ebase + (uint64_t)r * WAVE < N;
    const uint32_t d = (kk[r] >> shift) & 0xFFu;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t bal = __ballot((d >> b) & 1u);
      peers &= ((d >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
    const uint32_t cnt = (uint32_t)__popcll(peers);
    const uint32_t old = valid ? wcnt[w][d] : 0u;
    if (valid && below == 0) wcnt[w][d] = old + cnt;
    dig[r] = d;
    rnk[r] = old + below;
  }
  // The payload loads have landed during the ranking: wait for them here,
  // before any store is issued.  Loads and stores share one counter, so a
  // wait placed where the values are first used would also wait for the
  // stores of the fields written before.  (Encoding: vmcnt 0, expcnt and
  // lgkmcnt left at their maxima.)
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  // per digit: wave prefix (in place) and tile total
  uint32_t tot = 0;
  if (threadIdx.x < RADIX) {
    const int d = threadIdx.x;
    for (int ww = 0; ww < NW; ++ww) {
      const uint32_t c = wcnt[ww][d];
      wcnt[ww][d] = tot;
      tot += c;
    }
  }
  uint32_t dummy;
  const uint32_t st = block_excl_scan<uint32_t>(threadIdx.x < RADIX ? tot : 0u, tmp, dummy);
  if (threadIdx.x < RADIX) bin_start[threadIdx.x] = st;
  __syncthreads();

  uint32_t slot[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) slot[r] = bin_start[dig[r]] + wcnt[w][dig[r]] + rnk[r];
  const uint32_t tile_n = (uint32_t)min((uint64_t)STILE, N - tbase);

  // keys (with their output positions), then ids, fractions, masses.  LDS
  // reads are unconditional (slots past the tile hold stale values) and
  // issued together; only the stores are predicated.
  uint64_t gpos[SITEMS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (ebase + (uint64_t)r * WAVE < N) stage[slot[r]] = kk[r];
  __syncthreads();
  {
    uint32_t k[SITEMS], go[SITEMS], bs[SITEMS];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) k[i] = (uint32_t)stage[i * STB + threadIdx.x];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) {
      const uint32_t d = (k[i] >> shift) & 0xFFu;
      go[i] = gofs[d];
      bs[i] = bin_start[d];
    }
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) {
      const uint32_t s = (uint32_t)i * STB + threadIdx.x;
      gpos[i] = (uint64_t)go[i] + (s - bs[i]);
      if (s < tile_n) key_out[gpos[i]] = k[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (ebase + (uint64_t)r * WAVE < N) stage[slot[r]] = ii[r];
  __syncthreads();
  {
    uint32_t v[SITEMS];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) v[i] = (uint32_t)stage[i * STB + threadIdx.x];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i)
      if ((uint32_t)i * STB + threadIdx.x < tile_n) idx_out[gpos[i]] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (ebase + (uint64_t)r * WAVE < N) stage[slot[r]] = ll[r];
  __syncthreads();
  {
    uint64_t v[SITEMS];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) v[i] = stage[i * STB + threadIdx.x];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i)
      if ((uint32_t)i * STB + threadIdx.x < tile_n) {
        lo_out[gpos[i]] = (uint32_t)v[i];
        lz_out[gpos[i]] = (uint16_t)(v[i] >> 32);
      }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (ebase + (uint64_t)r * WAVE < N) stage[slot[r]] = (uint64_t)__float_as_uint(mm[r]);
  __syncthreads();
  {
    uint32_t v[SITEMS];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i) v[i] = (uint32_t)stage[i * STB + threadIdx.x];
#pragma unroll
    for (int i = 0; i < SITEMS; ++i)
      if ((uint32_t)i * STB + threadIdx.x < tile_n) m_out[gpos[i]] = __uint_as_float(v[i]);
  }
}

// ---------------------------------------------------------------------------
// density (run length of equal depth-L cells) and selection keys

template <bool MAXOP>
__device__ __forceinline__ uint32_t block_incl_scan_op(uint32_t v, uint32_t *tmp) {
  // inclusive max- or min-scan over threads in index order
  const int lane = threadIdx.x & (WAVE - 1);
  const int wid = threadIdx.x / WAVE;
  const int nw = blockDim.x / WAVE;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    uint32_t t = __shfl_up(v, o, WAVE);
    if (lane >= o) v = MAXOP ? max(v, t) : min(v, t);
  }
  if (lane == WAVE - 1) tmp[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = MAXOP ? 0u : ~0u;
    for (int ww = 0; ww < nw; ++ww) {
      uint32_t t = tmp[ww];
      tmp[ww] = run;
      run = MAXOP ? max(run, t) : min(run, t);
    }
  }
  __syncthreads();
  uint32_t pre = tmp[wid];
  __syncthreads();
  return MAXOP ? max(pre, v) : min(pre, v);
}

// Blocked layout: thread t owns tile elements [t*ITEMS, t*ITEMS+ITEMS).  A
// run's start is the largest run-start position at or before an element, its
// end the smallest run-end position after it; both come from a thread-local
// pass plus a block scan, and runs crossing the tile edge are closed by a
// binary search over the sorted keys.  The LDS arrays hold word i at
// i + i/16: blocked accesses (thread t at 16 t + k) would otherwise put a
// wave's lanes on four banks.  Bound by vector issue: the generator's ten
// rounds are about half of a particle's instructions (14 bytes of traffic take
// half of the time at the rate of a copy).  Its exclusive ors of three words
// are single instructions; run starts and ends share a word and scan in 32
// bits; a batch of snapshots has its own instance: 150 M particles 913 -> 836
// us, 60 M in 32 snapshots 468 -> 399.  Five waves per SIMD instead of four
// spill and give nothing (874).
constexpr int DPAD = (TILE + 2) / 16 + 1;
__device__ __forceinline__ int dpad(int i) { return i + (i >> 4); }
template <bool MULTI>
__global__ __launch_bounds__(TB) void k_density(BuildArgs a, const uint32_t *__restrict__ skey,
                                                const uint32_t *__restrict__ sidx,
                                                uint32_t *__restrict__ w_out, uint16_t *__restrict__ kb_out) {
  __shared__ uint32_t cell[TILE + 2 + DPAD];   // cell[dpad(i+1)] = cell of element base+i
  __shared__ uint32_t tmp[TB / WAVE + 1];
  __shared__ uint32_t incl_max[TB];
  __shared__ uint32_t rev_min[TB];
  __shared__ uint64_t first_start, last_end;
  const uint64_t N = a.N;
  const uint64_t base = (uint64_t)blockIdx.x * TILE;
  const uint32_t tile_n = (uint32_t)min((uint64_t)TILE, N - base);
  const int sh = a.shift_rho;
  {
    // clamped, unconditional loads first, then the selects
    constexpr int CI = (TILE + 2 + TB - 1) / TB;
    uint32_t kc[CI];
    const uint32_t first = base ? 0u : 1u;             // word 0 is element base - 1
    const uint32_t *kp = skey + (base ? base - 1 : 0);
    const uint32_t last = (uint32_t)min((uint64_t)TILE + 1, N - base) - first;
#pragma unroll
    for (int j = 0; j < CI; ++j) kc[j] = kp[min((uint32_t)max(j * TB + (int)threadIdx.x, (int)first) - first, last)];
#pragma unroll
    for (int j = 0; j < CI; ++j) {
      const int i = j * TB + (int)threadIdx.x;
      const int64_t e = (int64_t)base + i - 1;
      if (i < TILE + 2)
        cell[dpad(i)] = (e >= 0 && (uint64_t)e < N && i <= (int)tile_n + 1) ? (kc[j] >> sh) : 0xFFFFFFFFu;
    }
  }
  __syncthreads();
  const bool has_prev = base > 0;
  const bool has_next = base + tile_n < N;
  if (threadIdx.x == 0) {
    // runs crossing the tile edges: galloping search outward from the edge
    uint64_t s0 = base;
    if (has_prev && cell[dpad(0)] == cell[dpad(1)]) {
      const uint32_t c = cell[dpad(1)];
      uint64_t right = base, step = 1, lo = 0;
      while (true) {
        if (right < step) { lo = 0; break; }
        const uint64_t probe = right - step;
        if ((skey[probe] >> sh) < c) { lo = probe + 1; break; }
        right = probe;
        step <<= 1;
      }
      uint64_t l = lo, h = right;
      while (l < h) {
        const uint64_t mid = l + ((h - l) >> 1);
        if ((skey[mid] >> sh) < c) l = mid + 1; else h = mid;
      }
      s0 = l;
    }
    first_start = s0;
    uint64_t e0 = base + tile_n;
    if (has_next && cell[dpad(tile_n)] == cell[dpad(tile_n + 1)]) {
      const uint32_t c = cell[dpad(tile_n)];
      uint64_t known = base + tile_n - 1, step = 1, hi = N;
      while (true) {
        const uint64_t probe = known + step;
        if (probe >= N) { hi = N; break; }
        if ((skey[probe] >> sh) > c) { hi = probe; break; }
        known = probe;
        step <<= 1;
      }
      uint64_t l = known + 1, h = hi;
      while (l < h) {
        const uint64_t mid = l + ((h - l) >> 1);
        if ((skey[mid] >> sh) <= c) l = mid + 1; else h = mid;
      }
      e0 = l;
    }
    last_end = e0;
  }
  __syncthreads();
  const int t0 = threadIdx.x * ITEMS;
  // Positions within the tile are kept as 32-bit local offsets: a run start
  // as li + 1 (0: the run began before the tile, at first_start); a run end
  // as li + 1 < tile_n, or tile_n for the tile's last run (which ends at
  // last_end).
  // run starts: thread-local running max
  uint32_t se[ITEMS];                        // start | end << 16
  uint32_t runmax = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int li = t0 + i;
    const bool starts =
        (li == 0) ? (!has_prev || cell[dpad(0)] != cell[dpad(1)]) : (cell[dpad(li)] != cell[dpad(li + 1)]);
    if (li < (int)tile_n && starts) runmax = (uint32_t)li + 1;
    se[i] = runmax;
  }
  incl_max[threadIdx.x] = block_incl_scan_op<true>(runmax, tmp);
  // run ends: thread-local suffix min
  static_assert(TILE < 0xFFFF, "run starts and ends fit 16 bits");
  uint32_t runmin = 0xFFFFu;
#pragma unroll
  for (int i = ITEMS - 1; i >= 0; --i) {
    const int li = t0 + i;
    if (li < (int)tile_n) {
      if (li == (int)tile_n - 1) runmin = tile_n;
      else if (cell[dpad(li + 1)] != cell[dpad(li + 2)]) runmin = min(runmin, (uint32_t)li + 1);
    }
    se[i] |= runmin << 16;
  }
  __syncthreads();
  // suffix over threads: thread t scans the value of thread TB-1-t
  rev_min[threadIdx.x] = runmin;
  __syncthreads();
  const uint32_t mirrored = rev_min[TB - 1 - threadIdx.x];
  __syncthreads();
  rev_min[threadIdx.x] = block_incl_scan_op<false>(mirrored, tmp);
  __syncthreads();
  const uint32_t prev_max = threadIdx.x ? incl_max[threadIdx.x - 1] : 0u;
  // min over threads > t == reversed inclusive scan at position TB-2-t
  const uint32_t next_min = (threadIdx.x < TB - 1) ? rev_min[TB - 2 - threadIdx.x] : 0xFFFFu;
  const uint64_t fs = first_start, le = last_end;
  // run lengths, blocked -> LDS, then striped (coalesced) keys, ids and outputs
  uint32_t *wl = (uint32_t *)cell;           // cell[] is no longer needed; reuse it
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int li = t0 + i;
    if (li < (int)tile_n) {
      const uint32_t sl = max(se[i] & 0xFFFFu, prev_max), el = min(se[i] >> 16, next_min);
      const uint64_t sg = sl ? base + sl - 1 : fs;
      const uint64_t eg = (el == tile_n) ? le : base + el;
      wl[dpad(li)] = (uint32_t)(eg - sg);
    }
  }
  __syncthreads();
  const int sdb = 3 * a.D;
  constexpr int DCH = 8;                     // ids loaded together
  const uint32_t *ip = sidx + base, *sp = skey + base;
  uint32_t *wp = w_out + base;
  uint16_t *bp = kb_out + base;
#pragma unroll
  for (int c = 0; c < ITEMS; c += DCH) {
    uint32_t ids[DCH], snaps[DCH];
#pragma unroll
    for (int i = 0; i < DCH; ++i) {
      ids[i] = ip[min((uint32_t)((c + i) * TB + threadIdx.x), tile_n - 1)];
      snaps[i] = 0u;
    }
    if (MULTI) {
#pragma unroll
      for (int i = 0; i < DCH; ++i)
        snaps[i] = (uint32_t)((uint64_t)sp[min((uint32_t)((c + i) * TB + threadIdx.x), tile_n - 1)] >> sdb);
    }
    uint32_t exact = 0;                      // items whose bin needs the exact key (rare)
#pragma unroll
    for (int i = 0; i < DCH; ++i) {
      const uint32_t li = (c + i) * TB + threadIdx.x;
      if (li < tile_n) {
        const uint32_t w = wl[dpad(li)];
        // one snapshot: the counter's words 1-3 are zero, which folds the
        // first round's second product
        const uint64_t U = MULTI ? particle_U(local_id(a, snaps[i], ids[i]), snaps[i], a.seed)
                                        : (uint64_t)philox_word0(ids[i], 0u, 0u, 0u, (uint32_t)a.seed,
                                                                 (uint32_t)(a.seed >> 32)) + 1ull;
        wp[li] = w;
        uint32_t bin;
        if (a.alpha <= 0) bin = kbin(selection_key(U, w, a.alpha));
        else if (!kbin_div_fast(U, w, bin)) exact |= 1u << i;
        if (!((exact >> i) & 1u)) bp[li] = (uint16_t)bin;
      }
    }
    // one copy of the exact path, entered by few lanes
    while (exact) {
      const int i = __ffs(exact) - 1;
      exact &= exact - 1u;
      const int li = (c + i) * TB + threadIdx.x;
      const uint64_t e = base + li;
      const uint32_t snap = MULTI ? (uint32_t)((uint64_t)skey[e] >> sdb) : 0u;
      const uint64_t U = particle_U(local_id(a, snap, sidx[e]), snap, a.seed);
      kb_out[e] = (uint16_t)kbin(div_u2p31(U, wl[dpad(li)]));
    }
  }
}

// ---------------------------------------------------------------------------
// tree, level by level

struct TreeArgs {
  uint64_t *prefix;
  uint8_t *depth;
  uint32_t *parent;
  uint32_t *first_child;
  uint8_t *child_mask;
  uint64_t *part_begin;
  uint64_t *part_count;
  uint64_t *pt_begin;
  uint32_t *pt_count;
  double *node_mass;
  uint32_t *pt_id;
  uint16_t *qx, *qy, *qz;
  float *pt_mass;
  // workspace
  uint32_t *lvl;      // [D+3] level starts; lvl[d+1] = end of level d
  uint32_t *cs;       // [node_cap * 9] octant starts (sorted positions) of internal nodes
  uint32_t *sel_idx;  // [node_cap] rank among all selecting nodes (levels in order), or NONE
  uint32_t *sel_node; // [node_cap] node of each selecting rank (NONE if it was not emitted)
  uint32_t *wit;      // [node_cap] witness sorted position, or NONE
  uint32_t *pend;     // [node_cap] number of selecting children not yet reduced
  uint32_t *lsel;     // [D+3] selecting nodes at levels < d (cumulative)
};

__device__ __forceinline__ void set_status(const BuildArgs &a, uint32_t bits) {
  atomicOr((unsigned long long *)&a.counts[2], (unsigned long long)bits);
}

// Roots: one per non-empty snapshot (one block of 1024).
__device__ void make_roots(const BuildArgs &a, const TreeArgs &t, const uint32_t *__restrict__ skey) {
  __shared__ uint32_t tmp[1024 / WAVE + 1];
  __shared__ uint32_t base_nodes, base_sel;
  if (threadIdx.x == 0) { base_nodes = 0; base_sel = 0; t.lvl[0] = 0; t.lsel[0] = 0; }
  __syncthreads();
  const int D = a.D;
  for (uint32_t s0 = 0; s0 < a.n_snap; s0 += blockDim.x) {
    const uint32_t s = s0 + threadIdx.x;
    uint64_t lo = 0, hi = 0;
    if (s < a.n_snap) {
      if (a.n_snap == 1) { lo = 0; hi = a.N; }
      else {
        const uint64_t k0 = (uint64_t)s << (3 * D), k1 = (uint64_t)(s + 1) << (3 * D);
        uint64_t l = 0, h = a.N;
        while (l < h) { uint64_t mid = l + ((h - l) >> 1); if ((uint64_t)skey[mid] < k0) l = mid + 1; else h = mid; }
        lo = l; h = a.N;
        while (l < h) { uint64_t mid = l + ((h - l) >> 1); if ((uint64_t)skey[mid] < k1) l = mid + 1; else h = mid; }
        hi = l;
      }
    }
    const uint32_t ne = (s < a.n_snap && hi > lo) ? 1u : 0u;
    const uint32_t se = (ne && hi - lo > a.n) ? 1u : 0u;
    uint32_t tot_n, tot_s;
    uint32_t on = block_excl_scan<uint32_t>(ne, tmp, tot_n);
    uint32_t os = block_excl_scan<uint32_t>(se, tmp, tot_s);
    if (ne) {
      const uint32_t v = base_nodes + on;
      if (v < a.node_cap) {
        t.prefix[v] = s; t.depth[v] = 0; t.parent[v] = NONE; t.first_child[v] = NONE;
        t.child_mask[v] = 0; t.part_begin[v] = lo; t.part_count[v] = hi - lo;
        t.sel_idx[v] = se ? base_sel + os : NONE; t.wit[v] = NONE; t.pend[v] = 0;
        if (se && base_sel + os < a.node_cap) t.sel_node[base_sel + os] = v;
      } else {
        set_status(a, LOD_STATUS_CAPACITY);
        if (se && base_sel + os < a.node_cap) t.sel_node[base_sel + os] = NONE;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) { base_nodes += tot_n; base_sel += tot_s; }
    __syncthreads();
  }
  if (threadIdx.x == 0) { t.lvl[1] = min((uint64_t)base_nodes, a.node_cap); t.lsel[1] = base_sel; }
  __syncthreads();
}

// Octant boundaries of internal node v of level d, by one wave: eight lanes per
// octant search for its first key, reading eight keys of the remaining range
// at once (a ninth of it is left: eight dependent reads for 16 M particles,
// where a binary search takes 24).  Writes the node's nine boundaries and
// returns, on every lane, the number of non-empty octants and (nsel) of those
// holding more than n particles.
__device__ uint32_t search_octants(const BuildArgs &a, const TreeArgs &t, const uint32_t *__restrict__ skey, int d,
                                   uint32_t v, uint32_t &nsel) {
  const uint32_t lane = threadIdx.x & (WAVE - 1), o = lane / 8, sub = lane % 8;
  const uint64_t lo = t.part_begin[v], hi = lo + t.part_count[v];
  uint64_t l = lo, h = hi;
  if (o) {
    const uint64_t target = ((t.prefix[v] << 3) | o) << (3 * (a.D - d - 1));
    while (h - l > 8) {
      const uint64_t step = (h - l) / 9;
      const bool lt = (uint64_t)skey[l + step * (sub + 1)] < target;
      const uint32_t c = __popc((uint32_t)(__ballot(lt) >> (8 * o)) & 0xFFu);
      if (c < 8) h = l + step * (c + 1);
      if (c) l += step * c + 1;
    }
    const bool lt = l + sub < h && (uint64_t)skey[min(l + sub, hi - 1)] < target;
    l += __popc((uint32_t)(__ballot(lt) >> (8 * o)) & 0xFFu);
  }
  const uint32_t start = (uint32_t)l;
  const uint32_t next = __shfl_down(start, 8, WAVE);
  const uint32_t cnt = (o == 7 ? (uint32_t)hi : next) - start;
  if (sub == 0) t.cs[(uint64_t)v * 9 + o] = start;
  if (lane == WAVE - 1) t.cs[(uint64_t)v * 9 + 8] = (uint32_t)hi;
  nsel = (uint32_t)__popcll(__ballot(sub == 0 && cnt > a.n));
  return (uint32_t)__popcll(__ballot(sub == 0 && cnt > 0));
}

struct EmitOct {
  uint32_t v, cnt, begin;
  bool valid;
};

// Octant o = threadIdx.x % 8 of node v of level d (valid: the node exists).
__device__ __forceinline__ EmitOct emit_octant(const BuildArgs &a, const TreeArgs &t, int d, uint64_t v, bool valid) {
  EmitOct r{};
  r.valid = valid;
  r.v = (uint32_t)v;
  if (!valid) return r;
  const uint32_t o = threadIdx.x & 7u;
  if (t.part_count[v] > a.n && d < a.D) {
    r.begin = t.cs[v * 9 + o];
    r.cnt = t.cs[v * 9 + o + 1] - r.begin;
  }
  return r;
}

// The child of one octant, number c of the nodes and sidx of the selecting
// ones; every thread of the block calls it.
__device__ __forceinline__ void emit_child(const BuildArgs &a, const TreeArgs &t, int d, const EmitOct &x, uint64_t c,
                                           uint32_t sidx) {
  const uint32_t o = threadIdx.x & 7u;
  const bool ne = x.cnt > 0, se = x.cnt > a.n;
  // the node's 8 octants are 8 consecutive lanes of one wave
  const int sh = (int)(threadIdx.x & (WAVE - 1) & ~7u);
  const uint32_t mask = (uint32_t)(__ballot(ne) >> sh) & 0xFFu;
  const uint32_t nsel = (uint32_t)__popc((uint32_t)(__ballot(se) >> sh) & 0xFFu);
  if (x.valid && o == 0) {
    t.child_mask[x.v] = (uint8_t)mask;
    t.pend[x.v] = nsel;
    t.first_child[x.v] = (mask && c + __popc(mask) <= a.node_cap) ? (uint32_t)c : NONE;
  }
  if (!ne) return;
  if (c >= a.node_cap) {
    set_status(a, LOD_STATUS_CAPACITY);
    if (se && sidx < a.node_cap) t.sel_node[sidx] = NONE;
    return;
  }
  t.prefix[c] = (t.prefix[x.v] << 3) | (uint64_t)o;
  t.depth[c] = (uint8_t)(d + 1);
  t.parent[c] = x.v;
  t.first_child[c] = NONE;
  t.child_mask[c] = 0;
  t.part_begin[c] = x.begin;
  t.part_count[c] = x.cnt;
  t.sel_idx[c] = se ? sidx : NONE;
  if (se && sidx < a.node_cap) t.sel_node[sidx] = (uint32_t)c;
  t.wit[c] = NONE;
  t.pend[c] = 0;
}

// The roots and the children of levels 0 .. top - 1 by one block: levels that
// hold at most TOP_NODES nodes, a wave per node for the boundaries and a thread
// per octant for the children.  (Below, a level takes two launches; the first
// levels' few nodes are bound by latency, and each launch costs as much again.)
// Sixteen nodes: one for each of the block's waves; a second turn would take
// as long as the level's two launches.  Roots and levels 0 and 1 of 262,144
// particles take 13 us, of 16.7 M 22 us.
constexpr uint32_t TOP_NODES = 16;
__global__ __launch_bounds__(1024) void k_tree_top(BuildArgs a, TreeArgs t, const uint32_t *__restrict__ skey,
                                                   int top) {
  __shared__ uint32_t tmp[1024 / WAVE + 1];
  make_roots(a, t, skey);
  for (int d = 0; d < top; ++d) {
    const uint32_t b = t.lvl[d], e = t.lvl[d + 1];
    for (uint32_t v = b + threadIdx.x / WAVE; v < e; v += blockDim.x / WAVE) {
      uint32_t nsel;
      if (t.part_count[v] > a.n) search_octants(a, t, skey, d, v, nsel);
    }
    __syncthreads();
    // at most TOP_NODES nodes: 8 threads each
    const uint64_t v = (uint64_t)b + threadIdx.x / 8;
    const EmitOct x = emit_octant(a, t, d, v, v < e);
    uint32_t tk, ts;
    const uint32_t ok = block_excl_scan<uint32_t>(x.cnt > 0 ? 1u : 0u, tmp, tk);
    const uint32_t os = block_excl_scan<uint32_t>(x.cnt > a.n ? 1u : 0u, tmp, ts);
    emit_child(a, t, d, x, (uint64_t)e + ok, t.lsel[d + 1] + os);
    if (threadIdx.x == 0) {
      t.lvl[d + 2] = (uint32_t)min((uint64_t)e + tk, a.node_cap);
      t.lsel[d + 2] = t.lsel[d + 1] + ts;
    }
    __syncthreads();
  }
}

// A further level in two launches: the boundaries, a wave per node, with the
// children (and selecting children) of every EMIT_NODES nodes added to their
// total and to that of GROUP such blocks; then the children, a thread per
// octant.  A child's index is the node-major, octant-minor count of non-empty
// octants before it: the totals before the block, which it adds up itself (a
// scan of them would be a third launch), and a block scan.  The emission runs
// beside the density kernel, which fills the CUs: a 256-thread block finds room
// as soon as one density block ends, a 1024-thread block only when a whole CU
// drains.
// Roots and four levels of 262,144 particles: 34 us in five launches, against
// 79 in seventeen (binary search, count, scan, write); the whole build 309
// against 360 us, of 16.7 M particles 1778 against 1876.
constexpr int EMIT_BT = 256;
constexpr int EMIT_NODES = EMIT_BT / 8;   // nodes per block
constexpr uint32_t GROUP = 64;            // blocks per group of totals

__global__ __launch_bounds__(EMIT_BT) void k_tree_search(BuildArgs a, TreeArgs t, const uint32_t *__restrict__ skey,
                                                         int d, uint32_t *__restrict__ tot,
                                                         uint32_t *__restrict__ gtot) {
  const uint32_t b = t.lvl[d], e = t.lvl[d + 1];
  const uint32_t lane = threadIdx.x & (WAVE - 1);
  for (uint64_t i = ((uint64_t)blockIdx.x * EMIT_BT + threadIdx.x) / WAVE; b + i < e;
       i += (uint64_t)gridDim.x * (EMIT_BT / WAVE)) {
    const uint32_t v = b + (uint32_t)i;
    if (t.part_count[v] <= a.n) continue;
    uint32_t nsel;
    const uint32_t nk = search_octants(a, t, skey, d, v, nsel);
    // lanes 0 and 1: children and selecting children
    const uint32_t c = lane ? nsel : nk;
    const uint64_t j = i / EMIT_NODES;
    if (lane < 2 && c) {
      atomicAdd(&tot[2 * j + lane], c);
      atomicAdd(&gtot[2 * (j / GROUP) + lane], c);
    }
  }
}

__global__ __launch_bounds__(EMIT_BT) void k_tree_write(BuildArgs a, TreeArgs t, int d,
                                                        const uint2 *__restrict__ tot,
                                                        const uint2 *__restrict__ gtot) {
  __shared__ uint32_t tmp[EMIT_BT / WAVE + 1];
  const uint32_t b = t.lvl[d], e = t.lvl[d + 1];
  const uint32_t nb = (e - b + EMIT_NODES - 1) / EMIT_NODES;   // blocks with nodes
  if (blockIdx.x >= max(nb, 1u)) return;
  uint32_t bk = 0, bs = 0, ak = 0, as = 0;
  const uint32_t g = blockIdx.x / GROUP;
  for (uint32_t j = threadIdx.x; j * GROUP < nb && (j < g || blockIdx.x == 0); j += EMIT_BT) {
    const uint2 q = gtot[j];
    if (j < g) { bk += q.x; bs += q.y; }
    ak += q.x; as += q.y;
  }
  for (uint32_t j = g * GROUP + threadIdx.x; j < blockIdx.x; j += EMIT_BT) { bk += tot[j].x; bs += tot[j].y; }
  bk = block_reduce_sum<uint32_t>(bk, tmp);
  bs = block_reduce_sum<uint32_t>(bs, tmp);
  if (blockIdx.x == 0) {
    ak = block_reduce_sum<uint32_t>(ak, tmp);
    as = block_reduce_sum<uint32_t>(as, tmp);
    if (threadIdx.x == 0) {
      t.lvl[d + 2] = (uint32_t)min((uint64_t)e + ak, a.node_cap);
      t.lsel[d + 2] = t.lsel[d + 1] + as;
    }
  }
  const uint64_t v = (uint64_t)b + (uint64_t)blockIdx.x * EMIT_NODES + threadIdx.x / 8;
  const EmitOct x = emit_octant(a, t, d, v, v < e);
  uint32_t tk, ts;
  const uint32_t ok = block_excl_scan<uint32_t>(x.cnt > 0 ? 1u : 0u, tmp, tk);
  const uint32_t os = block_excl_scan<uint32_t>(x.cnt > a.n ? 1u : 0u, tmp, ts);
  emit_child(a, t, d, x, (uint64_t)e + bk + ok, t.lsel[d + 1] + bs + os);
}

// Stored point counts and offsets of every slot below node_cap (past the node
// count: 0 and the total), the node and point counts.  Block b scans PT_NODES
// nodes and leaves their total; then it adds up the totals before it, whole
// groups of them first.  gsums: a total per GROUP blocks, zero before.
constexpr int PT_NODES = 1024;
__global__ __launch_bounds__(PT_NODES) void k_pt_scan(BuildArgs a, TreeArgs t, int D, uint64_t *__restrict__ sums,
                                                      unsigned long long *__restrict__ gsums) {
  __shared__ uint64_t tmp[PT_NODES / WAVE + 1];
  const uint32_t nn = t.lvl[D + 1];
  const uint64_t v = (uint64_t)blockIdx.x * PT_NODES + threadIdx.x;
  uint32_t c = 0;
  if (v < nn) c = (uint32_t)min(t.part_count[v], (uint64_t)a.n);
  if (v < a.node_cap) t.pt_count[v] = c;
  if ((uint64_t)blockIdx.x * PT_NODES >= nn) return;   // uniform
  uint64_t total;
  const uint64_t o = block_excl_scan<uint64_t>(c, tmp, total);
  if (v < nn) t.pt_begin[v] = o;
  if (threadIdx.x == 0) {
    sums[blockIdx.x] = total;
    atomicAdd(&gsums[blockIdx.x / GROUP], (unsigned long long)total);
  }
}

__global__ __launch_bounds__(PT_NODES) void k_pt_finish(BuildArgs a, TreeArgs t, int D,
                                                        const uint64_t *__restrict__ sums,
                                                        const uint64_t *__restrict__ gsums) {
  __shared__ uint64_t tmp[PT_NODES / WAVE + 1];
  const uint32_t nn = t.lvl[D + 1];
  const uint64_t v = (uint64_t)blockIdx.x * PT_NODES + threadIdx.x;
  const uint32_t nb = (nn + PT_NODES - 1) / PT_NODES, g = blockIdx.x / GROUP;
  if (blockIdx.x < nb) {
    uint64_t before = 0;
    for (uint32_t j = threadIdx.x; j < g; j += PT_NODES) before += gsums[j];
    for (uint32_t j = g * GROUP + threadIdx.x; j < blockIdx.x; j += PT_NODES) before += sums[j];
    before = block_reduce_sum<uint64_t>(before, tmp);
    if (v < nn) t.pt_begin[v] += before;
  }
  // the last block of the grid has the counts to write; it and the blocks with
  // slots past the nodes need the total
  const bool last = blockIdx.x == gridDim.x - 1;
  if (!last && (uint64_t)(blockIdx.x + 1) * PT_NODES <= nn) return;
  uint64_t total = 0;
  for (uint32_t j = threadIdx.x; j * GROUP < nb; j += PT_NODES) total += gsums[j];
  total = block_reduce_sum<uint64_t>(total, tmp);
  if (last && threadIdx.x == 0) {
    a.counts[0] = nn;
    a.counts[1] = total;
    if (total > a.point_cap) set_status(a, LOD_STATUS_CAPACITY);
  }
  if (v >= nn && v < a.node_cap) t.pt_begin[v] = total;
}

// ---------------------------------------------------------------------------
// leaves: float64 node mass; leaves holding <= n copy their particles

struct Sorted {
  const uint32_t *key;
  const uint32_t *idx;
  const uint32_t *lo;   // x and y fractions (16 bits each)
  const uint16_t *lz;   // z fraction
  const float *m;
  const uint32_t *w;
  const uint16_t *kb;   // log-scale bin of the selection key
};

// A stored point's fields read from the sorted arrays (loads are issued for
// every lane; the stores are predicated by the caller).
struct PointIn {
  uint32_t k, id;
  uint64_t l;
};

__device__ __forceinline__ PointIn read_point(const Sorted &s, uint64_t pos) {
  return PointIn{s.key[pos], s.idx[pos], (uint64_t)s.lo[pos] | ((uint64_t)s.lz[pos] << 32)};
}

// A stored point's id and 16-bit codes (x in the low, y in the high half of xy).
struct PointOut {
  uint32_t id, xy, z;
};

__device__ __forceinline__ PointOut code_point(const BuildArgs &a, const PointIn &q, int d) {
  const int D = a.D;
  const uint32_t kk = D ? (q.k & (uint32_t)((1ull << (3 * D)) - 1)) : 0u;
  const uint32_t cx = compact3(kk), cy = compact3(kk >> 1), cz = compact3(kk >> 2);
  const uint32_t snap = (a.n_snap > 1) ? (uint32_t)((uint64_t)q.k >> (3 * D)) : 0u;
  return PointOut{(uint32_t)local_id(a, snap, q.id),
                  (uint32_t)quant_at(cx, (uint32_t)(q.l & 0xFFFFu), D, d) |
                      ((uint32_t)quant_at(cy, (uint32_t)((q.l >> 16) & 0xFFFFu), D, d) << 16),
                  (uint32_t)quant_at(cz, (uint32_t)((q.l >> 32) & 0xFFFFu), D, d)};
}

__device__ __forceinline__ void store_codes(const TreeArgs &t, const PointOut &o, uint64_t out) {
  t.pt_id[out] = o.id;
  t.qx[out] = (uint16_t)(o.xy & 0xFFFFu);
  t.qy[out] = (uint16_t)(o.xy >> 16);
  t.qz[out] = (uint16_t)o.z;
}

__device__ __forceinline__ void store_point(const BuildArgs &a, const TreeArgs &t, const PointIn &q, uint64_t out,
                                            int d, float mass) {
  store_codes(t, code_point(a, q, d), out);
  t.pt_mass[out] = mass;
}

// Exact selection key of the particle at sorted position p.
__device__ __forceinline__ uint64_t exact_K(const BuildArgs &a, const Sorted &s, uint32_t p) {
  const uint32_t snap = (a.n_snap > 1) ? (uint32_t)((uint64_t)s.key[p] >> (3 * a.D)) : 0u;
  const uint64_t U = particle_U(local_id(a, snap, s.idx[p]), snap, a.seed);
  return selection_key(U, s.w[p], a.alpha);
}

constexpr int LILP = 4;       // particles per thread per step when copying a leaf

// Copies leaf v's particles to its stored points (codes at the leaf's depth,
// float32 masses as given), whole block.
__device__ __forceinline__ void copy_leaf_points(const BuildArgs &a, const TreeArgs &t, const Sorted &s,
                                                 uint32_t v) {
  const uint64_t b = t.part_begin[v], c = t.part_count[v];
  const uint64_t ob = t.pt_begin[v];
  const int d = t.depth[v];
  const uint32_t BS = blockDim.x;
  for (uint64_t i0 = threadIdx.x; i0 < c; i0 += (uint64_t)BS * LILP) {
    float mm[LILP];
    PointIn q[LILP];
#pragma unroll
    for (int u = 0; u < LILP; ++u) {
      const uint64_t pos = b + min(i0 + (uint64_t)u * BS, c - 1);
      mm[u] = s.m[pos];
      q[u] = read_point(s, pos);
    }
#pragma unroll
    for (int u = 0; u < LILP; ++u) {
      const uint64_t i = i0 + (uint64_t)u * BS;
      if (i < c) store_point(a, t, q[u], ob + i, d, mm[u]);
    }
  }
}

// Leaves: float64 mass of every leaf and, with COPY, its stored points (the
// per-level schedule copies them inside the selection launches instead).
template <bool COPY>
__global__ __launch_bounds__(TB) void k_leaves(BuildArgs a, TreeArgs t, Sorted s) {
  __shared__ double red[TB / WAVE + 1];
  const uint32_t nn = t.lvl[a.D + 1];
  const bool cap_ok = a.counts[1] <= a.point_cap;
  for (uint32_t v = blockIdx.x; v < nn; v += gridDim.x) {
    if (t.first_child[v] != NONE) continue;
    const uint64_t b = t.part_begin[v], c = t.part_count[v];
    const bool copy = COPY && c <= a.n && cap_ok;
    const uint64_t ob = t.pt_begin[v];
    const int d = t.depth[v];
    double acc = 0.0;
    if (copy) {
      for (uint64_t i0 = threadIdx.x; i0 < c; i0 += TB * LILP) {
        float mm[LILP];
        PointIn q[LILP];
#pragma unroll
        for (int u = 0; u < LILP; ++u) {
          const uint64_t pos = b + min(i0 + (uint64_t)u * TB, c - 1);
          mm[u] = s.m[pos];
          q[u] = read_point(s, pos);
        }
#pragma unroll
        for (int u = 0; u < LILP; ++u) {
          const uint64_t i = i0 + (uint64_t)u * TB;
          if (i < c) {
            acc += (double)mm[u];
            store_point(a, t, q[u], ob + i, d, mm[u]);
          }
        }
      }
    } else {
      constexpr int MILP = 4 * LILP;
      for (uint64_t i0 = threadIdx.x; i0 < c; i0 += TB * MILP) {
        float mm[MILP];
#pragma unroll
        for (int u = 0; u < MILP; ++u) mm[u] = s.m[b + min(i0 + (uint64_t)u * TB, c - 1)];
#pragma unroll
        for (int u = 0; u < MILP; ++u)
          if (i0 + (uint64_t)u * TB < c) acc += (double)mm[u];
      }
    }
    const double M = block_reduce_sum<double>(acc, red);
    if (threadIdx.x == 0) t.node_mass[v] = M;
  }
}

// ---------------------------------------------------------------------------
// selection: per node holding > n particles, the n+1 smallest (K, id)

constexpr int SMALL = 512;
constexpr int KBINS = 4096;
constexpr int SILP = 8;       // candidates per lane per wave step of the (rare) exact-key rounds
constexpr int CILP = 8;       // 16-byte chunks of key bins per lane in flight
constexpr int OILP = 4;       // list entries per thread per step of the output pass
constexpr int QCAP = 2048;    // bin-b0 candidates queued in LDS by the collect pass
constexpr int MAXSEG = 9;     // segments of a node's candidates (8 children)
constexpr uint32_t CHUNK = 8; // key bins per 16-byte chunk
// chunks whose taken flags (a byte each) fit the histogram's storage: 131072
// candidates, which holds the eight lists of n <= 16383 points
constexpr uint32_t FLAG_CHUNKS = 4 * KBINS;
// Histograms of the lists' key bins (16 bits a bin) are kept for n in
// [2048, 65534]: below, they would take more memory than the lists (14 n bytes)
// and the lists are read as fast; above, a bin may not fit.
__host__ __device__ inline bool keeps_list_hist(uint64_t n) { return n >= 2048 && n < 65535; }

// A list entry is a sorted position, its key bin and the candidate's density
// weight and mass (so that the parent's output pass reads them in list order
// instead of gathering them from the sorted arrays).
struct SelArgs {
  uint32_t *lpos;             // top-(n+1) lists by selecting rank: sorted positions
  uint16_t *lkb;              // and their key bins (a separate array: the counting passes read only these)
  uint2 *lwm;                 // and (w, mass bits)
  uint32_t n_minus_1;         // N - 1
  uint16_t *lhist;            // [rank][KBINS] entries of each list by key bin, or null
  uint32_t *widx;             // [node] the witness's index in the node's list
  double *mhat;               // float64 mass scratch, one row of n per block
  uint32_t *src;              // candidate of each list entry, one row of n+1 per block
};

// sorted position of list entry i (clamped: the lists are workspace)
__device__ __forceinline__ uint32_t entry_pos(const SelArgs &sa, uint64_t i) { return min(sa.lpos[i], sa.n_minus_1); }

// A node's candidates: the concatenation of its segments, in sorted position
// order (runs of leaf children form one range segment).  Their key bins are
// read in 16-byte chunks, and the chunks of all segments form one sequence
// (first of segment k: cst[k]).  A candidate is named by 8 times its chunk plus
// its element in the chunk, its code: ascending codes are the candidate order.
struct Segs {
  uint32_t nseg;
  uint64_t base[MAXSEG];   // start sorted position (range) or list offset (list)
  uint32_t len[MAXSEG];
  uint32_t is_list[MAXSEG];
  uint32_t cst[MAXSEG + 1];      // first chunk; their number at [nseg], then ~0
  uint64_t adj[MAXSEG];          // sorted position or list offset of code x of segment k: adj[k] + x
  const uint16_t *kb[MAXSEG];    // key bin of code x of segment k: kb[k][x]
  uint32_t head[MAXSEG], tail[MAXSEG];         // valid elements (bits) of the first and of the last chunk
  // list segments: the child's selecting rank, the codes of its first entry and
  // of its witness, its first stored point and its octant (the bit each cell
  // coordinate gains from parent to child)
  uint32_t crank[MAXSEG], cx0[MAXSEG], cwx[MAXSEG];
  uint64_t cob[MAXSEG];
  uint32_t coct[MAXSEG];
};

// Segment of chunk c (entries past the last segment are ~0).
__device__ __forceinline__ uint32_t seg_of(const Segs &g, uint32_t c) {
  uint32_t k = 0;
#pragma unroll
  for (int i = 1; i < MAXSEG; ++i) k += c >= g.cst[i] ? 1u : 0u;
  return k;
}

// A node's children's fields, loaded by one lane each so that the loads of
// all children are in flight together.
struct Children {
  uint64_t pc[8], pb[8], ptb[8];
  uint32_t sel[8], widx[8], oct[8];
  double m[8];
};

__device__ __forceinline__ void build_segments(const BuildArgs &a, const TreeArgs &t, const Sorted &s,
                                               const SelArgs &sa, uint32_t v, uint32_t fc, int nk,
                                               const Children &ch, Segs &g) {
  const uint32_t n = a.n;
  uint32_t ns = 0;
  if (fc == NONE) {
    g.base[0] = t.part_begin[v]; g.len[0] = (uint32_t)t.part_count[v]; g.is_list[0] = 0; ns = 1;
  } else {
    for (int k = 0; k < nk; ++k) {
      if (ch.pc[k] > n) {
        g.base[ns] = (uint64_t)ch.sel[k] * (n + 1); g.len[ns] = n + 1; g.is_list[ns] = 1;
        g.crank[ns] = ch.sel[k]; g.cwx[ns] = ch.widx[k]; g.cob[ns] = ch.ptb[k]; g.coct[ns] = ch.oct[k];
        ++ns;
      } else if (ns > 0 && !g.is_list[ns - 1]) {
        g.len[ns - 1] += (uint32_t)ch.pc[k];   // siblings are adjacent in sorted order
      } else {
        g.base[ns] = ch.pb[k]; g.len[ns] = (uint32_t)ch.pc[k]; g.is_list[ns] = 0;
        ++ns;
      }
    }
  }
  g.nseg = ns;
  uint32_t c = 0;
  for (uint32_t k = 0; k < ns; ++k) {
    const uint64_t a0 = g.base[k] / CHUNK, a1 = (g.base[k] + g.len[k] - 1) / CHUNK;
    g.cst[k] = c;
    g.adj[k] = CHUNK * a0 - CHUNK * (uint64_t)c;
    g.kb[k] = (g.is_list[k] ? sa.lkb : s.kb) + g.adj[k];
    g.head[k] = 0xFFu << (g.base[k] % CHUNK);
    g.tail[k] = 0xFFu >> (CHUNK - 1 - (g.base[k] + g.len[k] - 1) % CHUNK);
    g.cx0[k] = (uint32_t)(CHUNK * c + g.base[k] % CHUNK);
    if (g.is_list[k]) g.cwx[k] += g.cx0[k];   // from the list index
    c += (uint32_t)(a1 - a0 + 1);
  }
  g.cst[ns] = c;
  for (uint32_t k = ns + 1; k <= MAXSEG; ++k) g.cst[k] = 0xFFFFFFFFu;
}

// Wave w of the block owns the w-th of W equal contiguous parts of a segment
// (exact-key rounds) or of the chunk sequence.
__device__ __forceinline__ void wave_part(uint32_t L, uint32_t w, uint32_t W, uint32_t &lo, uint32_t &hi) {
  const uint32_t P = (L + W - 1) / W;
  lo = min(L, w * P);
  hi = min(L, lo + P);
}

// Loads NL candidates (sorted position, key bin) of a wave step; indices
// are clamped into the part, so every load is issued unconditionally.
template <int NL>
__device__ __forceinline__ void load_step(const Segs &g, int k, const SelArgs &sa, const Sorted &s, uint32_t j0,
                                          uint32_t hi, uint32_t (&pos)[NL], uint32_t (&kb)[NL]) {
  const uint32_t lane = threadIdx.x & (WAVE - 1);
  const uint64_t base = g.base[k];
  if (g.is_list[k]) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const uint64_t i = base + min(j0 + u * WAVE + lane, hi - 1);
      pos[u] = entry_pos(sa, i);
      kb[u] = sa.lkb[i];
    }
  } else {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const uint64_t p = base + min(j0 + u * WAVE + lane, hi - 1);
      pos[u] = (uint32_t)p;
      kb[u] = s.kb[p];
    }
  }
}

// Calls f(c, k, valid, v) for the chunks [lo, hi) of this wave, in order of c
// within a lane: the chunk's segment, its valid elements (bits) and its eight
// key bins.  CILP 16-byte loads of a lane are in flight together, across
// segments, so a pass over a node's lists costs a few memory latencies, not
// one per list.  (Reads may run up to 16 bytes past a part; the key-bin arrays
// are padded for it.)
// A step's segment is found once per wave when all of its chunks lie in one
// segment (nearly always: a list of 16 k entries is 2 k chunks).
__device__ __forceinline__ uint32_t step_seg(const Segs &g, uint32_t c0, uint32_t hi) {
  const uint32_t lane = threadIdx.x & (WAVE - 1);
  const uint32_t k0 = __builtin_amdgcn_readfirstlane(seg_of(g, c0));
  if (min(c0 + WAVE, hi) <= g.cst[k0 + 1]) return k0;
  return seg_of(g, min(c0 + lane, hi - 1));
}

template <typename F>
__device__ __forceinline__ void for_chunks(const Segs &g, uint32_t lo, uint32_t hi, F f) {
  const uint32_t lane = threadIdx.x & (WAVE - 1);
  for (uint32_t c0 = lo; c0 < hi; c0 += WAVE * CILP) {
    uint4 v[CILP];
    uint32_t ks[CILP];
#pragma unroll
    for (int u = 0; u < CILP; ++u) {
      ks[u] = step_seg(g, min(c0 + u * WAVE, hi - 1), hi);
      v[u] = *reinterpret_cast<const uint4 *>(g.kb[ks[u]] + (uint64_t)min(c0 + u * WAVE + lane, hi - 1) * CHUNK);
    }
#pragma unroll
    for (int u = 0; u < CILP; ++u) {
      const uint32_t c = c0 + u * WAVE + lane, k = ks[u];
      if (c < hi) {
        uint32_t valid = 0xFFu;
        if (c == g.cst[k]) valid &= g.head[k];
        if (c + 1 == g.cst[k + 1]) valid &= g.tail[k];
        f(c, k, valid, v[u]);
      }
    }
  }
}

// Sorted position of the candidate of code x in segment k.
__device__ __forceinline__ uint32_t cand_pos(const Segs &g, const SelArgs &sa, uint32_t k, uint32_t x) {
  return g.is_list[k] ? entry_pos(sa, g.adj[k] + x) : (uint32_t)(g.adj[k] + x);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// Of a chunk's key bins: le = those at most b, eq = those equal to b (bits in
// element order).  A saturating packed subtraction leaves 0 below, 1 at and 2
// or more above b, for two bins at a time; the two-bit codes of all eight are
// gathered before the bits are taken apart.
__device__ __forceinline__ void compare_bins(uint4 v, uint32_t b, uint32_t &le, uint32_t &eq) {
  const uint32_t b1 = b ? b - 1 : 0u, up = b ? 0u : 0x00010001u;   // (k + 1) - 1 for b = 0: bins stay below 2^12
  const u16x2 bb = {(unsigned short)b1, (unsigned short)b1};
  const uint32_t wd[4] = {v.x + up, v.y + up, v.z + up, v.w + up};
  uint32_t p = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u16x2 d = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, wd[i]), bb);
    p |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(d, u16x2{2, 2})) << (2 * i);
  }
  const uint32_t above = (p >> 1) & 0x00550055u, at = p & 0x00550055u;
  le = ((above | (above >> 15)) & 0xFFu) ^ 0xFFu;
  eq = (at | (at >> 15)) & 0xFFu;
}

// Calls f(pos, kb) for every candidate of this wave's parts of the segments.
template <typename F>
__device__ __forceinline__ void for_parts(const Segs &g, const SelArgs &sa, const Sorted &s, F f) {
  const uint32_t W = blockDim.x / WAVE, w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  for (int k = 0; k < (int)g.nseg; ++k) {
    uint32_t lo, hi;
    wave_part(g.len[k], w, W, lo, hi);
    for (uint32_t j0 = lo; j0 < hi; j0 += WAVE * SILP) {
      uint32_t pos[SILP], kb[SILP];
      load_step(g, k, sa, s, j0, hi, pos, kb);
#pragma unroll 1
      for (int u = 0; u < SILP; ++u)
        if (j0 + u * WAVE + lane < hi) f(pos[u], kb[u]);
    }
  }
}

// Whether the candidate at sorted position p lies at or below the witness
// (K_t, id_t) in (K, id) order, from its exact key.
__device__ __forceinline__ bool taken_exact(const BuildArgs &a, const Sorted &s, uint32_t p, uint64_t Kt, uint32_t It) {
  const uint64_t K = exact_K(a, s, p);
  return K < Kt || (K == Kt && s.idx[p] <= It);
}

// m / min(1, w^alpha / tau) with one float64 division at most.
__device__ __forceinline__ double unscaled_mass(float m, uint32_t w, int alpha, double tau) {
  const double m64 = (double)m;
  if (alpha > 0) return (double)w >= tau ? m64 : m64 * tau / (double)w;
  if (alpha == 0) return tau <= 1.0 ? m64 : m64 * tau;
  return 1.0 >= tau * (double)w ? m64 : m64 * (tau * (double)w);
}

// Sum of row[0..n) in an order fixed by n alone, so that every block size and
// schedule stores the same bits: groups of RS_GROUP entries, lane i of a wave
// adding entries i, i + 64, ... of its group in order (absent entries 0), then
// a xor butterfly over the lanes; 64 group sums by one more butterfly, and
// those added in order by thread 0.  cs: RS_SUMS doubles of LDS; the result is
// returned to every thread (barriers inside).  (A butterfly per 64 entries was
// bound by its own instructions: 6.5 us for n = 16000.)
//
// The butterfly runs on lane swaps and row rotations instead of LDS permutes:
// once two halves hold equal sums, a rotation by o brings the value that the
// xor by o would.
__device__ __forceinline__ double wave_sum_xor(double x) {
  auto words = [](double d, uint32_t &lo, uint32_t &hi) {
    const uint64_t b = (uint64_t)__double_as_longlong(d);
    lo = (uint32_t)b; hi = (uint32_t)(b >> 32);
  };
  auto make = [](uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); };
  uint32_t lo, hi;
  words(x, lo, hi);
  {
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    x = make(a[0], b[0]) + make(a[1], b[1]);
  }
  words(x, lo, hi);
  {
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = make(a[0], b[0]) + make(a[1], b[1]);
  }
#define LOD_ROR(n)                                                                            \
  words(x, lo, hi);                                                                           \
  x += make((uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x120 + n, 0xF, 0xF, false),    \
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x120 + n, 0xF, 0xF, false));
  LOD_ROR(8) LOD_ROR(4) LOD_ROR(2) LOD_ROR(1)
#undef LOD_ROR
  return x;
}

constexpr uint32_t RS_ROWS = 16, RS_GROUP = RS_ROWS * WAVE, RS_SUMS = 64;
__device__ double row_sum_fixed(const double *row, uint32_t n, double *cs, double *res) {
  const uint32_t W = blockDim.x / WAVE, w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const uint32_t groups = (n + RS_GROUP - 1) / RS_GROUP;
  double total = 0.0;   // thread 0's
  for (uint32_t g0 = 0; g0 < groups; g0 += RS_SUMS) {
    const uint32_t g1 = min(groups, g0 + RS_SUMS);
    for (uint32_t g = g0 + w; g < g1; g += W) {
      double x[RS_ROWS];
#pragma unroll
      for (uint32_t k = 0; k < RS_ROWS; ++k) x[k] = row[min(g * RS_GROUP + k * WAVE + lane, n - 1)];
      double y = 0.0;
#pragma unroll
      for (uint32_t k = 0; k < RS_ROWS; ++k) y += g * RS_GROUP + k * WAVE + lane < n ? x[k] : 0.0;
      y = wave_sum_xor(y);
      if (lane == 0) cs[g - g0] = y;
    }
    __syncthreads();
    if (w == 0) {
      const double x = wave_sum_xor(lane < g1 - g0 ? cs[lane] : 0.0);
      if (lane == 0) total += x;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *res = total;
  __syncthreads();
  return *res;
}

// One selecting node, whole block: the n+1 smallest (K, id) among its
// candidates (children's lists or its own range) form its list, ascending by
// sorted position; the (n+1)-th smallest is the witness.  The other n are
// its stored points, written with their float64-renormalised masses.
//
// Round 0 histograms the 12-bit log-scale bin of K (stored per particle): the
// ranges' by reading them, the lists' from the histograms their nodes left.
// The exact K is recomputed only in the threshold bin b0 (rare further rounds
// split it by 8-bit digits of K, then of the id).  One pass over the key bins
// then leaves a flag per candidate (bin at most b0) in LDS, counts per wave
// those below b0 and queues those in b0, which are keyed and ranked; the flags
// of the ones not taken are cleared.  The flags are expanded into the list of
// taken candidates (wave offsets and popcount scans), and the output pass
// reads each taken candidate's fields, every lane busy.
//
// What bounds a node is the chain of memory latencies and barriers, not its
// bytes: a pass that reads 128 k key bins of eight lists one list after the
// other took 10-30 us, and there were three, with the 128 k histogram adds and
// a compaction that also read all 128 k positions.  A node of eight lists (1024
// threads, n = 16000) took 154 us at 16.7 M particles and takes 78: histogram
// 17 -> 5, collect 30 -> 12, compaction 43 -> 6, mass sum 11 -> 3; a node of
// ranges 86 -> 78 (its output pass, 40 us beside 140 others, moves 1.4 MB of
// fields, lists and points at the memory's rate).
__device__ void select_node(const BuildArgs &a, const TreeArgs &t, const Sorted &s, const SelArgs &sa,
                            uint32_t v) {
  __shared__ Segs g;
  __shared__ Children ch;
  __shared__ uint32_t hist[KBINS];               // later: a flag byte per chunk
  __shared__ uint64_t ck[SMALL];
  __shared__ uint32_t cidx[SMALL], cpos[SMALL], ccode[SMALL], crnk[SMALL];
  __shared__ uint32_t pcnt[1024 / WAVE];         // per wave: taken candidates, then list offset
  __shared__ uint32_t ccount, sh_total, nq;
  __shared__ uint32_t qcode[QCAP];
  __shared__ uint32_t red32[1024 / WAVE + 1];
  __shared__ double cs64[RS_SUMS];
  __shared__ double sh_mtot;
  __shared__ uint64_t sh_kt;
  __shared__ uint32_t sh_it, sh_pt, sh_px, sh_wj;
  __shared__ uint32_t sh_b, sh_below, sh_cnt;
  __shared__ double sh_tau;
  const uint32_t n = a.n;
  const int BS = blockDim.x;
  const uint32_t W = BS / WAVE, w = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  if (threadIdx.x < WAVE) {
    const uint32_t fc = t.first_child[v];
    const int nk = fc == NONE ? 0 : __popc((uint32_t)t.child_mask[v]);
    if ((int)threadIdx.x < nk) {
      const uint32_t u = fc + threadIdx.x;
      ch.pc[threadIdx.x] = t.part_count[u]; ch.pb[threadIdx.x] = t.part_begin[u];
      ch.ptb[threadIdx.x] = t.pt_begin[u]; ch.sel[threadIdx.x] = t.sel_idx[u];
      ch.widx[threadIdx.x] = sa.widx[u]; ch.oct[threadIdx.x] = (uint32_t)(t.prefix[u] & 7u);
      ch.m[threadIdx.x] = t.node_mass[u];
    }
    // the lanes' LDS writes before lane 0's reads (one wave)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (threadIdx.x == 0) {
      build_segments(a, t, s, sa, v, fc, nk, ch, g);
      // an internal node's float64 mass: its children's, summed in octant
      // order (read back by this block after the barriers below)
      if (fc != NONE) {
        double M = 0.0;
        for (int k = 0; k < nk; ++k) M += ch.m[k];
        t.node_mass[v] = M;
      }
    }
  }
  for (int i = threadIdx.x; i < KBINS; i += BS) hist[i] = 0;
  if (threadIdx.x < 1024 / WAVE) pcnt[threadIdx.x] = 0;
  if (threadIdx.x == 0) { sh_b = 0; sh_below = 0; sh_cnt = 0; }
  __syncthreads();
  // ranges (and lists without a histogram): segments' chunks split over the waves
  for (uint32_t k = 0; k < g.nseg; ++k) {
    if (sa.lhist && g.is_list[k]) continue;
    uint32_t lo, hi;
    wave_part(g.cst[k + 1] - g.cst[k], w, W, lo, hi);
    for_chunks(g, g.cst[k] + lo, g.cst[k] + hi, [&](uint32_t, uint32_t, uint32_t valid, uint4 x) {
      const uint32_t wd[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int h = 0; h < (int)CHUNK; ++h)
        if (valid & (1u << h)) atomicAdd(&hist[(wd[h >> 1] >> (16 * (h & 1))) & 0xFFFu], 1u);
    });
  }
  __syncthreads();
  uint32_t r = n;                            // 0-based rank of the witness among in-play
  {
    // a thread's run of bins: the ranges' counts plus the lists' histograms,
    // four bins (8 bytes) of every list loaded together
    const int per = KBINS / BS;              // 4 or more
    uint32_t loc = 0;
    for (int i0 = 0; i0 < per; i0 += 4) {
      const int b = threadIdx.x * per + i0;
      uint32_t h4[4] = {hist[b], hist[b + 1], hist[b + 2], hist[b + 3]};
      if (sa.lhist) {
        uint2 q[MAXSEG - 1];
        // absent segments and ranges read list 0's bins, not added
#pragma unroll
        for (int k = 0; k < MAXSEG - 1; ++k) {
          const bool use = k < (int)g.nseg && g.is_list[k];
          q[k] = *reinterpret_cast<const uint2 *>(sa.lhist + (uint64_t)(use ? g.crank[k] : 0u) * KBINS + b);
          if (!use) q[k] = make_uint2(0, 0);
        }
#pragma unroll
        for (int k = 0; k < MAXSEG - 1; ++k) {
          h4[0] += q[k].x & 0xFFFFu; h4[1] += q[k].x >> 16;
          h4[2] += q[k].y & 0xFFFFu; h4[3] += q[k].y >> 16;
        }
        for (int i = 0; i < 4; ++i) hist[b + i] = h4[i];
      }
      loc += (h4[0] + h4[1]) + (h4[2] + h4[3]);
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<uint32_t>(loc, red32, tot);
    if (r >= ex && r < ex + loc) {
      uint32_t below = ex;
      for (int i = 0; i < per; ++i) {
        const uint32_t h = hist[threadIdx.x * per + i];
        if (r < below + h) { sh_b = threadIdx.x * per + i; sh_below = below; sh_cnt = h; break; }
        below += h;
      }
    }
    __syncthreads();
    // this list's histogram: all of the bins below b0, what is left in b0
    if (sa.lhist) {
      const uint32_t b0 = sh_b, rest = n + 1 - sh_below;
      uint16_t *lh = sa.lhist + (uint64_t)t.sel_idx[v] * KBINS;
      for (int i0 = 0; i0 < per; i0 += 4) {
        const uint32_t b = threadIdx.x * per + i0;
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = b + i < b0 ? hist[b + i] : b + i == b0 ? rest : 0u;
        *reinterpret_cast<uint2 *>(lh + b) = make_uint2(x[0] | (x[1] << 16), x[2] | (x[3] << 16));
      }
    }
  }
  const uint32_t b0 = sh_b;
  r -= sh_below;
  uint32_t inplay = sh_cnt;
  const uint32_t sh_cnt0 = sh_cnt;           // candidates in bin b0
  int kshift;                                // K >> kshift == kp for the in-play candidates
  uint64_t kp;
  if (b0 < 128) { kp = b0; kshift = 0; }
  else {
    const int e = 7 + (int)((b0 - 128) / 64);
    kp = 64 + (b0 - 128) % 64;
    kshift = e - 6;
  }
  int phase = 0;                             // 0: K bits, 1: id bits
  int ishift = 32;
  uint32_t ip = 0;
  __syncthreads();
  // further rounds (rare): 8-bit digits of the exact K, then of the id
  while (inplay > SMALL && !(phase == 1 && ishift == 0)) {
    if (phase == 0 && kshift == 0) { phase = 1; continue; }
    const int wb = phase == 0 ? min(8, kshift) : min(8, ishift);
    const int sft = (phase == 0 ? kshift : ishift) - wb;
    for (int i = threadIdx.x; i < RADIX; i += BS) hist[i] = 0;
    __syncthreads();
    for_parts(g, sa, s, [&](uint32_t p, uint32_t kb) {
      if (kb != b0) return;
      const uint64_t K = exact_K(a, s, p);
      bool match;
      uint32_t dg;
      if (phase == 0) {
        match = (K >> kshift) == kp;
        dg = (uint32_t)((K >> sft) & ((1u << wb) - 1));
      } else {
        const uint32_t id = s.idx[p];
        match = (K == kp) && ((ishift >= 32) ? true : ((id >> ishift) == ip));
        dg = (id >> sft) & ((1u << wb) - 1);
      }
      if (match) atomicAdd(&hist[dg], 1u);
    });
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t below = 0, bsel = 0, cnt = 0;
      for (uint32_t bb = 0; bb < (1u << wb); ++bb) {
        const uint32_t h = hist[bb];
        if (r < below + h) { bsel = bb; cnt = h; break; }
        below += h;
      }
      sh_b = bsel; sh_below = below; sh_cnt = cnt;
    }
    __syncthreads();
    r -= sh_below;
    inplay = sh_cnt;
    if (phase == 0) { kp = (kp << wb) | sh_b; kshift = sft; }
    else { ip = (ip << wb) | sh_b; ishift = sft; }
    __syncthreads();
  }
  // One pass over the key bins: per wave, the candidates below b0; the flags;
  // those in b0 queued.  The flags and the queue have fixed room: a node with
  // more candidates (an overfull leaf, n above 16383) or more of them in b0
  // decides b0's candidates by their exact keys, and reads the key bins again
  // where it would have read the flags.
  const uint32_t C = g.cst[g.nseg];
  const bool flagged = C <= FLAG_CHUNKS && sh_cnt0 <= (uint32_t)QCAP;
  uint8_t *flags = reinterpret_cast<uint8_t *>(hist);
  const uint32_t part = ((C + W - 1) / W + 3u) & ~3u;   // chunks per wave: whole words of flags
  const uint32_t lo = min(C, w * part), hi = min(C, lo + part);
  if (threadIdx.x == 0) { ccount = 0; sh_pt = NONE; nq = 0; }
  __syncthreads();
  // a candidate of bin b0: in play (collected) or, if not, taken when it lies
  // below the in-play digits.  Returns false when it is surely not taken.
  auto visit_b0 = [&](uint32_t x, uint32_t p, uint32_t wave) -> bool {
    const uint64_t K = exact_K(a, s, p);
    const uint32_t id = s.idx[p];
    bool inp, lower;
    if (phase == 0) {
      inp = (K >> kshift) == kp;
      lower = (K >> kshift) < kp;
    } else {
      inp = (K == kp) && ((ishift >= 32) ? true : ((id >> ishift) == ip));
      lower = (K < kp) || (K == kp && ishift < 32 && (id >> ishift) < ip);
    }
    if (inp) {
      const uint32_t slot = atomicAdd(&ccount, 1u);
      if (slot < SMALL) { ck[slot] = K; cidx[slot] = id; cpos[slot] = p; ccode[slot] = x; crnk[slot] = 0; }
    } else if (lower) {
      atomicAdd(&pcnt[wave], 1u);
    }
    return inp || lower;
  };
  // the flags as bits: bit x % 32 of word x / 32 is candidate code x
  auto clear_flag = [&](uint32_t x) { atomicAnd(&hist[x / 32], ~(1u << (x % 32))); };
  {
    uint32_t below_cnt = 0;
    for_chunks(g, lo, hi, [&](uint32_t c, uint32_t k, uint32_t valid, uint4 x) {
      uint32_t le, eq;
      compare_bins(x, b0, le, eq);
      le &= valid; eq &= valid;
      below_cnt += __popc(le & ~eq);
      if (flagged) flags[c] = (uint8_t)le;
      for (; eq; eq &= eq - 1u) {
        const uint32_t x = c * CHUNK + __builtin_ctz(eq);
        if (flagged) qcode[atomicAdd(&nq, 1u)] = x;
        else visit_b0(x, cand_pos(g, sa, k, x), w);
      }
    });
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) below_cnt += __shfl_xor(below_cnt, o, WAVE);
    if (lane == 0 && below_cnt) atomicAdd(&pcnt[w], below_cnt);
    if (flagged) {
      __syncthreads();
      for (uint32_t q = threadIdx.x; q < nq; q += BS) {
        const uint32_t x = qcode[q], c = x / CHUNK;
        if (!visit_b0(x, cand_pos(g, sa, seg_of(g, c), x), c / part)) clear_flag(x);
      }
    }
  }
  __syncthreads();
  const uint32_t cc = min(ccount, (uint32_t)SMALL);
  {
    // Ranks of the in-play candidates: thread (f-quarter, pair of entries), so
    // that every wave of the block compares and each entry read from LDS
    // serves two.  Eight entries per step, every read issued before any
    // compare (clamped indices, masked counts), and no branches.
    const uint32_t half = (cc + 1) / 2, groups = max(1u, (uint32_t)BS / (uint32_t)(SMALL / 2));
    const uint32_t e0 = threadIdx.x % (SMALL / 2), q = threadIdx.x / (SMALL / 2);
    const uint32_t flen = (cc + groups - 1) / groups;
    const uint32_t fb = min(cc, q * flen), fe = min(cc, fb + flen);
    for (uint32_t e = e0; e < half; e += min((uint32_t)BS, (uint32_t)(SMALL / 2))) {
      const uint32_t e2 = min(e + half, cc - 1);
      const uint64_t K0 = ck[e], K1 = ck[e2];
      const uint32_t I0 = cidx[e], I1 = cidx[e2];
      uint32_t r0 = 0, r1 = 0;
      for (uint32_t f0 = fb; f0 < fe; f0 += 8) {
        uint64_t Kf[8];
        uint32_t If[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const uint32_t f = min(f0 + (uint32_t)u, cc - 1);
          Kf[u] = ck[f];
          If[u] = cidx[f];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const bool in = f0 + (uint32_t)u < fe;
          r0 += (in & ((Kf[u] < K0) | ((Kf[u] == K0) & (If[u] < I0)))) ? 1u : 0u;
          r1 += (in & ((Kf[u] < K1) | ((Kf[u] == K1) & (If[u] < I1)))) ? 1u : 0u;
        }
      }
      if (r0) atomicAdd(&crnk[e], r0);
      if (r1 && e + half < cc) atomicAdd(&crnk[e2], r1);
    }
  }
  __syncthreads();
  for (uint32_t e = threadIdx.x; e < cc; e += BS) {
    const uint32_t rank = crnk[e], x = ccode[e];
    if (rank == r) { sh_kt = ck[e]; sh_it = cidx[e]; sh_pt = cpos[e]; sh_px = x; }
    if (rank <= r) atomicAdd(&pcnt[x / CHUNK / part], 1u);
    else if (flagged) clear_flag(x);
  }
  __syncthreads();
  if (sh_pt == NONE || ccount > SMALL) {
    if (threadIdx.x == 0) set_status(a, STATUS_INTERNAL);
    __syncthreads();
    return;
  }
  const uint64_t Kt = sh_kt;
  const uint32_t It = sh_it;
  const uint32_t pt = sh_pt, px = sh_px;
  if (threadIdx.x < WAVE) {
    // list offsets of the waves' parts (exclusive, candidate order)
    const uint32_t c = threadIdx.x < W ? pcnt[threadIdx.x] : 0u;
    const uint32_t inc = wave_incl_scan<uint32_t>(c);
    if (threadIdx.x < W) pcnt[threadIdx.x] = inc - c;
    if (threadIdx.x == WAVE - 1) sh_total = inc;
  }
  if (threadIdx.x == (BS > WAVE ? WAVE : 0)) {
    // the witness's tau
    const uint32_t kt = s.key[pt];
    const uint32_t snap_t = (a.n_snap > 1) ? (uint32_t)((uint64_t)kt >> (3 * a.D)) : 0u;
    const uint64_t Ut = particle_U(local_id(a, snap_t, s.idx[pt]), snap_t, a.seed);
    sh_tau = weight_pow(s.w[pt], a.alpha) * 4294967296.0 / (double)Ut;
  }
  __syncthreads();
  if (sh_total != n + 1) {
    if (threadIdx.x == 0) set_status(a, STATUS_INTERNAL);
    __syncthreads();
    return;
  }
  // the taken candidates' codes, in candidate (= sorted position) order: a lane
  // takes 1, 2 or 4 chunks, so that all lanes have some (few candidates are
  // mostly taken: eight codes per lane and step; of many, one in eight is)
  uint32_t *srow = sa.src + (uint64_t)blockIdx.x * (n + 1);
  {
    uint32_t run = pcnt[w];
    const uint32_t q = part > 512 ? 4u : part > 256 ? 2u : 1u;   // part is a multiple of 4
    for (uint32_t c0 = lo; c0 < hi; c0 += q * WAVE) {
      const uint32_t c = c0 + q * lane;
      uint32_t m = 0;
      if (flagged) {
        if (c < hi) {
          const uint32_t nc = min(q, hi - c);
          m = (hist[c / 4] >> (CHUNK * (c % 4))) & (0xFFFFFFFFu >> (32 - CHUNK * nc));
        }
      } else {
        for (uint32_t i = 0; i < q && c + i < hi; ++i) {
          const uint32_t ci = c + i, k = seg_of(g, ci);
          const uint4 x = *reinterpret_cast<const uint4 *>(g.kb[k] + (uint64_t)ci * CHUNK);
          uint32_t valid = 0xFFu, le, eq;
          if (ci == g.cst[k]) valid &= g.head[k];
          if (ci + 1 == g.cst[k + 1]) valid &= g.tail[k];
          compare_bins(x, b0, le, eq);
          le &= valid; eq &= valid;
          for (; eq; eq &= eq - 1u) {
            const uint32_t h = __builtin_ctz(eq);
            if (!taken_exact(a, s, cand_pos(g, sa, k, ci * CHUNK + h), Kt, It)) le &= ~(1u << h);
          }
          m |= le << (CHUNK * i);
        }
      }
      const uint32_t cnt = __popc(m);
      const uint32_t inc = wave_incl_scan<uint32_t>(cnt);
      uint32_t o = run + inc - cnt;
      run += (uint32_t)__builtin_amdgcn_readlane((int)inc, WAVE - 1);
      const uint32_t x0 = c * CHUNK;
      if (px - x0 < q * CHUNK && c < hi) sh_wj = o + __popc(m & ((1u << (px - x0)) - 1u));
      for (; m; m &= m - 1u, ++o)
        if (o <= n) srow[o] = x0 + __builtin_ctz(m);
    }
  }
  __syncthreads();
  // output pass, one taken candidate per lane: the list entry and the stored
  // point with its unscaled float64 mass, kept in this block's scratch row
  const double tau = sh_tau;
  const bool out_ok = a.counts[1] <= a.point_cap;
  const uint64_t lbase = (uint64_t)t.sel_idx[v] * (n + 1);
  uint32_t *out_pos = sa.lpos + lbase;
  uint16_t *out_kb = sa.lkb + lbase;
  uint2 *out_wm = sa.lwm + lbase;
  double *mrow = sa.mhat + (uint64_t)blockIdx.x * n;
  const uint64_t ob = t.pt_begin[v];
  const int d = t.depth[v];
  const uint32_t wj = sh_wj;
  for (uint32_t j0 = threadIdx.x; j0 <= n; j0 += BS * OILP) {
    // An entry of a child's list takes position, key bin, weight and mass from
    // that list and, unless it is the child's witness, id and codes from the
    // child's stored point (each code gains the child's octant bit on top).
    // The others are read from the sorted arrays.  Every load of a step is
    // issued before any is used; a wave without entries of one kind skips its
    // loads.
    uint32_t cx[OILP], ks[OILP];
    bool li[OILP];
#pragma unroll
    for (int u = 0; u < OILP; ++u) {
      cx[u] = srow[min(j0 + u * BS, n)];
      ks[u] = seg_of(g, cx[u] / CHUNK);
      li[u] = g.is_list[ks[u]] != 0;
    }
    uint32_t pos[OILP], kbv[OILP];
    uint2 wm[OILP];
    PointOut pq[OILP];
    bool any_list = false, any_sorted = false;
#pragma unroll
    for (int u = 0; u < OILP; ++u) {
      any_list |= li[u];
      any_sorted |= !li[u];
    }
    if (__ballot(any_list)) {
      uint32_t cq[OILP][3];
#pragma unroll
      for (int u = 0; u < OILP; ++u) {
        const uint32_t k = ks[u];
        const uint64_t i = li[u] ? g.adj[k] + cx[u] : 0u;
        // the child's stored point (a witness has none: some point in its place)
        const uint64_t ci = li[u] ? g.cob[k] + min(cx[u] - g.cx0[k] - (cx[u] > g.cwx[k] ? 1u : 0u), n - 1) : 0u;
        pos[u] = entry_pos(sa, i);
        kbv[u] = sa.lkb[i];
        wm[u] = sa.lwm[i];
        pq[u].id = t.pt_id[ci];
        cq[u][0] = t.qx[ci]; cq[u][1] = t.qy[ci]; cq[u][2] = t.qz[ci];
      }
#pragma unroll
      for (int u = 0; u < OILP; ++u) {
        const uint32_t oc = g.coct[ks[u]];
        pq[u].xy = ((cq[u][0] >> 1) | ((oc & 1u) << 15)) | (((cq[u][1] >> 1) | (((oc >> 1) & 1u) << 15)) << 16);
        pq[u].z = (cq[u][2] >> 1) | (((oc >> 2) & 1u) << 15);
        if (li[u] && cx[u] == g.cwx[ks[u]]) pq[u] = code_point(a, read_point(s, pos[u]), d);   // one per list
      }
    }
    if (__ballot(any_sorted)) {
      PointIn q[OILP];
      uint32_t kk[OILP], ww[OILP], mm[OILP];
#pragma unroll
      for (int u = 0; u < OILP; ++u) {
        const uint64_t p = li[u] ? (uint64_t)pt : g.adj[ks[u]] + cx[u];
        kk[u] = s.kb[p]; ww[u] = s.w[p]; mm[u] = __float_as_uint(s.m[p]);
        q[u] = read_point(s, p);
        if (!li[u]) pos[u] = (uint32_t)p;
      }
#pragma unroll
      for (int u = 0; u < OILP; ++u)
        if (!li[u]) { kbv[u] = kk[u]; wm[u] = make_uint2(ww[u], mm[u]); pq[u] = code_point(a, q[u], d); }
    }
#pragma unroll
    for (int u = 0; u < OILP; ++u) {
      const uint32_t jl = j0 + u * BS;
      if (jl > n) continue;
      out_pos[jl] = pos[u];
      out_kb[jl] = (uint16_t)kbv[u];
      out_wm[jl] = wm[u];
      if (!out_ok || jl == wj) continue;
      const uint32_t j = jl - (jl > wj ? 1u : 0u);
      store_codes(t, pq[u], ob + j);
      mrow[j] = unscaled_mass(__uint_as_float(wm[u].y), wm[u].x, a.alpha, tau);
    }
  }
  __syncthreads();
  if (out_ok) {
    const double tot = row_sum_fixed(mrow, n, cs64, &sh_mtot);
    const double scale = t.node_mass[v] / tot;
    for (uint32_t j0 = threadIdx.x; j0 < n; j0 += BS * SILP) {
      double mv[SILP];
#pragma unroll
      for (int u = 0; u < SILP; ++u) mv[u] = mrow[min(j0 + u * BS, n - 1)];
#pragma unroll
      for (int u = 0; u < SILP; ++u)
        if (j0 + u * BS < n) t.pt_mass[ob + j0 + u * BS] = (float)(scale * mv[u]);
    }
  }
  if (threadIdx.x == 0) { t.wit[v] = pt; sa.widx[v] = wj; }
  __syncthreads();
}

// mode 1: one launch per level, one block per selecting node of that level.
// The stored points of the leaves (needed by nothing in the build) are copied
// by the same launches, so that the copy fills the chip while a level's last
// nodes are being selected.  Block j of every launch owns the nodes
// v = k G + j (G blocks per launch, k = 0, 1, ...) and resumes at its cursor
// leaf_ctl[j].  Above level 0 a block copies only while the level still has
// nodes being selected (done count in leaf_ctl[G + d]), and a block that
// selected a node only once every block with a node has started (count in
// leaf_ctl[G + D + 1 + d]), so that copying never holds back the dispatch of a
// selecting block.  Level 0, launched last, copies what is left.  No block
// waits for another.  leaf_ctl starts at zero.
__global__ __launch_bounds__(1024) void k_select_level(BuildArgs a, TreeArgs t, Sorted s, SelArgs sa, int d,
                                                       uint32_t *leaf_ctl) {
  __shared__ uint32_t sh_go;
  const uint32_t b = t.lvl[d], e = t.lvl[d + 1];
  const uint32_t G = gridDim.x;
  uint32_t *done = leaf_ctl ? leaf_ctl + G : nullptr;
  uint32_t *started = leaf_ctl ? leaf_ctl + G + a.D + 1 : nullptr;
  // the level's selecting nodes by rank, so that the blocks with a node come first
  const uint32_t r0 = t.lsel[d];
  const uint32_t r1 = (uint32_t)min((uint64_t)t.lsel[d + 1], a.node_cap);
  const uint32_t sel_blocks = r1 > r0 ? min(G, r1 - r0) : 0u;
  if (started && blockIdx.x < sel_blocks && threadIdx.x == 0) atomicAdd(&started[d], 1u);
  for (uint32_t r = r0 + blockIdx.x; r < r1; r += G) {
    const uint32_t v = t.sel_node[r];
    if (v == NONE || v < b || v >= e || t.part_count[v] <= a.n) continue;
    // the selecting waves ahead of the copying ones in each CU's instruction
    // arbitration (the level ends with its last node, not with the copy)
    __builtin_amdgcn_s_setprio(2);
    select_node(a, t, s, sa, v);
    __builtin_amdgcn_s_setprio(0);
    if (done && threadIdx.x == 0) atomicAdd(&done[d], 1u);
  }
  if (!leaf_ctl) return;
  const uint32_t total = t.lsel[d + 1] - t.lsel[d];   // selecting nodes of this level
  if (d > 0 && blockIdx.x < sel_blocks) {
    __syncthreads();
    if (threadIdx.x == 0)
      sh_go = __hip_atomic_load(&started[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= sel_blocks;
    __syncthreads();
    if (!sh_go) return;
  }
  const uint32_t nn = t.lvl[a.D + 1];
  const bool cap_ok = a.counts[1] <= a.point_cap;
  uint32_t k = leaf_ctl[blockIdx.x];
  while (true) {
    const uint64_t v = (uint64_t)k * G + blockIdx.x;
    if (v >= nn) break;
    if (d > 0) {
      __syncthreads();
      if (threadIdx.x == 0)
        sh_go = __hip_atomic_load(&done[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < total;
      __syncthreads();
      if (!sh_go) break;
    }
    if (t.first_child[v] == NONE && t.part_count[v] <= a.n && cap_ok) copy_leaf_points(a, t, s, (uint32_t)v);
    ++k;
  }
  if (threadIdx.x == 0) leaf_ctl[blockIdx.x] = k;
}

// mode 0: one launch per selecting node.
__global__ __launch_bounds__(1024) void k_select_one(BuildArgs a, TreeArgs t, Sorted s, SelArgs sa, uint32_t v) {
  if (v >= t.lvl[a.D + 1] || t.part_count[v] <= a.n) return;
  select_node(a, t, s, sa, v);
}

// Selecting nodes none of whose children select: the starting points of the
// persistent schedule (flags for a compaction).
__global__ void k_bottom_flags(BuildArgs a, TreeArgs t, uint32_t *__restrict__ flag) {
  const uint32_t nn = t.lvl[a.D + 1];
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v <= a.node_cap;
       v += (uint64_t)gridDim.x * blockDim.x)
    flag[v] = (v < nn && t.part_count[v] > a.n && t.pend[v] == 0) ? 1u : 0u;
}

__global__ void k_bottom_write(BuildArgs a, const uint32_t *__restrict__ flag, const uint32_t *__restrict__ scan,
                               uint32_t *__restrict__ bottom, uint32_t *__restrict__ ctl) {
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < a.node_cap;
       v += (uint64_t)gridDim.x * blockDim.x)
    if (flag[v]) bottom[scan[v]] = (uint32_t)v;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl[0] = scan[a.node_cap];   // number of starting nodes
    ctl[1] = 0;                  // ticket
    ctl[2] = 0;                  // leaf-copy cursor
  }
}

// mode 2: one persistent launch over every selecting node of every level.
// A block takes a starting node by ticket (deepest first), reduces it (node
// mass, selection, output) and then, if it was the last of its parent's
// selecting children to finish, continues with the parent; otherwise it takes
// the next ticket.  Once the tickets are gone a block copies leaves, a chunk
// of nodes at a time from a shared cursor, until none are left.  No block
// ever waits for another, so the grid drains without spinning.  (Copying a
// chunk between tickets, or by only part of the grid, measured slower: it
// delays the starting nodes, and the climbs near the root gain little from
// the bandwidth left to them.)
//
// The eight XCDs do not share an L2, so a hand-off between blocks needs an
// agent-scope release by the writer (its lists, mass and witness written back
// to memory) and an agent-scope acquire by the climber.  A release writes the
// whole L2 of the XCD back, so a block issues one per node, from one wave,
// once every wave's stores have completed (a workgroup barrier alone does not
// wait for them); each wave of a climbing block acquires for itself.  A
// starting node's inputs come from earlier launches and need no acquire.
constexpr uint32_t LEAF_CHUNK = 8;   // nodes per leaf-copy grab

// Copies the leaves among the next LEAF_CHUNK nodes of the shared cursor;
// false once the cursor has passed every node (uniform over the block).
__device__ __forceinline__ bool copy_leaf_chunk(const BuildArgs &a, const TreeArgs &t, const Sorted &s,
                                                uint32_t *cursor, uint32_t &sh) {
  const uint32_t nn = t.lvl[a.D + 1];
  if (threadIdx.x == 0) sh = atomicAdd(cursor, LEAF_CHUNK);
  __syncthreads();
  const uint32_t v0 = sh;
  __syncthreads();
  if (v0 >= nn) return false;
  const bool cap_ok = a.counts[1] <= a.point_cap;
  const uint32_t v1 = min(nn, v0 + LEAF_CHUNK);
  for (uint32_t v = v0; v < v1; ++v)
    if (t.first_child[v] == NONE && t.part_count[v] <= a.n && cap_ok) copy_leaf_points(a, t, s, v);
  return true;
}

__global__ __launch_bounds__(1024) void k_select_persistent(BuildArgs a, TreeArgs t, Sorted s, SelArgs sa,
                                                            const uint32_t *__restrict__ bottom,
                                                            uint32_t *__restrict__ ctl) {
  __shared__ uint32_t sh_v;
  while (true) {
    if (threadIdx.x == 0) {
      // deepest starting nodes first, so that climbs overlap the remaining work
      const uint32_t tk = atomicAdd(&ctl[1], 1u);
      sh_v = tk < ctl[0] ? bottom[ctl[0] - 1 - tk] : NONE;
    }
    __syncthreads();
    uint32_t v = sh_v;
    __syncthreads();
    if (v == NONE) break;
    while (true) {
      select_node(a, t, s, sa, v);
      // publish this node's outputs before its parent can be claimed: every
      // wave waits for its own stores (vmcnt 0: stores count there on this
      // architecture), then one wave writes the L2 back
      __syncthreads();
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt 0; expcnt and lgkmcnt at their maxima
      __syncthreads();
      if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const uint32_t par = t.parent[v];
        uint32_t nxt = NONE;
        if (par != NONE && atomicSub(&t.pend[par], 1u) == 1u) nxt = par;
        sh_v = nxt;
      }
      __syncthreads();
      v = sh_v;
      __syncthreads();
      if (v == NONE) break;
      // every child of v has released its outputs: see them (select_node
      // sums v's mass from its children and reads their lists)
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
  }
  // leaves read only the sorted arrays and the node table, both written by
  // earlier launches
  while (copy_leaf_chunk(a, t, s, &ctl[2], sh_v)) {
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// host side

namespace lodh {

namespace {
__global__ void k_copy32(const uint32_t *__restrict__ a, uint32_t *__restrict__ b, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

template <typename T>
__global__ void k_fill(T *p, uint64_t n, T v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}
}  // namespace

void fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t st) {
  if (!n) return;
  const unsigned g = (unsigned)std::min<uint64_t>(1024, (n + 255) / 256);
  LOD_LAUNCH(k_fill<uint64_t>, dim3(g), dim3(256), 0, st, p, n, v);
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Blocks of the emit kernels: enough for the largest level.  A level below
// the roots holds at most 8 children of each splitting node above it, and the
// splitting nodes of a level hold more than n particles each, disjointly.
static unsigned emit_blocks(uint64_t N, uint32_t n, uint32_t n_snap) {
  const uint64_t max_level = std::max<uint64_t>(8 * (N / ((uint64_t)n + 1)), n_snap);
  return (unsigned)std::max<uint64_t>(1, (max_level + EMIT_NODES - 1) / EMIT_NODES);
}

static uint64_t pt_blocks(uint64_t node_cap) { return (node_cap + PT_NODES - 1) / PT_NODES; }
static uint64_t groups(uint64_t blocks) { return (blocks + GROUP - 1) / GROUP; }

BuildLayout build_layout(uint64_t N, const lod_params &p, uint32_t n_snap) {
  BuildLayout L{};
  const uint64_t Np = N ? N : 1;
  const uint64_t tiles = (Np + STILE - 1) / STILE;
  L.tiles = tiles;
  uint64_t per_level = N / ((uint64_t)p.n + 1);
  L.node_cap = (uint64_t)n_snap + 8ull * p.max_depth * per_level;
  if (L.node_cap == 0) L.node_cap = 1;
  L.point_cap = N + (uint64_t)p.n * p.max_depth * per_level;
  if (L.point_cap == 0) L.point_cap = 1;
  // selecting nodes of one level are disjoint and hold > n particles each
  const uint64_t max_sel = (uint64_t)(p.max_depth + 1) * per_level + n_snap;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  L.keyA = take(4 * Np); L.keyB = take(4 * Np);
  L.idxA = take(4 * Np); L.idxB = take(4 * Np);
  L.loA = take(4 * Np); L.loB = take(4 * Np);
  L.lzA = take(2 * Np); L.lzB = take(2 * Np);
  L.mA = take(4 * Np); L.mB = take(4 * Np);
  L.thist = take(4 * (size_t)RADIX * tiles);
  L.scan32 = take(4 * std::max(scan_tmp_elems<uint32_t>((uint64_t)RADIX * tiles),
                               scan_tmp_elems<uint32_t>(L.node_cap + 1)));
  L.pt_sums = take(8 * (size_t)pt_blocks(L.node_cap));
  L.w = take(4 * Np);
  L.kb = take(2 * Np + 16);            // bulk selection reads may overrun by 16 bytes
  L.lsel = take(4 * (size_t)(p.max_depth + 4));
  L.cs = take(4 * 9 * (size_t)L.node_cap);
  L.sel_idx = take(4 * (size_t)L.node_cap);
  L.sel_node = take(4 * (size_t)L.node_cap);
  L.wit = take(4 * (size_t)L.node_cap);
  L.pend = take(4 * (size_t)L.node_cap);
  L.bflag = take(4 * (size_t)(L.node_cap + 1));
  L.bscan = take(4 * (size_t)(L.node_cap + 1));
  L.bottom = take(4 * (size_t)L.node_cap);
  L.ctl = take(64);
  // lists: position and key bin of each entry (the key bins padded for the
  // 16-byte reads of the counting passes)
  L.lpos = take(4 * std::max<uint64_t>(1, max_sel * ((uint64_t)p.n + 1)));
  L.lkb = take(2 * std::max<uint64_t>(1, max_sel * ((uint64_t)p.n + 1)) + 16);
  L.lwm = take(8 * std::max<uint64_t>(1, max_sel * ((uint64_t)p.n + 1)));
  L.lhist = keeps_list_hist(p.n) ? take(2 * KBINS * max_sel) : 0;
  L.widx = take(4 * (size_t)L.node_cap);
  L.sel_rows = (uint32_t)std::min<uint64_t>(4096, N / ((uint64_t)p.n + 1) + n_snap + 1);
  L.mhat = take(8 * (size_t)L.sel_rows * p.n);
  L.src = take(4 * (size_t)L.sel_rows * ((uint64_t)p.n + 1));
  // zeroed by the build's first launch: level starts, leaf-copy cursors and
  // level counts, child totals of every level (blocks, groups), point totals
  L.lvl = take(4 * (size_t)(p.max_depth + 4));
  L.leafctl = take(4 * ((size_t)L.sel_rows + 2 * (p.max_depth + 1)));
  const size_t eb = emit_blocks(N, p.n, n_snap);
  L.emit_tot = take(8 * (eb + groups(eb)) * std::max(1u, p.max_depth));
  L.pt_gsums = take(8 * (size_t)groups(pt_blocks(L.node_cap)));
  L.zero_end = off;
  L.total = off;
  return L;
}

// A second stream of the device (default priority) and two events: the density
// kernel runs on it beside the tree construction, which does not read its
// output.  Created at the first build outside stream capture; a build captured
// before that runs on one stream.
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  // Held from the fork event's record on the caller's stream to the side
  // stream's wait on it: builds issued by several host threads then each
  // fork from their own stream.  The join needs no lock: a later record of
  // it lies later on the side stream, so waiting on it only waits longer.
  std::mutex mu;
};

static SideStream *side_stream(hipStream_t st) {
  static std::mutex mu;
  static SideStream per_dev[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(mu);
  SideStream &r = per_dev[dev];
  if (!r.s) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return nullptr;
    hipStream_t s = nullptr;
    hipEvent_t a = nullptr, b = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&a, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b, hipEventDisableTiming) != hipSuccess) {
      if (a) (void)hipEventDestroy(a);
      (void)hipStreamDestroy(s);
      return nullptr;
    }
    r.s = s; r.fork = a; r.join = b;
  }
  return &r;
}

int key_bits(const lod_params &p, uint32_t n_snap) {
  int sb = 0;
  while ((1ull << sb) < n_snap) ++sb;
  return 3 * (int)p.max_depth + sb;
}

lod_status launch_build(const lod_input &in, const lod_params &p, void *ws, const BuildLayout &L,
                        lod_tree &out, hipStream_t st) {
  char *W = (char *)ws;
  const uint64_t N = in.n_particles;
  const uint32_t n_snap = in.snap_offsets ? in.n_snapshots : 1;
  BuildArgs a{};
  a.N = N; a.n = p.n; a.D = (int)p.max_depth; a.shift_rho = 3 * ((int)p.max_depth - (int)p.density_level);
  a.alpha = p.alpha; a.seed = p.seed; a.n_snap = n_snap; a.snap_off = in.snap_offsets;
  a.node_cap = L.node_cap; a.point_cap = out.point_capacity; a.counts = out.counts;

  // a kernel instead of memsets: the build may be captured into a graph
  uint32_t *lvl = (uint32_t *)(W + L.lvl);
  const uint64_t n_zero = (L.zero_end - L.lvl) / 4;
  LOD_LAUNCH(k_build_init, dim3((unsigned)std::min<uint64_t>(1024, (n_zero + 255) / 256)), dim3(256), 0, st, a, lvl,
             n_zero);
  if (N == 0) return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;

  uint32_t *keyA = (uint32_t *)(W + L.keyA), *keyB = (uint32_t *)(W + L.keyB);
  uint32_t *idxA = (uint32_t *)(W + L.idxA), *idxB = (uint32_t *)(W + L.idxB);
  uint32_t *loA = (uint32_t *)(W + L.loA), *loB = (uint32_t *)(W + L.loB);
  uint16_t *lzA = (uint16_t *)(W + L.lzA), *lzB = (uint16_t *)(W + L.lzB);
  float *mA = (float *)(W + L.mA), *mB = (float *)(W + L.mB);
  uint32_t *thist = (uint32_t *)(W + L.thist);
  uint32_t *scan32 = (uint32_t *)(W + L.scan32);
  const uint64_t tiles = (N + STILE - 1) / STILE;
  const uint64_t hist_n = (uint64_t)RADIX * tiles;
  const uint64_t dtiles = (N + TILE - 1) / TILE;

  LOD_LAUNCH(k_keygen, dim3((unsigned)tiles), dim3(TB), 0, st, in.x, in.y, in.z, a, thist, tiles);
  const int kb = key_bits(p, n_snap);
  const int passes = std::max(1, (kb + 7) / 8);
  // pass 0 reads the particles (keys recomputed, ids implicit) and writes B
  device_scan_blocks<uint32_t>(thist, hist_n, scan32, st);
  LOD_LAUNCH(k_scatter<true>, dim3((unsigned)tiles), dim3(STB), 0, st, a, 0, thist, scan32, tiles,
             ScatterIn{nullptr, nullptr, nullptr, nullptr, in.x, in.y, in.z, in.mass}, keyB, idxB, loB, lzB, mB);
  uint32_t *ks = keyB, *is = idxB, *ls = loB; uint16_t *zs = lzB; float *ms = mB;
  uint32_t *kd = keyA, *id = idxA, *ld = loA; uint16_t *zd = lzA; float *md = mA;
  for (int ps = 1; ps < passes; ++ps) {
    LOD_LAUNCH(k_upsweep, dim3((unsigned)tiles), dim3(TB), 0, st, ks, N, 8 * ps, thist, tiles);
    device_scan_blocks<uint32_t>(thist, hist_n, scan32, st);
    LOD_LAUNCH(k_scatter<false>, dim3((unsigned)tiles), dim3(STB), 0, st, a, 8 * ps, thist, scan32, tiles,
               ScatterIn{ks, is, ls, zs, nullptr, nullptr, nullptr, ms}, kd, id, ld, zd, md);
    std::swap(ks, kd); std::swap(is, id); std::swap(ls, ld); std::swap(zs, zd); std::swap(ms, md);
  }
  Sorted s{ks, is, ls, zs, ms, (const uint32_t *)(W + L.w), (const uint16_t *)(W + L.kb)};

  // density weights and key bins on the side stream, beside the tree
  // construction; joined before the selection
  SideStream *side = side_stream(st);
  hipStream_t dst = st;
  if (side) {
    std::lock_guard<std::mutex> lk(side->mu);
    if (hipEventRecord(side->fork, st) != hipSuccess || hipStreamWaitEvent(side->s, side->fork, 0) != hipSuccess)
      return LOD_EDEVICE;
    dst = side->s;
  }
  LOD_LAUNCH_NAMED("k_density", n_snap > 1 ? k_density<true> : k_density<false>, dim3((unsigned)dtiles), dim3(TB), 0, dst, a, ks, is,
             (uint32_t *)(W + L.w), (uint16_t *)(W + L.kb));
  if (side && hipEventRecord(side->join, side->s) != hipSuccess) return LOD_EDEVICE;

  TreeArgs t{};
  t.prefix = out.prefix; t.depth = out.depth; t.parent = out.parent; t.first_child = out.first_child;
  t.child_mask = out.child_mask; t.part_begin = out.part_begin; t.part_count = out.part_count;
  t.pt_begin = out.pt_begin; t.pt_count = out.pt_count; t.node_mass = out.node_mass;
  t.pt_id = out.pt_id; t.qx = out.qx; t.qy = out.qy; t.qz = out.qz; t.pt_mass = out.pt_mass;
  t.lvl = lvl; t.cs = (uint32_t *)(W + L.cs); t.sel_idx = (uint32_t *)(W + L.sel_idx);
  t.sel_node = (uint32_t *)(W + L.sel_node);
  t.wit = (uint32_t *)(W + L.wit); t.pend = (uint32_t *)(W + L.pend); t.lsel = (uint32_t *)(W + L.lsel);

  const int D = (int)p.max_depth;
  const uint64_t per_level = N / ((uint64_t)p.n + 1) + n_snap;
  // nodes of a level: at most 8 per node above, and emit_blocks' bound
  const unsigned emit_grid = emit_blocks(N, p.n, n_snap);
  auto level_nodes = [&](int d) {
    return std::min<uint64_t>((uint64_t)n_snap << std::min(3 * d, 32), (uint64_t)emit_grid * EMIT_NODES);
  };
  int top = 0;
  while (top < D && level_nodes(top) <= TOP_NODES) ++top;
  LOD_LAUNCH(k_tree_top, dim3(1), dim3(1024), 0, st, a, t, ks, top);
  for (int d = top; d < D; ++d) {
    uint32_t *tot = (uint32_t *)(W + L.emit_tot) + 2 * (size_t)(emit_grid + groups(emit_grid)) * d;
    uint32_t *gtot = tot + 2 * (size_t)emit_grid;
    const uint64_t ln = level_nodes(d);
    LOD_LAUNCH(k_tree_search, dim3((unsigned)std::min<uint64_t>(4096, (ln * WAVE + EMIT_BT - 1) / EMIT_BT)),
               dim3(EMIT_BT), 0, st, a, t, ks, d, tot, gtot);
    LOD_LAUNCH(k_tree_write, dim3((unsigned)((ln + EMIT_NODES - 1) / EMIT_NODES)), dim3(EMIT_BT), 0, st, a, t, d,
               (const uint2 *)tot, (const uint2 *)gtot);
  }
  const unsigned pt_grid = (unsigned)pt_blocks(L.node_cap);
  uint64_t *pt_sums = (uint64_t *)(W + L.pt_sums), *pt_gsums = (uint64_t *)(W + L.pt_gsums);
  LOD_LAUNCH(k_pt_scan, dim3(pt_grid), dim3(PT_NODES), 0, st, a, t, D, pt_sums, (unsigned long long *)pt_gsums);
  LOD_LAUNCH(k_pt_finish, dim3(pt_grid), dim3(PT_NODES), 0, st, a, t, D, pt_sums, pt_gsums);

  const unsigned node_grid = (unsigned)std::min<uint64_t>(8192, L.node_cap);
  // the per-level and persistent schedules copy the leaves' points inside
  // their selection launches
  uint32_t *leaf_ctl = p.mode == 1 ? (uint32_t *)(W + L.leafctl) : nullptr;
  if (p.mode == 0) {
    LOD_LAUNCH(k_leaves<true>, dim3(node_grid), dim3(TB), 0, st, a, t, s);
  } else {
    LOD_LAUNCH(k_leaves<false>, dim3(node_grid), dim3(TB), 0, st, a, t, s);
  }
  if (side && hipStreamWaitEvent(st, side->join, 0) != hipSuccess) return LOD_EDEVICE;

  SelArgs sa{(uint32_t *)(W + L.lpos), (uint16_t *)(W + L.lkb), (uint2 *)(W + L.lwm), (uint32_t)(N - 1),
             keeps_list_hist(p.n) ? (uint16_t *)(W + L.lhist) : nullptr, (uint32_t *)(W + L.widx),
             (double *)(W + L.mhat), (uint32_t *)(W + L.src)};
  const unsigned sel_threads = p.select_threads ? p.select_threads : 1024;
  // one scratch row of float64 masses per block
  const unsigned sel_grid = (unsigned)std::min<uint64_t>(L.sel_rows, per_level + 1);
  if (p.mode == 2) {
    uint32_t *bflag = (uint32_t *)(W + L.bflag), *bscan = (uint32_t *)(W + L.bscan);
    uint32_t *ctl = (uint32_t *)(W + L.ctl);
    const unsigned fg = (unsigned)std::min<uint64_t>(4096, (L.node_cap + 256) / 256);
    LOD_LAUNCH(k_bottom_flags, dim3(fg), dim3(256), 0, st, a, t, bflag);
    LOD_LAUNCH(k_copy32, dim3(fg), dim3(256), 0, st, bflag, bscan, L.node_cap + 1);
    device_scan<uint32_t>(bscan, L.node_cap + 1, (uint32_t *)(W + L.scan32), st);
    LOD_LAUNCH(k_bottom_write, dim3(fg), dim3(256), 0, st, a, bflag, bscan, (uint32_t *)(W + L.bottom), ctl);
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return LOD_EDEVICE;
    const unsigned pgrid = std::min<unsigned>(L.sel_rows, p.persistent_blocks ? p.persistent_blocks
                                                                              : (unsigned)(2 * cus));
    LOD_LAUNCH(k_select_persistent, dim3(pgrid), dim3(sel_threads), 0, st, a, t, s, sa,
               (const uint32_t *)(W + L.bottom), ctl);
    return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
  }
  // the per-node reference schedule needs the level sizes on the host
  std::vector<uint32_t> hl;
  std::vector<uint64_t> hcount;
  if (p.mode == 0) {
    hl.resize(D + 4);
    if (hipMemcpyAsync(hl.data(), lvl, 4 * (D + 4), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
      return LOD_EDEVICE;
    hcount.resize(hl[D + 1] + 1);
    if (hl[D + 1] &&
        (hipMemcpyAsync(hcount.data(), out.part_count, 8ull * hl[D + 1], hipMemcpyDeviceToHost, st) != hipSuccess ||
         hipStreamSynchronize(st) != hipSuccess))
      return LOD_EDEVICE;
  }
  for (int d = D; d >= 0; --d) {
    if (p.mode == 0) {
      for (uint32_t v = hl[d]; v < hl[d + 1]; ++v) {
        if (hcount[v] <= p.n) continue;
        LOD_LAUNCH(k_select_one, dim3(1), dim3(sel_threads), 0, st, a, t, s, sa, v);
      }
    } else {
      // a level of at most 64 nodes cannot fill the chip: give each node 1024 threads
      const bool few = d <= 2 && ((uint64_t)n_snap << (3 * d)) <= 64;
      LOD_LAUNCH(k_select_level, dim3(sel_grid), dim3(few ? 1024u : sel_threads), 0, st, a, t, s, sa, d,
                 leaf_ctl);
    }
  }
  return hipGetLastError() == hipSuccess ? LOD_OK : LOD_EDEVICE;
}

void *workspace_view(void *ws, const BuildLayout &L, uint32_t which, uint64_t N, int passes, uint64_t *count) {
  char *W = (char *)ws;
  const bool inB = (passes % 2) == 1;
  switch (which) {
    case 0: *count = N; return W + (inB ? L.keyB : L.keyA);
    case 1: *count = N; return W + (inB ? L.idxB : L.idxA);
    case 2: *count = N; return W + L.w;
    case 3: *count = N; return W + L.kb;
    case 4: *count = L.node_cap; return W + L.wit;
    default: *count = 0; return nullptr;
  }
}

}  // namespace lodh
