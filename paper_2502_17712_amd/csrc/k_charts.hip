// Chart stages of the per-frame path on gfx950:
//   clip transform, union-find charts (Appendix "GPU Union Find", Alg. 1),
//   root compaction, per-triangle conservative boxes (Sec. "Computing Bounding
//   Boxes of Projected Visible Sub-Charts") reduced per chart.
//
// Visible triangles are a small fraction of a scene (about 13% of the 2.2M
// triangles of a 4K frame), so the prologue compacts them once, in ascending
// index order, into a dense list; every later per-triangle kernel walks that
// list with full waves instead of masking out invisible lanes.
#include <algorithm>
#include <climits>
#include <cstddef>
#include <type_traits>

#include "fa_internal.h"

namespace fa {
namespace {

// ---------------------------------------------------------------------------
// union-find over visible triangles. parent[x] <= x always holds; a root has
// parent[x] == x. Walks inside a join use plain loads: a stale value (the
// eight XCDs have separate L2 caches) is an older ancestor, and the hooking
// compare-and-swap always sees the current value. Reads whose value is the
// result (vertex minima, the flattened root, the root test) are agent-scope
// atomic loads; every write of parent[] is an agent-scope atomic store.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int aload(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void astore(int32_t* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int uf_root(int32_t* parent, int x) {
  int cur = parent[x];
  if (cur == x) return x;
  int prev = x;
  for (;;) {
    int nxt = parent[cur];
    if (nxt >= cur) return cur;  // parent[cur] == cur
    astore(&parent[prev], nxt);
    prev = cur;
    cur = nxt;
  }
}

// The roots of u and of v by uf_root's walk, the two walks advancing
// together so that their dependent loads overlap.
__device__ __forceinline__ void uf_root2(int32_t* parent, int u, int v, int& ru, int& rv) {
  int cu = parent[u], cv = parent[v], pu = u, pv = v;
  bool du = cu == u, dv = cv == v;
  while (!(du && dv)) {
    const int nu = du ? cu : parent[cu];
    const int nv = dv ? cv : parent[cv];
    if (!du) {
      if (nu >= cu) {
        du = true;
      } else {
        astore(&parent[pu], nu);
        pu = cu;
        cu = nu;
      }
    }
    if (!dv) {
      if (nv >= cv) {
        dv = true;
      } else {
        astore(&parent[pv], nv);
        pv = cv;
        cv = nv;
      }
    }
  }
  ru = cu;
  rv = cv;
}

// Join the trees of u and v: the larger root is hooked below the smaller one
// with a compare-and-swap; on failure continue from the value that won.
__device__ __forceinline__ void uf_join(int32_t* parent, int u, int v) {
  int ru, rv;
  uf_root2(parent, u, v, ru, rv);
  while (ru != rv) {
    if (ru < rv) {
      int old = atomicCAS(&parent[rv], rv, ru);
      if (old == rv) return;
      rv = old;
    } else {
      int old = atomicCAS(&parent[ru], ru, rv);
      if (old == ru) return;
      ru = old;
    }
  }
}

constexpr int kProVerts = 16;  // vertices per prologue thread
constexpr int kTilesPer = kBlock / kWave;  // triangle tiles per workgroup: one a wave
constexpr int kTileSteps = kTriTile / (4 * kWave);  // four triangles a lane each
// Added to the visible count of a tile that holds a bad index: sums of counts
// stay below it, and a sum of every tile's stays below 2^32.
constexpr uint32_t kBadTile = 1u << 17;
static_assert(FA_STATIC_MAX_TRIANGLES < (int64_t)kBadTile &&
                  (FA_STATIC_MAX_TRIANGLES / kTriTile + 2) * (int64_t)kBadTile < (int64_t(1) << 32),
              "kBadTile separates counts from bad tiles");

inline __host__ __device__ bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Fill x[i .. i + 4) below n (i a multiple of four; wide: x is 16-byte aligned).
__device__ __forceinline__ void fill4(int32_t* __restrict__ x, int64_t i, int64_t n, int32_t v,
                                      bool wide) {
  if (wide && i + 4 <= n) {
    *reinterpret_cast<int4*>(x + i) = make_int4(v, v, v, v);
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i + e < n) x[i + e] = v;
}

// Which of the triangles [t, t + 4) below T are visible, as four bits (t a
// multiple of four; wide: vis is 4-byte aligned).
__device__ __forceinline__ uint32_t visible4(const uint8_t* __restrict__ vis, int64_t t, int64_t T,
                                             bool wide) {
  uint32_t m = 0;
  if (wide && t + 4 <= T) {
    const uint32_t x = *reinterpret_cast<const uint32_t*>(vis + t);
#pragma unroll
    for (int e = 0; e < 4; ++e) m |= ((x >> (8 * e)) & 0xFFu) ? 1u << e : 0u;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) m |= t + e < T && vis[t + e] ? 1u << e : 0u;
  }
  return m;
}

// The neighbours of the triangles [t, t + 4) below T (t a multiple of four; nbr
// comes from an allocation of its own, so four triangles' are three aligned
// words); -1 past the end.
__device__ __forceinline__ void neighbours4(const int32_t* __restrict__ nbr, int64_t t, int64_t T,
                                            int (&n)[12]) {
  if (t + 4 <= T) {
    const int4* w = reinterpret_cast<const int4*>(nbr + 3 * t);
    const int4 a = w[0], b = w[1], c = w[2];
    n[0] = a.x; n[1] = a.y; n[2] = a.z; n[3] = a.w;
    n[4] = b.x; n[5] = b.y; n[6] = b.z; n[7] = b.w;
    n[8] = c.x; n[9] = c.y; n[10] = c.z; n[11] = c.w;
    return;
  }
#pragma unroll
  for (int e = 0; e < 12; ++e) n[e] = t + e / 3 < T ? nbr[3 * t + e] : -1;
}

// Prologue of a frame: frame state, per-vertex scratch (vertex minima and
// chart_of_vert = -1; clip positions are computed where they are read),
// chart_of_tri = -1, the union-find start of every visible triangle and the
// visible count of every tile of kTriTile triangles. With check_idx (the
// allocation-free entry point, whose indices no resident scene has checked) a
// tile with an index outside [0, V) adds kBadTile to its count. Blocks
// [0, vblocks) handle vertices, the rest triangle tiles, one a wave. Bound by
// the stores: 16 bytes a lane each, and few enough workgroups that starting
// them does not count (with one tile or 1024 vertices a workgroup in single
// words 2.2M triangles took 8.1 us, now 6.5, and the compaction 7.4, now 5.3;
// 16 views 102 and 45, now 84 and 20). UF_INIT 2: a visible triangle
// starts linked to the smallest of itself and its visible edge neighbours
// (Alg. 1, first loop); 1: as its own root (same labels); 0: not written (a
// later pass writes it). The neighbours are a chain of two loads a triangle, so
// they want waves: a tile a workgroup then (2.2M triangles: a tile a wave 26 us,
// so 11.0; one word at a time, a tile a workgroup, 12.6).
template <int UF_INIT>
__device__ __forceinline__ void k_prologue_body(int64_t V, int32_t* __restrict__ vmin,
                           int32_t* __restrict__ cov, const uint8_t* __restrict__ vis,
                           const int32_t* __restrict__ nbr, int64_t T,
                           int32_t* __restrict__ parent, int32_t* __restrict__ cot,
                           uint32_t* __restrict__ tile_vis,
                           unsigned vblocks, FrameState* st,
                           unsigned long long* __restrict__ big_counter,
                           const int32_t* __restrict__ check_idx = nullptr) {
  if (blockIdx.x < vblocks) {
    if (blockIdx.x == 0) {
      // (FA_OK is 0)
      static_assert(sizeof(FrameState) % 4 == 0 && FA_OK == 0, "the state clears word by word");
      for (unsigned i = threadIdx.x; i < sizeof(FrameState) / 4; i += blockDim.x)
        reinterpret_cast<uint32_t*>(st)[i] = 0u;
      if (threadIdx.x == 0) *big_counter = 0ull;
    }
    const int64_t v0 = (int64_t)blockIdx.x * (kBlock * kProVerts) + 4 * threadIdx.x;
    const bool wide_min = aligned16(vmin), wide_cov = aligned16(cov);
#pragma unroll
    for (int k = 0; k < kProVerts / 4; ++k) {
      const int64_t v = v0 + (int64_t)k * 4 * kBlock;
      fill4(vmin, v, V, INT_MAX, wide_min);
      fill4(cov, v, V, -1, wide_cov);
    }
    return;
  }
  // (with neighbours to look up, a step of the tile by each wave)
  constexpr int kSteps = UF_INIT == 2 ? 1 : kTileSteps;
  static_assert(kTileSteps == kTilesPer, "a wave takes a tile or a step of one");
  const int w = threadIdx.x / kWave;
  const int64_t tile = UF_INIT == 2 ? (int64_t)(blockIdx.x - vblocks)
                                    : (int64_t)(blockIdx.x - vblocks) * kTilesPer + w;
  if (tile * kTriTile >= T) return;
  const int64_t t0 = tile * kTriTile + 4 * lane_id() + (UF_INIT == 2 ? w * 4 * kWave : 0);
  const bool wide_vis = ((uintptr_t)vis & 3u) == 0, wide_cot = aligned16(cot);
  uint32_t m[kSteps];
#pragma unroll
  for (int k = 0; k < kSteps; ++k) m[k] = visible4(vis, t0 + k * 4 * kWave, T, wide_vis);
  uint32_t nv = 0;
#pragma unroll
  for (int k = 0; k < kSteps; ++k) {
    const int64_t t = t0 + k * 4 * kWave;
    fill4(cot, t, T, -1, wide_cot);
    nv += (uint32_t)__popc(m[k]);
    if (UF_INIT != 2 && check_idx) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (t + j >= T) break;
        const int3 v = reinterpret_cast<const int3*>(check_idx)[t + j];
        if (v.x < 0 || v.x >= V || v.y < 0 || v.y >= V || v.z < 0 || v.z >= V)
          nv += 2 * kTriTile;  // (a tile counts at most kTriTile visible)
      }
    }
    if (UF_INIT == 0) continue;
    int q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = (int)(t + j);
    if (UF_INIT == 2 && m[k]) {
      // four triangles' neighbours, then the bytes of all of them, in flight together
      int n[12];
      neighbours4(nbr, t, T, n);
      uint32_t seen = 0;
#pragma unroll
      for (int e = 0; e < 12; ++e)
        seen |= (m[k] >> (e / 3) & 1u) && n[e] >= 0 && vis[n[e]] ? 1u << e : 0u;
#pragma unroll
      for (int e = 0; e < 12; ++e) q[e / 3] = seen >> e & 1u ? min(q[e / 3], n[e]) : q[e / 3];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (m[k] >> j & 1u) astore(&parent[t + j], q[j]);
  }
  if (UF_INIT == 2) {
    __shared__ uint32_t sh[kBlock / kWave];
    nv = block_sum<uint32_t>(nv, sh);
    if (threadIdx.x == 0) tile_vis[tile] = nv;
    return;
  }
  nv = wave_sum<uint32_t>(nv);
  if (check_idx) nv = nv % (2 * kTriTile) + (nv >= 2 * kTriTile ? kBadTile : 0u);
  if (lane_id() == 0) tile_vis[tile] = nv;
}
template <int UF_INIT>
__global__ void k_prologue(int64_t V, int32_t* __restrict__ vmin,
                           int32_t* __restrict__ cov, const uint8_t* __restrict__ vis,
                           const int32_t* __restrict__ nbr, int64_t T,
                           int32_t* __restrict__ parent, int32_t* __restrict__ cot,
                           uint32_t* __restrict__ tile_vis,
                           unsigned vblocks, FrameState* st,
                           unsigned long long* __restrict__ big_counter,
                           const int32_t* __restrict__ check_idx) {
  k_prologue_body<UF_INIT>(V, vmin, cov, vis, nbr, T, parent, cot, tile_vis, vblocks, st,
                           big_counter, check_idx);
}

// Sum of cnt[0 .. n) by one workgroup (the exclusive prefix of tile n);
// each thread issues eight loads before it adds any.
__device__ __forceinline__ uint32_t tiles_before(const uint32_t* __restrict__ cnt, int64_t n,
                                                 uint32_t* sh) {
  uint32_t v = 0;
  for (int64_t u0 = threadIdx.x; u0 < n; u0 += 8 * (int64_t)blockDim.x) {
    uint32_t x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t u = u0 + (int64_t)j * blockDim.x;
      x[j] = u < n ? cnt[u] : 0u;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) v += x[j];
  }
  return block_sum<uint32_t>(v, sh);
}

// Exclusive prefix of the tiles' visible counts, in place, by one
// workgroup: each thread takes kScanPer consecutive tiles, one block scan
// (the compaction of a batched launch then reads its tile's offset instead of
// summing every earlier tile, which with many views in one launch costs more
// than this extra launch; one frame keeps the sums).
constexpr int kScanPer = 4;
__device__ __forceinline__ void k_tile_scan_body(uint32_t* tile_vis, unsigned tiles) {
  __shared__ uint32_t sh[1024 / kWave];
  uint32_t run = 0;
  for (unsigned b0 = 0; b0 < tiles; b0 += blockDim.x * kScanPer) {
    const unsigned i0 = b0 + threadIdx.x * kScanPer;
    uint32_t v[kScanPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = i0 + k < tiles ? tile_vis[i0 + k] : 0u;
      mine += v[k];
    }
    uint32_t tot;
    uint32_t at = run + block_incl_scan<uint32_t>(mine, sh, &tot) - mine;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (i0 + k < tiles) tile_vis[i0 + k] = at;
      at += v[k];
    }
    run += tot;
  }
}

// Stable compaction of the visible triangles into vlist (ascending index), a
// tile by each wave. For one frame each workgroup sums the visible counts of
// the tiles before its own (a few thousand words at most) instead of waiting
// for a separate scan; batched launches scan first (scanned). The last tile's
// wave records the total; of a checked frame with a bad index (kBadTile) it ends the frame
// with FA_ERR_INVALID_ARG.
__device__ __forceinline__ void k_vis_compact_body(const uint8_t* __restrict__ vis, int64_t T,
                              const uint32_t* __restrict__ tile_vis, int32_t* __restrict__ vlist,
                              FrameState* __restrict__ st, bool scanned = false,
                              bool checked = false) {
  __shared__ uint32_t sh[kBlock / kWave];
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int64_t tiles = (T + kTriTile - 1) / kTriTile;
  const int64_t first = (int64_t)blockIdx.x * kTilesPer, tile = first + w;
  const int64_t t0 = tile * kTriTile + 4 * lane;
  const bool wide = ((uintptr_t)vis & 3u) == 0;
  uint32_t m[kTileSteps];
#pragma unroll
  for (int k = 0; k < kTileSteps; ++k) m[k] = visible4(vis, t0 + k * 4 * kWave, T, wide);
  uint32_t off;
  if (scanned) {  // tile_vis holds each tile's exclusive prefix (k_tile_scan_body)
    if (tile >= tiles) return;
    off = tile_vis[tile];
  } else {
    off = tiles_before(tile_vis, first, sh);
    if (tile >= tiles) return;
    for (int j = 0; j < w; ++j) off += tile_vis[first + j];
  }
  const uint32_t bad = checked ? off / kBadTile : 0u;  // earlier tiles with a bad index
  if (checked) off %= kBadTile;
  // two steps' counts a scan (a step has at most 256)
#pragma unroll
  for (int k = 0; k < kTileSteps; k += 2) {
    const uint32_t c = (uint32_t)__popc(m[k]) | (uint32_t)__popc(m[k + 1]) << 16;
    const uint32_t incl = wave_incl_scan_dpp(c);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const uint32_t before = incl - c;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t at = off + (h ? before >> 16 : before & 0xFFFFu);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (m[k + h] >> j & 1u) vlist[at++] = (int32_t)(t0 + (k + h) * 4 * kWave + j);
      off += h ? tot >> 16 : tot & 0xFFFFu;
    }
  }
  if (tile == tiles - 1 && lane == 0) {
    if (checked && (bad || tile_vis[tile] >= kBadTile)) {
      st->status = FA_ERR_INVALID_ARG;  // and an empty list: no later kernel reads an index
      st->visible = 0;
    } else {
      st->visible = (int32_t)off;
    }
  }
}
static_assert(kTileSteps % 2 == 0, "the compaction scans two steps at a time");
__global__ void k_vis_compact(const uint8_t* __restrict__ vis, int64_t T,
                              const uint32_t* __restrict__ tile_vis, int32_t* __restrict__ vlist,
                              FrameState* __restrict__ st, bool checked) {
  k_vis_compact_body(vis, T, tile_vis, vlist, st, false, checked);
}

// Threads per vertex-hook workgroup: one workgroup's pair set then covers
// 1024 list entries (four times the repeats of 256-thread workgroups; one
// frame's hook 21.6 -> 19.7 us).
constexpr unsigned kHookThreads = 1024;

// Ordered (a, b) pairs that a workgroup has joined or is joining: a repeated
// pair needs no second join.
constexpr int kPairSlots = 512;
__device__ __forceinline__ void pairs_clear(unsigned long long* pairs) {
  for (int h = threadIdx.x; h < kPairSlots; h += blockDim.x) pairs[h] = ~0ull;
  __syncthreads();
}
__device__ __forceinline__ void join_once(unsigned long long* pairs, int32_t* parent, int a,
                                          int b) {
  const unsigned long long key = ((unsigned long long)(uint32_t)a << 32) | (uint32_t)b;
  uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 40) & (kPairSlots - 1);
  bool fresh = true;
  // (as a loop: unrolled, the vertex hook of one million triangles took 61 us
  // in place of 56, and without the tiles' joins before it 375 in place of 315)
#pragma unroll 1
  for (int probe = 0; probe < 16; ++probe) {
    const unsigned long long old = atomicCAS(&pairs[h], ~0ull, key);
    if (old == ~0ull) break;
    if (old == key) {
      fresh = false;
      break;
    }
    h = (h + 1) & (kPairSlots - 1);
  }
  if (fresh) uf_join(parent, a, b);  // a full table only costs extra joins
}

// Edges of more than two triangles (FANS): nbr goes from one to the next and
// from the last to the first, so a hidden triangle is passed over to the next
// visible one, or -1 where there is none but t. Each edge's visible triangles
// are then joined in a row. n: the neighbour of t across its edge e.
__device__ __forceinline__ int next_visible(const int32_t* __restrict__ idx,
                                            const int32_t* __restrict__ nbr,
                                            const uint8_t* __restrict__ vis, int t, int e, int n,
                                            int64_t T) {
  // (an edge is walked once around at most)
  for (int64_t step = 0; step < T && n >= 0 && n != t && !vis[n]; ++step) {
    const int k = same_edge(idx, t, e, n);
    n = k < 0 ? -1 : nbr[3 * (int64_t)n + k];
  }
  return n == t ? -1 : n;
}

// Hook across every shared edge once (u < v) (Alg. 1, second loop).
// With tile > 0 only edges leaving the entry's tile of `tile` consecutive
// list entries are hooked (the others were joined inside the tile).
template <bool FANS>
__global__ void k_uf_hook(const uint8_t* __restrict__ vis, const int32_t* __restrict__ nbr,
                          const int32_t* __restrict__ vlist, int32_t* parent, int tile,
                          const FrameState* __restrict__ st, const int32_t* __restrict__ mesh_idx,
                          int64_t T) {
  const int nv = st->visible;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    const int t = vlist[i];
    const int last = tile > 0 ? vlist[min(nv, (i / tile + 1) * tile) - 1] : -1;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      int n = nbr[3 * (int64_t)t + e];
      if (FANS) n = next_visible(mesh_idx, nbr, vis, t, e, n, T);
      if (n > t && n > last && vis[n]) uf_join(parent, t, n);
    }
  }
}

// Edges between tiles, after the LDS pass: an edge (t, n) joins the sets of
// parent[t] and parent[n] (ancestors of t and n). Lanes of a wave whose edges
// name the same pair of parents keep only the lowest lane, and a workgroup
// takes a pair once, so a pair that many edges along a tile border share is not
// hooked by every lane contending for the same root. Bound by the chain of
// loads and the walks of the joins; the loads of a triangle's three edges go
// out together.
template <bool FANS>
__global__ __launch_bounds__(kHookThreads) void k_uf_cross(
    const uint8_t* __restrict__ vis, const int32_t* __restrict__ nbr,
    const int32_t* __restrict__ vlist, int32_t* parent, int tile,
    const FrameState* __restrict__ st, const int32_t* __restrict__ mesh_idx, int64_t T) {
  __shared__ unsigned long long pairs[kPairSlots];
  pairs_clear(pairs);
  const int nv = st->visible;
  const int lane = lane_id();
  for (int i0 = blockIdx.x * blockDim.x; i0 < nv; i0 += gridDim.x * blockDim.x) {
    const int i = i0 + threadIdx.x;
    const bool valid = i < nv;
    const int t = valid ? vlist[i] : 0;
    const int last = valid ? vlist[min(nv, (i / tile + 1) * tile) - 1] : 0;
    int n[3] = {-1, -1, -1};
    if (valid) {
      const int3 x = reinterpret_cast<const int3*>(nbr)[t];
      n[0] = x.x; n[1] = x.y; n[2] = x.z;
      if (FANS) {
#pragma unroll
        for (int e = 0; e < 3; ++e) n[e] = next_visible(mesh_idx, nbr, vis, t, e, n[e], T);
      }
    }
    // the three edges' loads together (a hidden neighbour's parent is read in
    // vain)
    const int pt = valid ? aload(&parent[t]) : 0;
    bool seen[3];
    int pn[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const bool out = valid && n[e] > last;
      seen[e] = false;
      pn[e] = pt;
      if (out) {
        seen[e] = vis[n[e]] != 0;
        pn[e] = aload(&parent[n[e]]);
      }
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const bool want = seen[e] && pn[e] != pt;
      const int a = min(pt, pn[e]), b = max(pt, pn[e]);
      // keep the lowest lane of every distinct (a, b)
      unsigned long long todo = __ballot(want);
      bool keep = false;
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int la = __builtin_amdgcn_readlane(a, leader), lb = __builtin_amdgcn_readlane(b, leader);
        if (lane == leader) keep = true;
        todo &= ~__ballot(want && a == la && b == lb);
      }
      if (keep) join_once(pairs, parent, a, b);
    }
  }
}

// Edge hooks inside one tile of TILE consecutive entries of the visible
// list, in LDS: entries are local indices (ascending with the triangle index),
// a shared edge whose other triangle lies in the tile joins the two local sets
// (larger local root hooked below the smaller by compare-and-swap). Then every
// entry's parent becomes the smallest triangle of its local set, which is a
// valid union-find start for the vertex passes; edges leaving the tile are
// shared vertices too, so those passes complete the charts.
// Bound by the latency of the loads and LDS walks, so a tile has few entries a
// thread (two of 2048: more of them end their turns one after another), whose
// loads go out together, and a neighbour's entry is looked for where it is if
// everything in between is visible before it is searched for. Edge-connected
// charts of 1.1M city triangles: 29 us with tiles of 4096 searched in full, 14
// so; whole frames of 5k to 2.2M triangles of three scenes take 5 to 25% less.

__device__ __forceinline__ int lds_get(int* a, int i) {
  return __hip_atomic_load(&a[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_put(int* a, int i, int v) {
  __hip_atomic_store(&a[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int lds_root(int* lp, int x) {
  int p = lds_get(lp, x);
  while (p != x) {  // path splitting
    const int gp = lds_get(lp, p);
    if (gp != p) lds_put(lp, x, gp);
    x = p;
    p = gp;
  }
  return x;
}
__device__ __forceinline__ void lds_join(int* lp, int a, int b) {
  int ra = lds_root(lp, a), rb = lds_root(lp, b);
  while (ra != rb) {
    if (ra > rb) { const int s = ra; ra = rb; rb = s; }
    const int old = atomicCAS(&lp[rb], rb, ra);
    if (old == rb) return;
    rb = lds_root(lp, old);
  }
}

// With idx (hook mode 4), every entry also lowers the minimum of its three
// vertices to its local root: a vertex minimum only has to name some
// triangle of a set that touches the vertex, so the local root serves, and
// the vertex hook then joins every set that touches a common vertex (which
// covers the edges between tiles too).
template <int TILE, int NT, bool FANS>
__global__ __launch_bounds__(NT) void k_uf_local(const int32_t* __restrict__ nbr,
                                                 const int32_t* __restrict__ vlist,
                                                 int32_t* __restrict__ parent,
                                                 const int32_t* __restrict__ idx,
                                                 int32_t* __restrict__ vmin,
                                                 const FrameState* __restrict__ st,
                                                 const uint8_t* __restrict__ vis,
                                                 const int32_t* __restrict__ mesh_idx, int64_t T) {
  constexpr int kPer = TILE / NT;  // entries per thread: i = threadIdx.x + k NT
  __shared__ int lv[TILE];
  __shared__ int lp[TILE];
  const int nv = st->visible;
  const int64_t s0 = (int64_t)blockIdx.x * TILE;
  if (s0 >= nv) return;
  const int cnt = (int)min<int64_t>(TILE, nv - s0);
  // the loads of a thread's entries overlap
  int tk[kPer], nk[kPer][3];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    tk[k] = i < cnt ? vlist[s0 + i] : 0;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    nk[k][0] = nk[k][1] = nk[k][2] = -1;
    if (i < cnt) {
      const int3 x = reinterpret_cast<const int3*>(nbr)[tk[k]];
      nk[k][0] = x.x; nk[k][1] = x.y; nk[k][2] = x.z;
      if (FANS) {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          nk[k][e] = next_visible(mesh_idx, nbr, vis, tk[k], e, nk[k][e], T);
      }
      lv[i] = tk[k];
      lp[i] = i;
    }
  }
  __syncthreads();
  const int last = lv[cnt - 1];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT, t = tk[k];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int n = nk[k][e];
      if (n <= t || n > last) continue;
      // n, if visible, is one of the n - t entries after i: at the last of them
      // where everything in between is visible. A hidden neighbour is one that
      // is not found here; nothing else keeps it out.
      int lo = i + 1, hi = min(cnt - 1, i + (n - t));
      if (lv[hi] != n) {
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (lv[mid] < n) lo = mid + 1; else hi = mid;
        }
        if (lv[hi] != n) continue;
      }
      lds_join(lp, i, hi);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
    const int t = lv[i], r = lv[lds_root(lp, i)];
    astore(&parent[t], r);
    if (idx) {
#pragma unroll
      for (int e = 0; e < 3; ++e) atomicMin(&vmin[idx[3 * (int64_t)t + e]], r);
    }
  }
}

// Hook mode 5: the tile of TILE list entries is joined in LDS through shared
// vertices instead of shared edges (a shared edge is a shared vertex): every
// vertex reference is entered into an LDS hash table of (vertex << 32 |
// entry) words, where the first entry to claim a vertex owns it; every entry
// is joined with the owners of its vertices, and so all entries naming one
// vertex end in one set. This also merges the pieces of a chart that touch
// only at a vertex inside the tile. A vertex that finds no free slot is
// skipped (the global vertex pass merges through every vertex anyway). Then,
// as in mode 4, each entry's parent becomes its local root and its vertices'
// minima are lowered to it.
// Workgroups past the tiles fill the occupancy map with -1 (occ_fill, n4
// 16-byte words) while the tiles' dependent loads leave memory bandwidth free.
template <int TILE, int NT, int HS>
__device__ __forceinline__ void k_uf_local_vertex_body(const int32_t* __restrict__ idx,
                                                        const int32_t* __restrict__ vlist,
                                                        int32_t* __restrict__ parent,
                                                        int32_t* __restrict__ vmin,
                                                        const FrameState* __restrict__ st,
                                                        int4* __restrict__ occ_fill, int64_t n4) {
  static_assert((HS & (HS - 1)) == 0, "hash slots: a power of two");
  static_assert(TILE % NT == 0, "whole entries per thread");
  constexpr int kPer = TILE / NT;  // entries per thread: i = threadIdx.x + k NT
  constexpr unsigned long long kFree = ~0ull;
  __shared__ int lv[TILE];
  __shared__ int lp[TILE];
  __shared__ unsigned long long tab[HS];
  const int nv = st->visible;
  const int64_t s0 = (int64_t)blockIdx.x * TILE;
  if (s0 >= nv) {
    if (occ_fill) {
      const int64_t active = ((int64_t)nv + TILE - 1) / TILE;
      const int64_t nb = (int64_t)gridDim.x - active;
      const int4 neg = make_int4(-1, -1, -1, -1);
      for (int64_t i = ((int64_t)blockIdx.x - active) * NT + threadIdx.x; i < n4; i += nb * NT)
        occ_fill[i] = neg;
    }
    return;
  }
  const int cnt = (int)min<int64_t>(TILE, nv - s0);
  // every entry's triangle and vertices are loaded up front (the loads of
  // a thread's entries overlap) and kept in registers until the end
  int tk[kPer], vk[kPer][3];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    tk[k] = i < cnt ? vlist[s0 + i] : 0;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
#pragma unroll
    for (int e = 0; e < 3; ++e) vk[k][e] = 0;
    if (i < cnt) {
      const int3 v = reinterpret_cast<const int3*>(idx)[tk[k]];
      vk[k][0] = v.x; vk[k][1] = v.y; vk[k][2] = v.z;
      lv[i] = tk[k];
      lp[i] = i;
    }
  }
  for (int h = threadIdx.x; h < HS; h += NT) tab[h] = kFree;
  __syncthreads();
  // 1. every vertex reference enters the hash table; the first entry to
  //    claim a vertex's slot owns it
  int hs[kPer][3];  // slot of each reference, -1 when the table had no room
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      hs[k][e] = -1;
      if (i >= cnt) continue;
      const int v = vk[k][e];
      const unsigned long long mine = ((unsigned long long)(uint32_t)v << 32) | (uint32_t)i;
      uint32_t h = ((uint32_t)v * 2654435761u) & (HS - 1);
      for (int probe = 0; probe < 32; ++probe) {
        const unsigned long long old = atomicCAS(&tab[h], kFree, mine);
        if (old == kFree) {  // first entry with this vertex
          hs[k][e] = (int)h;
          break;
        }
        if ((uint32_t)(old >> 32) == (uint32_t)v) {  // another entry owns it
          hs[k][e] = (int)h;
          break;
        }
        h = (h + 1) & (HS - 1);
      }
    }
  }
  __syncthreads();
  // 2. each entry starts linked to the smallest of itself and the owners of
  //    its vertices (never above itself, so no cycles), then one step
  //    towards that node's own start
  int mo[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    mo[k] = i;
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (hs[k][e] >= 0) mo[k] = min(mo[k], (int)(uint32_t)tab[hs[k][e]]);
    if (i < cnt) lp[i] = mo[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    if (i >= cnt) continue;
    const int q = lds_get(lp, mo[k]);
    if (q != mo[k]) lds_put(lp, i, q);
  }
  __syncthreads();
  // 3. each entry joins the owners of its other vertices (none when both
  //    already hang from the same node)
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      if (hs[k][e] < 0) continue;
      const int o = (int)(uint32_t)tab[hs[k][e]];
      if (o == mo[k] || lds_get(lp, o) == lds_get(lp, i)) continue;
      lds_join(lp, i, o);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * NT;
    if (i >= cnt) continue;
    const int r = lv[lds_root(lp, i)];
    astore(&parent[tk[k]], r);
    // every reference to a vertex in the tile is in this set, so the owner's
    // reference alone lowers the vertex minimum (and each reference that
    // found no slot lowers its own)
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (hs[k][e] < 0 || (int)(uint32_t)tab[hs[k][e]] == i) atomicMin(&vmin[vk[k][e]], r);
  }
}
template <int TILE, int NT, int HS>
__global__ __launch_bounds__(NT) void k_uf_local_vertex(const int32_t* __restrict__ idx,
                                                        const int32_t* __restrict__ vlist,
                                                        int32_t* __restrict__ parent,
                                                        int32_t* __restrict__ vmin,
                                                        const FrameState* __restrict__ st,
                                                        int4* __restrict__ occ_fill, int64_t n4) {
  k_uf_local_vertex_body<TILE, NT, HS>(idx, vlist, parent, vmin, st, occ_fill, n4);
}

// Vertex minimum (Alg. 1, third loop): every visible triangle is compressed
// to its current root and every vertex records the smallest root among its
// visible triangles. The compression keeps the vertex hook's walks short.
__global__ void k_uf_vertex_min(const int32_t* __restrict__ idx,
                                const int32_t* __restrict__ vlist, int32_t* parent,
                                int32_t* __restrict__ vmin, const FrameState* __restrict__ st) {
  const int nv = st->visible;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    const int t = vlist[i];
    const int r = uf_root(parent, t);
    if (r != t) astore(&parent[t], r);
#pragma unroll
    for (int e = 0; e < 3; ++e) atomicMin(&vmin[idx[3 * (int64_t)t + e]], r);
  }
}

// Vertex hook: join every visible triangle with the recorded root of each of
// its vertices, merging charts that share only a vertex. parent[t] is an
// ancestor of t: a vertex whose minimum equals it needs no join, which skips
// most of them; along a tile border many lanes of a wave name the same
// (parent, minimum) pair, and only the lowest lane of each pair joins, once
// per workgroup (an LDS set of the pairs taken).
__device__ __forceinline__ void k_uf_vertex_hook_body(const int32_t* __restrict__ idx,
                                 const int32_t* __restrict__ vlist, int32_t* parent,
                                 const int32_t* __restrict__ vmin,
                                 const FrameState* __restrict__ st) {
  __shared__ unsigned long long pairs[kPairSlots];
  pairs_clear(pairs);
  const int nv = st->visible;
  const int lane = lane_id();
  for (int i0 = blockIdx.x * blockDim.x; i0 < nv; i0 += gridDim.x * blockDim.x) {
    const int i = i0 + threadIdx.x;
    const bool valid = i < nv;
    int pt = 0, m[3] = {0, 0, 0};
    if (valid) {
      const int t = vlist[i];
#pragma unroll
      for (int e = 0; e < 3; ++e) m[e] = aload(&vmin[idx[3 * (int64_t)t + e]]);
      pt = aload(&parent[t]);
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      bool want = valid && m[e] != pt && (e < 1 || m[e] != m[0]) && (e < 2 || m[e] != m[1]);
      const int a = min(pt, m[e]), b = max(pt, m[e]);
      unsigned long long todo = __ballot(want);
      bool keep = false;
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int la = __shfl(a, leader, kWave), lb = __shfl(b, leader, kWave);
        if (lane == leader) keep = true;
        todo &= ~__ballot(want && a == la && b == lb);
      }
      if (keep) join_once(pairs, parent, a, b);
    }
  }
}
__global__ __launch_bounds__(kHookThreads) void k_uf_vertex_hook(const int32_t* __restrict__ idx,
                                 const int32_t* __restrict__ vlist, int32_t* parent,
                                 const int32_t* __restrict__ vmin,
                                 const FrameState* __restrict__ st) {
  k_uf_vertex_hook_body(idx, vlist, parent, vmin, st);
}

// Flatten every visible triangle to its root and count roots per tile of
// kTriTile consecutive entries of the visible list. The walk here only reads:
// a path-halving store by one thread (parent[x] = a grandparent it read
// earlier) could land after another thread has set parent[x] to the root and
// leave x pointing at a non-root, which the later stages would read as the
// chart's root.
__device__ __forceinline__ void k_uf_flatten_count_body(const int32_t* __restrict__ vlist, int32_t* parent,
                                   uint32_t* __restrict__ tile_count,
                                   const FrameState* __restrict__ st) {
  __shared__ uint32_t sh[kBlock / kWave];
  const int nv = st->visible;
  const int64_t base = (int64_t)blockIdx.x * kTriTile + (int64_t)threadIdx.x * 4;
  if ((int64_t)blockIdx.x * kTriTile >= nv) return;
  // the four walks of a thread advance together, so that their dependent
  // loads are in flight at the same time (constant indices keep the arrays
  // in registers)
  int t[4], r[4], up[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) t[k] = base + k < nv ? vlist[base + k] : -1;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r[k] = t[k];
    up[k] = t[k] >= 0 ? aload(&parent[t[k]]) : t[k];
  }
  bool more = true;
  while (more) {
    more = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (up[k] != r[k]) {
        r[k] = up[k];
        up[k] = aload(&parent[r[k]]);
        more = true;
      }
    }
  }
  uint32_t roots = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (t[k] < 0) continue;
    if (r[k] != t[k]) astore(&parent[t[k]], r[k]);
    roots += (r[k] == t[k]);
  }
  roots = block_sum<uint32_t>(roots, sh);
  if (threadIdx.x == 0) tile_count[blockIdx.x] = roots;
}
__global__ void k_uf_flatten_count(const int32_t* __restrict__ vlist, int32_t* parent,
                                   uint32_t* __restrict__ tile_count,
                                   const FrameState* __restrict__ st) {
  k_uf_flatten_count_body(vlist, parent, tile_count, st);
}

// Chart index of each root = its rank among roots; the visible list ascends
// with the triangle index, so chart indices ascend with the chart's lowest
// triangle. Each workgroup sums the root counts of the tiles before its own;
// the last one records the chart count (above max_charts: FA_ERR_CAPACITY;
// no chart index at or past max_charts is written, and every later stage
// stops on the status). The status is not read here: the last workgroup may set
// it while others start, and a frame that ended before has an empty list.
__device__ __forceinline__ void k_assign_roots_body(const int32_t* __restrict__ vlist,
                               const int32_t* __restrict__ parent,
                               const uint32_t* __restrict__ tile_count, int32_t* __restrict__ cot,
                               fa_chart* __restrict__ charts, uint32_t* __restrict__ accum,
                               int32_t max_charts, FrameState* __restrict__ st) {
  __shared__ uint32_t sh[kBlock / kWave];
  const int nv = st->visible;
  if ((int64_t)blockIdx.x * kTriTile >= nv) return;
  const uint32_t off = tiles_before(tile_count, blockIdx.x, sh);
  const int64_t base = (int64_t)blockIdx.x * kTriTile + (int64_t)threadIdx.x * 4;
  bool root[4];
  int tv[4];
  uint32_t mine = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = base + k;
    tv[k] = i < nv ? vlist[i] : -1;
    root[k] = tv[k] >= 0 && aload(&parent[tv[k]]) == tv[k];
    mine += root[k];
  }
  uint32_t tot;
  uint32_t c = off + block_incl_scan<uint32_t>(mine, sh, &tot) - mine;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!root[k]) continue;
    if (c < (uint32_t)max_charts) {
      cot[tv[k]] = (int32_t)c;
      charts[c].root_tri = tv[k];
      reinterpret_cast<uint4*>(accum)[c] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u);
    }
    ++c;
  }
  if ((int64_t)(blockIdx.x + 1) * kTriTile >= nv && threadIdx.x == 0) {
    const uint32_t total = off + tot;
    st->num_charts = (int32_t)total;  // reported even when above the capacity
    if (total > (uint32_t)max_charts) st->status = FA_ERR_CAPACITY;
  }
}
__global__ void k_assign_roots(const int32_t* __restrict__ vlist,
                               const int32_t* __restrict__ parent,
                               const uint32_t* __restrict__ tile_count, int32_t* __restrict__ cot,
                               fa_chart* __restrict__ charts, uint32_t* __restrict__ accum,
                               int32_t max_charts, FrameState* __restrict__ st) {
  k_assign_roots_body(vlist, parent, tile_count, cot, charts, accum, max_charts, st);
}

// ---------------------------------------------------------------------------
// small meshes: everything before the boxes in one workgroup
// ---------------------------------------------------------------------------
// For meshes of up to kFrontTris triangles and kFrontVerts vertices one
// workgroup does what the prologue, the compaction, the union-find (through
// shared vertices) and the root assignment do in six launches, with the
// vertices' first triangles and the parents of the triangles in LDS, indexed
// directly. Six launches of little work each cost about 4 us of launch and
// drain. This one is bound by LDS latency, the walks of the joins above all.
// A whole frame with the six launches and with this one: 66 and 47 us at 2048
// triangles, 68 and 58 at 4096, 73 and 69 at 8192 (grids in row order; objects
// 66 and 54 at 2048, 75 and 76 at 8000) and 81 and 92 at 15842, so the line lies
// at 8192.
// Workgroups past the first fill the occupancy map.
constexpr int kFrontTris = 8192;
constexpr int kFrontVerts = 16384;
constexpr int kFrontThreads = 1024;
constexpr int kFrontMasks = kFrontTris / kWave;

inline bool use_front(const FrameParams& p, int64_t T, int64_t V) {
  return T > 0 && T <= kFrontTris && V <= kFrontVerts && !(p.flags & FA_FLAG_EDGE_ONLY_CHARTS);
}
inline size_t front_lds(int64_t T, int64_t V) { return 4 * (size_t)(T + V); }

// Exclusive prefix of the set bits of mask[0 .. n) into pre, the total into
// *total, by the first wave (n <= 4 waves).
__device__ __forceinline__ void mask_prefix(const unsigned long long* mask, int n, uint32_t* pre,
                                            uint32_t* total) {
  const int lane = lane_id();
  uint32_t c[4], sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = 4 * lane + k;
    c[k] = i < n ? (uint32_t)__popcll(mask[i]) : 0u;
    sum += c[k];
  }
  const uint32_t incl = wave_incl_scan_dpp(sum);
  uint32_t at = incl - sum;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = 4 * lane + k;
    if (i < n) pre[i] = at;
    at += c[k];
  }
  if (lane == kWave - 1) *total = incl;
}
static_assert(kFrontMasks <= 4 * kWave, "four masks per lane of one wave");
constexpr int kFrontFew = 2 * kFrontThreads;  // up to this many: two triangles a thread, else 8

template <int PER>
__device__ __forceinline__ void k_front_body(
    const uint8_t* __restrict__ vis, const int32_t* __restrict__ idx, int T, int V,
    int32_t* __restrict__ cov, int32_t* __restrict__ cot, int32_t* __restrict__ vlist,
    fa_chart* __restrict__ charts, uint32_t* __restrict__ accum, int32_t max_charts,
    FrameState* __restrict__ st, unsigned long long* __restrict__ big_counter, bool check,
    int4* __restrict__ occ_fill, int64_t n4) {
  extern __shared__ uint32_t dyn[];
  __shared__ unsigned long long vm[kFrontMasks], rm[kFrontMasks];
  __shared__ uint32_t vp[kFrontMasks], rp[kFrontMasks], total[2], bad_index;
  const int tid = threadIdx.x, lane = lane_id();
  if (blockIdx.x > 0) {
    const int4 neg = make_int4(-1, -1, -1, -1);
    const int64_t step = (int64_t)(gridDim.x - 1) * kFrontThreads;
    if (occ_fill)
      for (int64_t i = (int64_t)(blockIdx.x - 1) * kFrontThreads + tid; i < n4; i += step)
        occ_fill[i] = neg;
    return;
  }
  uint32_t* own = dyn;                           // [V] smallest visible triangle of a vertex
  int* lp = reinterpret_cast<int*>(dyn + V);     // [T] parents of the visible triangles
  constexpr uint32_t kNone = ~0u;
  bool on[PER];
  int vk[PER][3];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = k * kFrontThreads + tid;
    on[k] = t < T && vis[t];
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = k * kFrontThreads + tid;
#pragma unroll
    for (int e = 0; e < 3; ++e) vk[k][e] = t < T ? idx[3 * t + e] : 0;  // (beside vis)
  }
  if (tid == 0) {
    bad_index = 0u;
    *big_counter = 0ull;
  }
  for (int v = tid; v < V; v += kFrontThreads) own[v] = kNone;
  __syncthreads();
  if (check) {
    bool bad = false;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (k * kFrontThreads + tid < T) {
#pragma unroll
        for (int e = 0; e < 3; ++e) bad = bad || vk[k][e] < 0 || vk[k][e] >= V;
      }
    if (bad) bad_index = 1u;
    __syncthreads();
  }
  // a bad index ends the frame with an empty visible list
  const bool dead = check && bad_index != 0u;
  const int w = tid / kWave;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    on[k] = on[k] && !dead;
    const unsigned long long m = __ballot(on[k]);
    if (lane == 0) vm[k * (kFrontThreads / kWave) + w] = m;
    if (on[k]) {
#pragma unroll
      for (int e = 0; e < 3; ++e) atomicMin(&own[vk[k][e]], (uint32_t)(k * kFrontThreads + tid));
    }
  }
  __syncthreads();
  const int masks = PER * (kFrontThreads / kWave);
  if (w == 0) mask_prefix(vm, masks, vp, &total[0]);
  // each triangle starts linked to the smallest triangle at its vertices (vk
  // becomes the vertices' first triangles); then the links are halved until
  // none changes (a grid in row order starts with a link per row)
  int up[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    up[k] = 0;
    if (on[k]) {
#pragma unroll
      for (int e = 0; e < 3; ++e) vk[k][e] = (int)own[vk[k][e]];
      up[k] = min(vk[k][0], min(vk[k][1], vk[k][2]));
      lp[k * kFrontThreads + tid] = up[k];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = k * kFrontThreads + tid;
    if (on[k]) vlist[vp[t / kWave] + __popcll(vm[t / kWave] & lanes_below())] = t;
  }
  for (int round = 0; round < 16; ++round) {
    bool more = false;
    int q[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) q[k] = on[k] ? lds_get(lp, up[k]) : 0;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (on[k] && q[k] != up[k]) {
        up[k] = q[k];
        lds_put(lp, k * kFrontThreads + tid, q[k]);
        more = true;
      }
    if (!__syncthreads_or(more)) break;
  }
  // every triangle joins the first triangles of its vertices
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (!on[k]) continue;
    const int t = k * kFrontThreads + tid;
    int q[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) q[e] = lds_get(lp, vk[k][e]);
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (q[e] != up[k]) lds_join(lp, t, vk[k][e]);
  }
  __syncthreads();
  int r[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = k * kFrontThreads + tid;
    r[k] = on[k] ? lds_root(lp, t) : -1;
    const unsigned long long m = __ballot(r[k] == t);
    if (lane == 0) rm[k * (kFrontThreads / kWave) + w] = m;
  }
  __syncthreads();  // (every walk has ended: a walk's own stores may not follow these)
  if (w == 0) mask_prefix(rm, masks, rp, &total[1]);
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (on[k]) lp[k * kFrontThreads + tid] = r[k];
  __syncthreads();
  // chart = rank of the root among the roots
  const uint32_t charts_n = total[1];
  const bool over = charts_n > (uint32_t)max_charts;
  auto chart_of_root = [&](int root) {
    return (int)(rp[root / kWave] +
                 (uint32_t)__popcll(rm[root / kWave] & ((1ull << (root & (kWave - 1))) - 1ull)));
  };
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int t = k * kFrontThreads + tid;
    if (t >= T) continue;
    int c = on[k] ? chart_of_root(r[k]) : -1;
    const bool root = on[k] && r[k] == t;
    if (root && c < max_charts) {
      charts[c].root_tri = t;
      reinterpret_cast<uint4*>(accum)[c] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u);
    }
    if (over && !(root && c < max_charts)) c = -1;
    cot[t] = c;
  }
  for (int v = tid; v < V; v += kFrontThreads) {
    const uint32_t o = own[v];
    cov[v] = o == kNone || over ? -1 : chart_of_root(lp[o]);
  }
  static_assert(sizeof(FrameState) % 4 == 0 && FA_OK == 0, "the state clears word by word");
  constexpr unsigned kStatus = offsetof(FrameState, status) / 4,
                     kCharts = offsetof(FrameState, num_charts) / 4,
                     kVisible = offsetof(FrameState, visible) / 4;
  for (unsigned i = tid; i < sizeof(FrameState) / 4; i += kFrontThreads)
    reinterpret_cast<uint32_t*>(st)[i] =
        i == kStatus ? (uint32_t)(dead ? FA_ERR_INVALID_ARG : over ? FA_ERR_CAPACITY : FA_OK)
        : i == kCharts ? charts_n
        : i == kVisible ? total[0] : 0u;
}
template <int PER>
__global__ __launch_bounds__(kFrontThreads) void k_front(
    const uint8_t* __restrict__ vis, const int32_t* __restrict__ idx, int T, int V,
    int32_t* __restrict__ cov, int32_t* __restrict__ cot, int32_t* __restrict__ vlist,
    fa_chart* __restrict__ charts, uint32_t* __restrict__ accum, int32_t max_charts,
    FrameState* __restrict__ st, unsigned long long* __restrict__ big_counter, bool check,
    int4* __restrict__ occ_fill, int64_t n4) {
  k_front_body<PER>(vis, idx, T, V, cov, cot, vlist, charts, accum, max_charts, st, big_counter,
                    check, occ_fill, n4);
}

// ---------------------------------------------------------------------------
// per-triangle conservative box (NDC)
// ---------------------------------------------------------------------------
// plane distances: 0 left w+x, 1 right w-x, 2 bottom w+y, 3 top w-y,
//                  4 near w+z, 5 far w-z
template <int P>
__device__ __forceinline__ float pdist(const float4& q) {
  if (P == 0) return q.w + q.x;
  if (P == 1) return q.w - q.x;
  if (P == 2) return q.w + q.y;
  if (P == 3) return q.w - q.y;
  if (P == 4) return q.w + q.z;
  return q.w - q.z;
}

struct Quad {
  float4 v0, v1, v2, v3;
  int n;
};

// Append a vertex. Value selects on every slot (not a branch per slot, which
// the optimizer turns into a runtime-indexed store that moves the polygon to
// scratch memory).
__device__ __forceinline__ float4 pick(bool c, const float4& a, const float4& b) {
  return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}
__device__ __forceinline__ void quad_put(Quad& q, const float4& p) {
  const int n = q.n;
  q.v0 = pick(n == 0, p, q.v0);
  q.v1 = pick(n == 1, p, q.v1);
  q.v2 = pick(n == 2, p, q.v2);
  q.v3 = pick(n >= 3, p, q.v3);
  q.n = n + 1;
}

// One edge S->E of a Sutherland-Hodgman pass against plane P.
template <int P>
__device__ __forceinline__ void sh_edge(Quad& q, const float4& S, const float4& E) {
  const float dS = pdist<P>(S), dE = pdist<P>(E);
  const bool inS = dS >= 0.0f, inE = dE >= 0.0f;
  if (inS != inE) {
    const float4 A = inS ? S : E;
    const float4 B = inS ? E : S;
    const float dA = inS ? dS : dE;
    const float dB = inS ? dE : dS;
    const float t = dA / (dA - dB);
    float4 I;
    I.x = A.x + t * (B.x - A.x);
    I.y = A.y + t * (B.y - A.y);
    I.z = A.z + t * (B.z - A.z);
    I.w = A.w + t * (B.w - A.w);
    quad_put(q, I);
  }
  if (inE) quad_put(q, E);
}

template <int P>
__device__ __forceinline__ Quad clip_tri(const float4& a, const float4& b, const float4& c) {
  Quad q;
  q.n = 0;
  q.v0 = q.v1 = q.v2 = q.v3 = a;
  sh_edge<P>(q, a, b);
  sh_edge<P>(q, b, c);
  sh_edge<P>(q, c, a);
  return q;
}

__device__ __forceinline__ void blinn_vertex(const float4& p, float& nx, float& ny) {
  nx = fminf(fmaxf(p.x, -p.w), p.w) / p.w;
  ny = fminf(fmaxf(p.y, -p.w), p.w) / p.w;
}

// Blinn's coverage estimate of a polygon of 3 or 4 vertices.
__device__ __forceinline__ float4 blinn_box(const Quad& q) {
  bool bad = !(q.v0.w > 0.0f) || !(q.v1.w > 0.0f) || !(q.v2.w > 0.0f) ||
             (q.n == 4 && !(q.v3.w > 0.0f));
  if (bad) return make_float4(-1.0f, -1.0f, 1.0f, 1.0f);
  float x0, y0, x, y;
  blinn_vertex(q.v0, x0, y0);
  float4 b = make_float4(x0, y0, x0, y0);
  blinn_vertex(q.v1, x, y);
  b.x = fminf(b.x, x); b.y = fminf(b.y, y); b.z = fmaxf(b.z, x); b.w = fmaxf(b.w, y);
  blinn_vertex(q.v2, x, y);
  b.x = fminf(b.x, x); b.y = fminf(b.y, y); b.z = fmaxf(b.z, x); b.w = fmaxf(b.w, y);
  if (q.n == 4) {
    blinn_vertex(q.v3, x, y);
    b.x = fminf(b.x, x); b.y = fminf(b.y, y); b.z = fmaxf(b.z, x); b.w = fmaxf(b.w, y);
  }
  return b;
}

__device__ __forceinline__ float box_area(const float4& b) { return (b.z - b.x) * (b.w - b.y); }

template <int P>
__device__ __forceinline__ void try_plane(const float4& a, const float4& b, const float4& c,
                                          float4& best, float& best_area) {
  if (pdist<P>(a) < 0.0f || pdist<P>(b) < 0.0f || pdist<P>(c) < 0.0f) {
    float4 bp = blinn_box(clip_tri<P>(a, b, c));
    float ar = box_area(bp);
    if (ar < best_area) { best = bp; best_area = ar; }
  }
}

template <int P>
__device__ __forceinline__ bool all_out(const float4& a, const float4& b, const float4& c) {
  return pdist<P>(a) < 0.0f && pdist<P>(b) < 0.0f && pdist<P>(c) < 0.0f;
}

// Returns false when the triangle is entirely outside one plane of the view
// volume; otherwise the near-clipped or best-single-plane-clipped Blinn box.
__device__ __forceinline__ bool triangle_ndc_box(const float4& a, const float4& b,
                                                 const float4& c, bool side_clip, float4& box) {
  if (all_out<0>(a, b, c) || all_out<1>(a, b, c) || all_out<2>(a, b, c) ||
      all_out<3>(a, b, c) || all_out<4>(a, b, c) || all_out<5>(a, b, c))
    return false;
  if (pdist<4>(a) < 0.0f || pdist<4>(b) < 0.0f || pdist<4>(c) < 0.0f) {
    box = blinn_box(clip_tri<4>(a, b, c));
    return true;
  }
  Quad t;
  t.v0 = a; t.v1 = b; t.v2 = c; t.v3 = a; t.n = 3;
  float4 best = blinn_box(t);
  if (side_clip) {
    float ar = box_area(best);
    try_plane<0>(a, b, c, best, ar);
    try_plane<1>(a, b, c, best, ar);
    try_plane<2>(a, b, c, best, ar);
    try_plane<3>(a, b, c, best, ar);
    try_plane<5>(a, b, c, best, ar);
  }
  box = best;
  return true;
}

// Gather: chart of every visible triangle and its vertices (unless they are
// labelled already, by k_front), and the chart's box as the union of its
// triangles' boxes. Each thread handles kGatherItems
// entries of the visible list, issuing the dependent loads of all its entries
// level by level (list, root, chart and indices, clip vertices) so that their
// latencies overlap; the boxes are merged into a per-workgroup table of charts
// in LDS, and only the table is flushed with global atomics (large charts
// would otherwise serialize on their four accumulator words).
//
// Into the table, a chart that kGatherGroup or more lanes of a wave name is
// reduced in registers first (large charts: 64 lanes on one LDS word would
// serialize); lanes of smaller groups each do their own four LDS atomics. One
// reduction per distinct chart and a table of 64 slots, whose overflow went
// to global atomics, took 108 us for 142k visible triangles in 23.7k charts
// and 116 us for 165k in 2.5k edge-connected charts; now 10 and 24 us (one
// large terrain chart and 256 others: 14.5 -> 13.0 us).
constexpr int kGatherItems = 2;
// threads per gather workgroup: one LDS chart table per 1024 entries
// (256: 16.4 us, 512: 13.9 us, 1024: 16.4 us for one city frame)
constexpr int kGatherBlock = 512;
constexpr int kSlots = kGatherBlock * kGatherItems;  // as many charts as entries
constexpr int kSlotProbes = 32;
constexpr int kGatherGroup = 8;
static_assert((kSlots & (kSlots - 1)) == 0, "table slots: a power of two");
constexpr unsigned kFillBlocks = 1024;  // least workgroups that fill the occupancy map
constexpr unsigned kFillGroups = 256;   // the same for the 1024-thread union-find tiles
// Workgroups of 1024 threads that fill a map of n4 16-byte words beside one
// other: four stores a thread, at most kFillGroups.
inline unsigned fill_groups(int64_t n4) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n4 / 4096, kFillGroups));
}

__device__ __forceinline__ void k_gather_boxes_body(
    const int32_t* __restrict__ vlist, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ parent, const float* __restrict__ pos, int32_t* cot,
    int32_t* __restrict__ cov, uint32_t* __restrict__ accum, const FrameParams& p,
    const FrameState* __restrict__ st, int4* __restrict__ occ_fill, int64_t n4, bool labelled) {
  __shared__ int32_t skey[kSlots];
  __shared__ uint32_t sbox[4][kSlots];
  const int nv = st->visible;
  const int64_t per = kGatherBlock * kGatherItems;
  const int64_t active = (nv + per - 1) / per;
  if ((int64_t)blockIdx.x >= active) {
    // workgroups past the gather's own fill the occupancy map with -1
    if (occ_fill) {
      const int64_t nb = (int64_t)gridDim.x - active;
      const int4 neg = make_int4(-1, -1, -1, -1);
      for (int64_t i = ((int64_t)blockIdx.x - active) * kGatherBlock + threadIdx.x; i < n4;
           i += nb * kGatherBlock)
        occ_fill[i] = neg;
    }
    return;
  }
  if (st->status != FA_OK) return;
  for (int i = threadIdx.x; i < kSlots; i += blockDim.x) {
    skey[i] = -1;
    sbox[0][i] = sbox[1][i] = 0xFFFFFFFFu;
    sbox[2][i] = sbox[3][i] = 0u;
  }
  __syncthreads();
  for (int64_t blk = blockIdx.x; blk < active; blk += gridDim.x) {
    int tv[kGatherItems], cv[kGatherItems], vi[kGatherItems][3];
    float4 q[kGatherItems][3];
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k) {
      const int64_t i = blk * per + (int64_t)k * kGatherBlock + threadIdx.x;
      tv[k] = i < nv ? vlist[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k)
      cv[k] = tv[k] < 0 ? 0 : labelled ? tv[k] : aload(&parent[tv[k]]);
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k) {
      const int t = max(tv[k], 0);
      cv[k] = tv[k] >= 0 ? cot[cv[k]] : -1;
      vi[k][0] = vi[k][1] = vi[k][2] = 0;
      if (tv[k] >= 0) {
        const int3 v = reinterpret_cast<const int3*>(idx)[t];
        vi[k][0] = v.x; vi[k][1] = v.y; vi[k][2] = v.z;
      }
    }
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k)
#pragma unroll
      for (int e = 0; e < 3; ++e) q[k][e] = clip_of(pos, vi[k][e], p);
    // items are taken from slot 0 and shifted down after each one: constant
    // indices keep the arrays in registers (the clipping body is too large to
    // unroll, and a runtime index would move them to scratch memory)
    for (int k = 0; k < kGatherItems; ++k) {
      const bool valid = tv[0] >= 0;
      const int c = cv[0];
      bool has = false;
      float4 box = make_float4(0.f, 0.f, 0.f, 0.f);
      if (valid) {
        if (labelled) {
          // (chart_of_tri and chart_of_vert are written)
        } else if (p.flags & FA_FLAG_EDGE_ONLY_CHARTS) {
          cot[tv[0]] = c;
          // a vertex may touch several edge-connected charts: keep the smallest
          // (chart_of_vert starts at -1, the largest unsigned value)
#pragma unroll
          for (int e = 0; e < 3; ++e)
            atomicMin(reinterpret_cast<uint32_t*>(&cov[vi[0][e]]), (uint32_t)c);
        } else {
          cot[tv[0]] = c;
          cov[vi[0][0]] = c;
          cov[vi[0][1]] = c;
          cov[vi[0][2]] = c;
        }
        has = triangle_ndc_box(q[0][0], q[0][1], q[0][2], !(p.flags & FA_FLAG_NO_SIDE_CLIP), box);
      }
#pragma unroll
      for (int m = 0; m + 1 < kGatherItems; ++m) {
        tv[m] = tv[m + 1];
        cv[m] = cv[m + 1];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          vi[m][e] = vi[m + 1][e];
          q[m][e] = q[m + 1][e];
        }
      }
      uint32_t e0 = ord_of(box.x), e1 = ord_of(box.y), e2 = ord_of(box.z), e3 = ord_of(box.w);
      bool put = has;  // this lane enters its box (its own or its group's) into the table
      unsigned long long todo = __ballot(has);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int cl = __builtin_amdgcn_readlane(c, leader);
        const bool mine = has && c == cl;
        const unsigned long long grp = __ballot(mine);
        if (__popcll(grp) >= kGatherGroup) {
          const uint32_t a0 = wave_min_dpp(mine ? e0 : 0xFFFFFFFFu);
          const uint32_t a1 = wave_min_dpp(mine ? e1 : 0xFFFFFFFFu);
          const uint32_t a2 = ~wave_min_dpp(mine ? ~e2 : 0xFFFFFFFFu);
          const uint32_t a3 = ~wave_min_dpp(mine ? ~e3 : 0xFFFFFFFFu);
          if (mine) {
            e0 = a0; e1 = a1; e2 = a2; e3 = a3;
            put = lane_id() == leader;
          }
        }
        todo &= ~grp;
      }
      if (put) {
        int h = c & (kSlots - 1), slot = -1;
        for (int probe = 0; probe < kSlotProbes; ++probe) {
          const int prev = atomicCAS(&skey[h], -1, c);
          if (prev == -1 || prev == c) { slot = h; break; }
          h = (h + 1) & (kSlots - 1);
        }
        if (slot >= 0) {
          atomicMin(&sbox[0][slot], e0);
          atomicMin(&sbox[1][slot], e1);
          atomicMax(&sbox[2][slot], e2);
          atomicMax(&sbox[3][slot], e3);
        } else {
          atomicMin(&accum[4 * c + 0], e0);
          atomicMin(&accum[4 * c + 1], e1);
          atomicMax(&accum[4 * c + 2], e2);
          atomicMax(&accum[4 * c + 3], e3);
        }
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSlots; i += blockDim.x) {
    const int cl = skey[i];
    if (cl < 0) continue;
    atomicMin(&accum[4 * cl + 0], sbox[0][i]);
    atomicMin(&accum[4 * cl + 1], sbox[1][i]);
    atomicMax(&accum[4 * cl + 2], sbox[2][i]);
    atomicMax(&accum[4 * cl + 3], sbox[3][i]);
  }
}
__global__ __launch_bounds__(kGatherBlock) void k_gather_boxes(
    const int32_t* __restrict__ vlist, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ parent, const float* __restrict__ pos, int32_t* cot,
    int32_t* __restrict__ cov, uint32_t* __restrict__ accum, FrameParams p,
    const FrameState* __restrict__ st, int4* __restrict__ occ_fill, int64_t n4, bool labelled) {
  k_gather_boxes_body(vlist, idx, parent, pos, cot, cov, accum, p, st, occ_fill, n4, labelled);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// ---- batched wrappers (view = blockIdx.y) --------------------------------
__global__ void k_prologue_b(const BatchView* __restrict__ bv, int64_t V, const int32_t* __restrict__ nbr, int64_t T,
                             unsigned vblocks) {
  const BatchView& v = bv[blockIdx.y];
  k_prologue_body<0>(V, in_global(v.w.vmin), in_global(v.cov), in_global(v.visible), nbr, T, in_global(v.w.parent), in_global(v.cot),
                  in_global(v.w.tile_vis), vblocks, in_global(v.w.state), in_global(v.w.big_counter));
}
__global__ __launch_bounds__(1024) void k_tile_scan_b(const BatchView* __restrict__ bv,
                                                      unsigned tiles) {
  k_tile_scan_body(in_global(bv[blockIdx.y].w.tile_vis), tiles);
}
__global__ void k_vis_compact_b(const BatchView* __restrict__ bv, int64_t T) {
  const BatchView& v = bv[blockIdx.y];
  k_vis_compact_body(in_global(v.visible), T, in_global(v.w.tile_vis), in_global(v.w.vlist), in_global(v.w.state), true);
}
__global__ __launch_bounds__(1024) void k_uf_local_vertex_b(const BatchView* __restrict__ bv,
                                                            const int32_t* __restrict__ idx) {
  const BatchView& v = bv[blockIdx.y];
  k_uf_local_vertex_body<2048, 1024, 4096>(idx, in_global(v.w.vlist), in_global(v.w.parent), in_global(v.w.vmin), in_global(v.w.state),
                                           reinterpret_cast<int4*>(in_global(v.occ)),
                                           (int64_t)v.p.omega * v.p.omega / 4);
}
__global__ __launch_bounds__(kHookThreads) void k_uf_vertex_hook_b(const BatchView* __restrict__ bv,
                                   const int32_t* __restrict__ idx) {
  const BatchView& v = bv[blockIdx.y];
  k_uf_vertex_hook_body(idx, in_global(v.w.vlist), in_global(v.w.parent), in_global(v.w.vmin), in_global(v.w.state));
}
__global__ void k_uf_flatten_count_b(const BatchView* __restrict__ bv) {
  const BatchView& v = bv[blockIdx.y];
  k_uf_flatten_count_body(in_global(v.w.vlist), in_global(v.w.parent), in_global(v.w.tile_count), in_global(v.w.state));
}
__global__ void k_assign_roots_b(const BatchView* __restrict__ bv) {
  const BatchView& v = bv[blockIdx.y];
  k_assign_roots_body(in_global(v.w.vlist), in_global(v.w.parent), in_global(v.w.tile_count), in_global(v.cot), in_global(v.charts), in_global(v.w.accum),
                      v.p.max_charts, in_global(v.w.state));
}
__global__ __launch_bounds__(kGatherBlock) void k_gather_boxes_b(const BatchView* __restrict__ bv,
                                                           const int32_t* __restrict__ idx,
                                                           bool labelled) {
  const BatchView& v = bv[blockIdx.y];
  k_gather_boxes_body(in_global(v.w.vlist), idx, in_global(v.w.parent), in_global(v.w.pos), in_global(v.cot), in_global(v.cov), in_global(v.w.accum), v.p,
                      in_global(v.w.state), nullptr, 0, labelled);
}
template <int PER>
__global__ __launch_bounds__(kFrontThreads) void k_front_b(const BatchView* __restrict__ bv,
                                                           const int32_t* __restrict__ idx, int T,
                                                           int V) {
  const BatchView& v = bv[blockIdx.y];
  k_front_body<PER>(in_global(v.visible), idx, T, V, in_global(v.cov), in_global(v.cot), in_global(v.w.vlist), in_global(v.charts), in_global(v.w.accum),
                    v.p.max_charts, in_global(v.w.state), in_global(v.w.big_counter), false,
                    reinterpret_cast<int4*>(in_global(v.occ)), (int64_t)v.p.omega * v.p.omega / 4);
}

}  // namespace

unsigned view_groups(int64_t T, int64_t items, int threads, int n) {
  const int64_t most = std::max<int64_t>(kViewThreads / ((int64_t)threads * n), 16);
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((T + items - 1) / items, most));
}

unsigned visible_grid(int64_t T) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((T + kBlock - 1) / kBlock, 2048));
}

hipError_t launch_prologue(int64_t V, const uint8_t* vis, const int32_t* nbr,
                           int64_t T, const FrameParams& p, const Work& w, int32_t* cov,
                           int32_t* cot, int uf_init, const int32_t* check_idx, Marker& mk,
                           hipStream_t st) {
  const unsigned vb = std::max(1u, grid_for(V, kBlock * kProVerts));
  const unsigned tt = grid_for(T, kTriTile * kTilesPer);
  // (neighbours are known of checked meshes only)
  if (uf_init == 2 && check_idx) return hipErrorInvalidValue;
  auto prologue = [&](auto kernel, unsigned tile_groups) {
    kernel<<<vb + tile_groups, kBlock, 0, st>>>(V, w.vmin, cov, vis, nbr, T, w.parent, cot, w.tile_vis, vb,
                                       w.state, w.big_counter, check_idx);
  };
  if (uf_init == 2) prologue(k_prologue<2>, grid_for(T, kTriTile));
  else if (uf_init == 1) prologue(k_prologue<1>, tt);
  else prologue(k_prologue<0>, tt);
  mk(st);
  mk(st);  // (the visible-count scan is part of the compaction)
  if (T > 0)
    k_vis_compact<<<tt, kBlock, 0, st>>>(vis, T, w.tile_vis, w.vlist, w.state,
                                         check_idx != nullptr);
  mk(st);
  return hipGetLastError();
}

hipError_t front_kernel_attributes() {
  const void* ks[4] = {(const void*)k_front<2>, (const void*)k_front<8>,
                       (const void*)k_front_b<2>, (const void*)k_front_b<8>};
  for (const void* k : ks) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)front_lds(kFrontTris, kFrontVerts));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool launch_front(const uint8_t* vis, const int32_t* idx, int64_t T, int64_t V,
                  const FrameParams& p, const Work& w, int32_t* cot, int32_t* cov,
                  fa_chart* charts, int32_t* occ_fill, bool check, Marker& mk, hipStream_t st,
                  hipError_t* err) {
  if (!use_front(p, T, V)) return false;
  const int64_t n4 = (int64_t)p.omega * p.omega / 4;
  const unsigned grid = 1u + (occ_fill ? fill_groups(n4) : 0u);
  auto launch = [&](auto kernel) {
    kernel<<<grid, kFrontThreads, front_lds(T, V), st>>>(
        vis, idx, (int)T, (int)V, cov, cot, w.vlist, charts, w.accum, p.max_charts, w.state,
        w.big_counter, check, reinterpret_cast<int4*>(occ_fill), n4);
  };
  if (T <= kFrontFew) launch(k_front<2>);
  else launch(k_front<8>);
  for (int k = 0; k < 9; ++k) mk(st);  // (prologue to root assignment in one)
  k_gather_boxes<<<grid_for(T, kGatherBlock * kGatherItems), kGatherBlock, 0, st>>>(
      w.vlist, idx, w.parent, w.pos, cot, cov, w.accum, p, w.state, nullptr, 0, true);
  mk(st);
  *err = hipGetLastError();
  return true;
}

hipError_t launch_charts(const uint8_t* vis, const int32_t* idx, const int32_t* nbr, int64_t T,
                         const FrameParams& p, const Work& w, int32_t* cot, int32_t* cov,
                         fa_chart* charts, int32_t* occ_fill, Marker& mk, hipStream_t st) {
  const unsigned g = visible_grid(T);
  const unsigned vt = std::max(1u, grid_for(T, kTriTile));
  const int64_t n4 = (int64_t)p.omega * p.omega / 4;
  bool fill_done = false;
  if (T > 0 && (p.flags & FA_FLAG_EDGE_ONLY_CHARTS)) {
    // edge-connected charts: shared edges only, no vertex passes
    const int tile = p.uf_tile;
    auto join = [&](auto fans) {
      constexpr bool F = decltype(fans)::value;
      if (p.edge_hooks == 1) {
        k_uf_hook<F><<<g, kBlock, 0, st>>>(vis, nbr, w.vlist, w.parent, 0, w.state, idx, T);
        return;
      }
      if (tile == 8192)
        k_uf_local<8192, 1024, F><<<std::max(1u, grid_for(T, 8192)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, nullptr, w.vmin, w.state, vis, idx, T);
      else if (tile == 4096)
        k_uf_local<4096, 1024, F><<<std::max(1u, grid_for(T, 4096)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, nullptr, w.vmin, w.state, vis, idx, T);
      else
        k_uf_local<2048, 1024, F><<<std::max(1u, grid_for(T, 2048)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, nullptr, w.vmin, w.state, vis, idx, T);
      k_uf_cross<F><<<std::max(1u, g * kBlock / kHookThreads), kHookThreads, 0, st>>>(
          vis, nbr, w.vlist, w.parent, tile, w.state, idx, T);
    };
    if (p.edge_fans) join(std::true_type{});
    else join(std::false_type{});
    mk(st);
    mk(st);
    mk(st);
    k_uf_flatten_count<<<vt, kBlock, 0, st>>>(w.vlist, w.parent, w.tile_count, w.state);
  } else if (T > 0) {
    if (p.edge_hooks == 1) {
      k_uf_hook<false><<<g, kBlock, 0, st>>>(vis, nbr, w.vlist, w.parent, 0, w.state, idx, T);
    } else if (p.edge_hooks == 5) {
      // tiles of 2048 entries and a 4096-slot table (at most ~3/4 full); at
      // least kFillGroups workgroups past the largest visible list fill the
      // occupancy map
      k_uf_local_vertex<2048, 1024, 4096>
          <<<std::max(1u, grid_for(T, 2048)) + (occ_fill ? kFillGroups : 0u), 1024, 0, st>>>(
              idx, w.vlist, w.parent, w.vmin, w.state, reinterpret_cast<int4*>(occ_fill), n4);
      fill_done = true;
    } else if (p.edge_hooks >= 2) {
      const int tile = p.uf_tile;
      const int32_t* vidx = p.edge_hooks == 4 ? idx : nullptr;
      if (tile == 8192)
        k_uf_local<8192, 1024, false><<<std::max(1u, grid_for(T, 8192)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, vidx, w.vmin, w.state, vis, idx, T);
      else if (tile == 4096)
        k_uf_local<4096, 1024, false><<<std::max(1u, grid_for(T, 4096)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, vidx, w.vmin, w.state, vis, idx, T);
      else
        k_uf_local<2048, 1024, false><<<std::max(1u, grid_for(T, 2048)), 1024, 0, st>>>(
            nbr, w.vlist, w.parent, vidx, w.vmin, w.state, vis, idx, T);
      if (p.edge_hooks == 2)
        k_uf_cross<false><<<std::max(1u, g * kBlock / kHookThreads), kHookThreads, 0, st>>>(
            vis, nbr, w.vlist, w.parent, tile, w.state, idx, T);
    }
    mk(st);
    if (p.edge_hooks < 4)  // modes 4, 5: the tile kernel lowered the vertex minima
      k_uf_vertex_min<<<g, kBlock, 0, st>>>(idx, w.vlist, w.parent, w.vmin, w.state);
    mk(st);
    k_uf_vertex_hook<<<std::max(1u, g * kBlock / kHookThreads), kHookThreads, 0, st>>>(
        idx, w.vlist, w.parent, w.vmin, w.state);
    mk(st);
    k_uf_flatten_count<<<vt, kBlock, 0, st>>>(w.vlist, w.parent, w.tile_count, w.state);
  } else {
    mk(st);
    mk(st);
    mk(st);
  }
  mk(st);
  mk(st);  // (the root-count scan is part of the root assignment)
  if (T > 0) {
    k_assign_roots<<<vt, kBlock, 0, st>>>(w.vlist, w.parent, w.tile_count, cot, charts, w.accum,
                                          p.max_charts, w.state);
    mk(st);
    // the fill, unless the union-find tile kernel did it: at least kFillBlocks
    // workgroups beyond the largest visible list
    int32_t* gfill = fill_done ? nullptr : occ_fill;
    const unsigned fill_blocks = gfill ? kFillBlocks : 0u;
    k_gather_boxes<<<grid_for(T, kGatherBlock * kGatherItems) + fill_blocks, kGatherBlock, 0,
                     st>>>(
        w.vlist, idx, w.parent, w.pos, cot, cov, w.accum, p, w.state,
        reinterpret_cast<int4*>(gfill), n4, false);
  } else {
    mk(st);
  }
  mk(st);
  return hipGetLastError();
}

hipError_t launch_charts_batched(const BatchView* dev, int n, const int32_t* idx,
                                 const int32_t* nbr, int64_t T, int64_t V, int max_omega,
                                 hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (T > 0 && T <= kFrontTris && V <= kFrontVerts) {  // (batched views have vertex charts)
    const dim3 grid(1u + fill_groups((int64_t)max_omega * max_omega / 4), n);
    if (T <= kFrontFew)
      k_front_b<2><<<grid, kFrontThreads, front_lds(T, V), st>>>(dev, idx, (int)T, (int)V);
    else
      k_front_b<8><<<grid, kFrontThreads, front_lds(T, V), st>>>(dev, idx, (int)T, (int)V);
    k_gather_boxes_b<<<dim3(grid_for(T, kGatherBlock * kGatherItems), n), kGatherBlock, 0, st>>>(
        dev, idx, true);
    return hipGetLastError();
  }
  const unsigned vb = std::max(1u, grid_for(V, kBlock * kProVerts));
  const unsigned tt = grid_for(T, kTriTile * kTilesPer);
  const unsigned vt = std::max(1u, grid_for(T, kTriTile));
  k_prologue_b<<<dim3(vb + tt, n), kBlock, 0, st>>>(dev, V, nbr, T, vb);
  if (T > 0) {
    k_tile_scan_b<<<dim3(1, n), 1024, 0, st>>>(dev, vt);
    k_vis_compact_b<<<dim3(tt, n), kBlock, 0, st>>>(dev, T);
    k_uf_local_vertex_b<<<dim3(std::max(1u, grid_for(T, 2048)) + kFillGroups, n), 1024, 0, st>>>(
        dev, idx);
    k_uf_vertex_hook_b<<<dim3(view_groups(T, kHookThreads, kHookThreads, n), n), kHookThreads, 0,
                         st>>>(dev, idx);
    k_uf_flatten_count_b<<<dim3(vt, n), kBlock, 0, st>>>(dev);
    k_assign_roots_b<<<dim3(vt, n), kBlock, 0, st>>>(dev);
    k_gather_boxes_b<<<dim3(view_groups(T, kGatherBlock * kGatherItems, kGatherBlock, n), n),
                       kGatherBlock, 0, st>>>(dev, idx, false);
  }
  return hipGetLastError();
}

}  // namespace fa
