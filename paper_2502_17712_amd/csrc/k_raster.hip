// Atlas-space stages on gfx950:
//   UV emission (Appendix "Shading and Rasterization": every chart is scaled
//   by the chosen uniform scale, then moved rigidly from its NDC box to its
//   atlas box) and the atlas occupancy map (which chart owns each texel).
//
// Occupancy of texel (tx, ty) is chart c iff its centre lies in c's placed
// box (exact integer test in layout space, gutter included) and inside one of
// c's visible triangles mapped to the atlas (near-clipped when the triangle
// crosses the near plane), snapped to 1/256 texel with round-to-nearest-even,
// fan-triangulated from the first vertex, edges inclusive. Small footprints
// are rasterized by one lane, medium ones by their wave, large ones are queued
// and cut into 16x16 tiles shared by all waves.
#include <algorithm>
#include <climits>

#include "fa_internal.h"

namespace fa {
namespace {

struct ChartXform {
  float x0, y1, tw, halfW, halfH, rate, s, q, ox, oy;
  int rot;
};

__device__ __forceinline__ ChartXform chart_xform(const fa_chart& ch, const FrameParams& p,
                                                  const FrameState& st) {
  ChartXform m;
  m.x0 = ch.ndc_box[0];
  m.y1 = ch.ndc_box[3];
  m.tw = ch.target_w;
  m.halfW = 0.5f * (float)p.W;
  m.halfH = 0.5f * (float)p.H;
  m.rate = p.rate;
  m.s = st.s_star;
  m.q = (float)p.omega / (float)st.layout_w;  // omega/L (the atlas side being drawn)
  m.ox = (float)(ch.x + p.gutter);
  m.oy = (float)(ch.y + p.gutter);
  m.rot = ch.rotated;
  return m;
}

// clip-space point (w > 0) -> atlas texel coordinates
__device__ __forceinline__ float2 to_atlas(const ChartXform& m, float X, float Y, float w) {
  const float nx = X / w, ny = Y / w;
  const float px = ((nx - m.x0) * m.halfW) * m.rate;
  const float py = ((m.y1 - ny) * m.halfH) * m.rate;
  const float lx = m.rot ? py : px;
  const float ly = m.rot ? (m.tw - px) : py;
  return make_float2((m.ox + lx * m.s) * m.q, (m.oy + ly * m.s) * m.q);
}

// Per-vertex UVs of workgroup ub of a UV grid (k_uv, or the workgroups past
// the small-footprint raster's own, which need the same placement and run
// beside the raster instead of after it): each thread takes PER vertices a
// workgroup apart, so every load and store of a wave is one contiguous run,
// and issues their chart loads before any dependent load.
template <int PER>
__device__ __forceinline__ void uv_block(unsigned ub, const FrameParams& p,
                                         const float* __restrict__ pos,
                                         const int32_t* __restrict__ cov,
                                         const fa_chart* __restrict__ charts,
                                         float2* __restrict__ uv, int64_t V,
                                         const FrameState* __restrict__ stp) {
  const FrameState st = *stp;
  const int64_t v0 = (int64_t)ub * (blockDim.x * PER) + threadIdx.x;
  int c[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t v = v0 + (int64_t)k * blockDim.x;
    c[k] = (v < V && st.status == FA_OK) ? cov[v] : -1;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t v = v0 + (int64_t)k * blockDim.x;
    float2 r = make_float2(__builtin_nanf(""), __builtin_nanf(""));
    if (c[k] >= 0) {  // a vertex without a chart needs no position
      const float4 q = clip_of(pos, v, p);
      if (q.w > 0.0f) r = to_atlas(chart_xform(charts[c[k]], p, st), q.x, q.y, q.w);
    }
    if (v < V) uv[v] = r;
  }
}

// Vertices per UV thread: 4 for one frame; 8 in batched launches, whose
// grids hold every view's UV workgroups (fewer, longer waves launch faster
// there, and cost one frame about 0.2 us).
constexpr int kUvPerFrame = 4, kUvPerBatch = 8;

__global__ void k_uv(int64_t V, FrameParams p, const float* __restrict__ pos,
                     const int32_t* __restrict__ cov, const fa_chart* __restrict__ charts,
                     float2* __restrict__ uv, const FrameState* __restrict__ stp) {
  uv_block<kUvPerFrame>(blockIdx.x, p, pos, cov, charts, uv, V, stp);
}

// Per-corner UVs of edge-connected charts: corner k of triangle t is its
// vertex mapped through the chart of t (a vertex on a seam between charts
// gets one UV per chart). One thread per triangle writes its 24 bytes.
__global__ void k_uv_corners(int64_t T, FrameParams p, const int32_t* __restrict__ idx,
                             const float* __restrict__ pos, const int32_t* __restrict__ cot,
                             const fa_chart* __restrict__ charts, float2* __restrict__ uv,
                             const FrameState* __restrict__ stp) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const FrameState st = *stp;
  const int c = st.status == FA_OK ? cot[t] : -1;
  const float nan = __builtin_nanf("");
  if (c < 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) uv[3 * t + k] = make_float2(nan, nan);
    return;
  }
  const ChartXform m = chart_xform(charts[c], p, st);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float4 q = clip_of(pos, idx[3 * t + k], p);
    uv[3 * t + k] = q.w > 0.0f ? to_atlas(m, q.x, q.y, q.w) : make_float2(nan, nan);
  }
}

// ---------------------------------------------------------------------------
// occupancy
// ---------------------------------------------------------------------------
struct Footprint {
  int32_t ax, ay;          // vertex a (1/256 texel)
  int32_t bx, by, cx, cy;  // vertices b and c relative to a
  int tx0, tx1, ty0, ty1;  // inclusive texel range to test (non-empty)
  int chart;
  int neg;                 // signed area < 0
};

template <int P>
__device__ __forceinline__ float pd(const float4& q) {
  if (P == 0) return q.w + q.x;
  if (P == 1) return q.w - q.x;
  if (P == 2) return q.w + q.y;
  if (P == 3) return q.w - q.y;
  if (P == 4) return q.w + q.z;
  return q.w - q.z;
}
template <int P>
__device__ __forceinline__ bool outside(const float4& a, const float4& b, const float4& c) {
  return pd<P>(a) < 0.0f && pd<P>(b) < 0.0f && pd<P>(c) < 0.0f;
}

__device__ __forceinline__ float4 pick4(bool c, const float4& a, const float4& b) {
  return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}

// near-plane Sutherland-Hodgman of one triangle into up to 4 vertices; each
// output slot is written with value selects (a runtime index into `o` would
// move the polygon to scratch memory)
__device__ __forceinline__ int near_clip(const float4& a, const float4& b, const float4& c,
                                         float4* o) {
  int n = 0;
  float4 o0 = a, o1 = a, o2 = a, o3 = a;
  auto put = [&](const float4& v) {
    o0 = pick4(n == 0, v, o0);
    o1 = pick4(n == 1, v, o1);
    o2 = pick4(n == 2, v, o2);
    o3 = pick4(n >= 3, v, o3);
    ++n;
  };
  const float4 in[3] = {a, b, c};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float4 S = in[i], E = in[i == 2 ? 0 : i + 1];
    const float dS = pd<4>(S), dE = pd<4>(E);
    const bool iS = dS >= 0.0f, iE = dE >= 0.0f;
    if (iS != iE) {
      const float4 A = iS ? S : E, B = iS ? E : S;
      const float dA = iS ? dS : dE, dB = iS ? dE : dS;
      const float t = dA / (dA - dB);
      float4 I;
      I.x = A.x + t * (B.x - A.x);
      I.y = A.y + t * (B.y - A.y);
      I.z = A.z + t * (B.z - A.z);
      I.w = A.w + t * (B.w - A.w);
      put(I);
    }
    if (iE) put(E);
  }
  o[0] = o0;
  o[1] = o1;
  o[2] = o2;
  o[3] = o3;
  return n;
}

__device__ __forceinline__ int32_t snap(float u) {
  const float lim = 268435456.0f;  // 2^28 (1/256-texel units)
  return (int32_t)__builtin_rintf(fminf(fmaxf(u * 256.0f, -lim), lim));
}

// The near-clipped polygon of visible triangle t mapped to snapped atlas
// coordinates (1/256 texel, |value| <= 2^28); n = 0 when it claims nothing.
struct SnapPoly {
  int32_t u[4], v[4];
  int n;
  int chart;
};

__device__ __forceinline__ void snap_polygon(int64_t t, const int32_t* __restrict__ idx,
                                             const float* __restrict__ pos,
                                             const int32_t* __restrict__ cot,
                                             const fa_chart* __restrict__ charts,
                                             const FrameParams& p, const FrameState& st,
                                             SnapPoly& sp) {
  sp.n = 0;
  const int c = cot[t];
  sp.chart = c;
  if (c < 0) return;
  const float4 a = clip_of(pos, idx[3 * t], p), b = clip_of(pos, idx[3 * t + 1], p),
               cc = clip_of(pos, idx[3 * t + 2], p);
  if (outside<0>(a, b, cc) || outside<1>(a, b, cc) || outside<2>(a, b, cc) ||
      outside<3>(a, b, cc) || outside<4>(a, b, cc) || outside<5>(a, b, cc))
    return;
  float4 poly[4];
  int n;
  if (pd<4>(a) < 0.0f || pd<4>(b) < 0.0f || pd<4>(cc) < 0.0f) {
    n = near_clip(a, b, cc, poly);
  } else {
    poly[0] = a; poly[1] = b; poly[2] = cc; poly[3] = cc; n = 3;
  }
  // constant indices only (a runtime index would place the polygon in memory)
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (k < n && !(poly[k].w > 0.0f)) return;
  const ChartXform m = chart_xform(charts[c], p, st);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < n) {
      const float2 q = to_atlas(m, poly[k].x, poly[k].y, poly[k].w);
      sp.u[k] = snap(q.x);
      sp.v[k] = snap(q.y);
    }
  }
  sp.n = n;
}

// Fan triangle f (0 or 1) of a snapped polygon: vertices 0, f+1, f+2, with
// its texel range: texel centres (256 t + 128) inside the bounding box of the
// snapped triangle and inside the chart's placed box (`box` = lo_x, hi_x,
// lo_y, hi_y, the exact integer membership range of the box).
__device__ __forceinline__ bool fan_footprint(const SnapPoly& sp, int f, const int4 box, int omega,
                                              Footprint& fp) {
  if (f + 2 >= sp.n) return false;
  const int32_t ax = sp.u[0], ay = sp.v[0];
  // constant indices only (a runtime index would put the polygon in scratch)
  const bool f1 = f != 0;
  const int32_t ub = f1 ? sp.u[2] : sp.u[1], vb = f1 ? sp.v[2] : sp.v[1];
  const int32_t uc = f1 ? sp.u[3] : sp.u[2], vc = f1 ? sp.v[3] : sp.v[2];
  fp.ax = ax; fp.ay = ay;
  fp.bx = ub - ax; fp.by = vb - ay;
  fp.cx = uc - ax; fp.cy = vc - ay;
  const int64_t area = (int64_t)fp.bx * fp.cy - (int64_t)fp.by * fp.cx;
  if (area == 0) return false;
  fp.neg = area < 0;
  const int32_t umin = min(ax, min(ub, uc)), umax = max(ax, max(ub, uc));
  const int32_t vmin = min(ay, min(vb, vc)), vmax = max(ay, max(vb, vc));
  // ceil((x - 128) / 256) and floor((x - 128) / 256) as arithmetic shifts
  const int lo_x = max(box.x, max(0, (umin + 127) >> 8));
  const int hi_x = min(box.y, min(omega - 1, (umax - 128) >> 8));
  const int lo_y = max(box.z, max(0, (vmin + 127) >> 8));
  const int hi_y = min(box.w, min(omega - 1, (vmax - 128) >> 8));
  if (lo_x > hi_x || lo_y > hi_y) return false;
  fp.tx0 = lo_x; fp.tx1 = hi_x; fp.ty0 = lo_y; fp.ty1 = hi_y;
  fp.chart = sp.chart;
  return true;
}

// A queued footprint travels whole (three 16-byte words), so the tile kernel
// needs no dependent loads to rebuild it.
__device__ __forceinline__ void put_footprint(int4* d, const Footprint& f) {
  d[0] = make_int4(f.ax, f.ay, f.bx, f.by);
  d[1] = make_int4(f.cx, f.cy, f.tx0, f.tx1);
  d[2] = make_int4(f.ty0, f.ty1, f.chart, f.neg);
}
__device__ __forceinline__ Footprint get_footprint(const int4* d) {
  const int4 a = d[0], b = d[1], c = d[2];
  Footprint f;
  f.ax = a.x; f.ay = a.y; f.bx = a.z; f.by = a.w;
  f.cx = b.x; f.cy = b.y; f.tx0 = b.z; f.tx1 = b.w;
  f.ty0 = c.x; f.ty1 = c.y; f.chart = c.z; f.neg = c.w;
  return f;
}

// The three edge functions at the centre of texel (tx, ty), exact in 64-bit
// integers (inputs within 2^31, products within 2^61), negated when the
// triangle is clockwise so that "covered" is always "all three >= 0":
//   e0 = (b-a) x (p-a), e1 = (c-b) x (p-b), e2 = (a-c) x (p-c).
struct Edges {
  int64_t e0, e1, e2;
};
__device__ __forceinline__ Edges edges_at(const Footprint& fp, int tx, int ty) {
  const int32_t px = 256 * tx + 128 - fp.ax, py = 256 * ty + 128 - fp.ay;
  Edges e;
  e.e0 = (int64_t)fp.bx * py - (int64_t)fp.by * px;
  e.e1 = (int64_t)(fp.cx - fp.bx) * (py - fp.by) - (int64_t)(fp.cy - fp.by) * (px - fp.bx);
  e.e2 = (int64_t)fp.cy * px - (int64_t)fp.cx * py;
  if (fp.neg) { e.e0 = -e.e0; e.e1 = -e.e1; e.e2 = -e.e2; }
  return e;
}
// change of the edge functions per texel step in x and in y
__device__ __forceinline__ Edges step_x(const Footprint& fp) {
  const int64_t s = fp.neg ? -256 : 256;
  return Edges{-s * fp.by, -s * (fp.cy - fp.by), s * fp.cy};
}
__device__ __forceinline__ Edges step_y(const Footprint& fp) {
  const int64_t s = fp.neg ? -256 : 256;
  return Edges{s * fp.bx, s * (fp.cx - fp.bx), -s * fp.cx};
}
__device__ __forceinline__ bool inside(const Edges& e) { return (e.e0 | e.e1 | e.e2) >= 0; }
__device__ __forceinline__ void add(Edges& e, const Edges& d) {
  e.e0 += d.e0; e.e1 += d.e1; e.e2 += d.e2;
}
__device__ __forceinline__ Edges madd(const Edges& a, int64_t k, const Edges& b) {
  return Edges{a.e0 + k * b.e0, a.e1 + k * b.e1, a.e2 + k * b.e2};
}

// The same in 32 bits. At texel (tx0 + i, ty0 + j) an edge function is its
// value at (tx0, ty0) plus 256 (i dx + j dy) with dx, dy differences of the
// vertices, so its sign is that of (value >> 8) + i dx + j dy (the shift rounds
// down). With every vertex within 2^17 (512 texels) of the first one the
// texel range is at most 1024 a side, |dx|, |dy| < 2^18 and |value| < 2^37, so
// that these stay below 2^30 over the range and a 16-texel tile past its end.
struct Edges32 {
  int32_t e0, e1, e2;
};
constexpr int32_t kNear32 = 1 << 17;
__device__ __forceinline__ bool fits32(const Footprint& f) {
  return max(max(abs(f.bx), abs(f.by)), max(abs(f.cx), abs(f.cy))) < kNear32;
}
__device__ __forceinline__ Edges32 start32(const Footprint& f) {
  const Edges e = edges_at(f, f.tx0, f.ty0);
  return Edges32{(int32_t)(e.e0 >> 8), (int32_t)(e.e1 >> 8), (int32_t)(e.e2 >> 8)};
}
__device__ __forceinline__ Edges32 dx32(const Footprint& f) {
  const int32_t s = f.neg ? -1 : 1;
  return Edges32{-s * f.by, -s * (f.cy - f.by), s * f.cy};
}
__device__ __forceinline__ Edges32 dy32(const Footprint& f) {
  const int32_t s = f.neg ? -1 : 1;
  return Edges32{s * f.bx, s * (f.cx - f.bx), -s * f.cx};
}
__device__ __forceinline__ bool inside(const Edges32& e) { return (e.e0 | e.e1 | e.e2) >= 0; }
__device__ __forceinline__ void add(Edges32& e, const Edges32& d) {
  e.e0 += d.e0; e.e1 += d.e1; e.e2 += d.e2;
}

__global__ void k_occ_fill(int4* __restrict__ occ, int64_t n4) {
  const int4 neg = make_int4(-1, -1, -1, -1);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x)
    occ[i] = neg;
}

// All texels of a footprint by one lane, row by row, edge functions stepped.
template <typename E>
__device__ __forceinline__ void raster_rows(const Footprint& fp, E r, const E dx, const E dy,
                                            int32_t* __restrict__ occ, int omega) {
  for (int ty = fp.ty0; ty <= fp.ty1; ++ty) {
    int32_t* row = occ + (int64_t)ty * omega;
    E e = r;
    for (int tx = fp.tx0; tx <= fp.tx1; ++tx) {
      if (inside(e)) row[tx] = fp.chart;
      add(e, dx);
    }
    add(r, dy);
  }
}
__device__ __forceinline__ void raster_lane(const Footprint& fp, int32_t* __restrict__ occ,
                                            int omega) {
  if (fits32(fp))
    raster_rows(fp, start32(fp), dx32(fp), dy32(fp), occ, omega);
  else
    raster_rows(fp, edges_at(fp, fp.tx0, fp.ty0), step_x(fp), step_y(fp), occ, omega);
}

__device__ __forceinline__ int rl(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

// The texels of every lane's footprint (n texels; 0 for none), concatenated in
// lane order and row-major inside a footprint, by the whole wave 64 at a time:
// the lane taking texel g finds the footprint holding it, the last one that
// starts at or before g, from marks where they start (`mark`, 64 words of the
// wave's own) and a prefix maximum, and fetches that footprint from its lane.
// Neighbouring lanes then write neighbouring texels of one row, so the stores
// coalesce (one lane per footprint scatters 4-byte stores over the map, several
// times slower). Bound by the chain of lane exchanges: with a binary search for
// the footprint and 64-bit edge functions the small raster of an 8k-triangle
// frame took 8.8 us, 8.1 so.
__device__ __forceinline__ void raster_expand(const Footprint& f, int n, int32_t* __restrict__ occ,
                                              int omega, uint32_t* mark) {
  const int lane = lane_id();
  const int incl = (int)wave_incl_scan_dpp((uint32_t)n);
  const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
  const int start = incl - n;
  const bool near = __ballot(n > 0 && !fits32(f)) == 0;
  const Edges32 e0 = start32(f);
  for (int c = 0; c < total; c += kWave) {
    const int g = c + lane;
    mark[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (n > 0 && incl > c && start < c + kWave) mark[max(start - c, 0)] = (uint32_t)lane + 1u;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int pos = (int)wave_incl_max_dpp(mark[lane]) - 1;  // (texel c has a footprint)
    Footprint o;
    o.bx = __shfl(f.bx, pos, kWave);
    o.by = __shfl(f.by, pos, kWave);
    o.cx = __shfl(f.cx, pos, kWave);
    o.cy = __shfl(f.cy, pos, kWave);
    o.tx0 = __shfl(f.tx0, pos, kWave);
    o.tx1 = __shfl(f.tx1, pos, kWave);
    o.ty0 = __shfl(f.ty0, pos, kWave);
    o.chart = __shfl(f.chart, pos, kWave);
    o.neg = __shfl(f.neg, pos, kWave);
    const int li = g - __shfl(start, pos, kWave);
    const int nx = max(o.tx1 - o.tx0 + 1, 1);  // lanes past the total read an unused lane
    int row = (int)((float)li / (float)nx);
    if (row * nx > li) --row;
    else if ((row + 1) * nx <= li) ++row;
    const int i = li - row * nx, tx = o.tx0 + i, ty = o.ty0 + row;
    bool in;
    if (near) {
      const Edges32 dx = dx32(o), dy = dy32(o);
      in = inside(Edges32{__shfl(e0.e0, pos, kWave) + i * dx.e0 + row * dy.e0,
                          __shfl(e0.e1, pos, kWave) + i * dx.e1 + row * dy.e1,
                          __shfl(e0.e2, pos, kWave) + i * dx.e2 + row * dy.e2});
    } else {
      o.ax = __shfl(f.ax, pos, kWave);
      o.ay = __shfl(f.ay, pos, kWave);
      in = inside(edges_at(o, tx, ty));
    }
    if (g < total && in) occ[(int64_t)ty * omega + tx] = o.chart;
  }
}

constexpr int kOccTile = 16;                   // queued footprints are cut into 16x16 tiles
constexpr unsigned long long kSlotShift = 40;  // queue counter: footprints << 40 | tiles

// Occupancy of the visible triangles. Per fan footprint (texel range of n
// texels): n <= lane_texels by its own lane; lane_texels < n <= small_texels
// by the wave's coalesced expansion; larger ones are queued for k_occ_big. Both fans of every
// triangle are set up first and the queue is reserved with one atomic per
// workgroup and step (a single counter serializes at about 12 ns per atomic);
// the rasterization after it runs without barriers.
constexpr int kOccSmallBlock = 256;

__device__ __forceinline__ uint32_t tiles_of(const Footprint& fp, uint32_t* tiles_x) {
  *tiles_x = (uint32_t)((fp.tx1 - fp.tx0 + kOccTile) / kOccTile);
  return *tiles_x * (uint32_t)((fp.ty1 - fp.ty0 + kOccTile) / kOccTile);
}

template <int UV_PER>
__device__ __forceinline__ void k_occ_small_body(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ vlist, FrameParams p,
    const float* __restrict__ pos, const int32_t* __restrict__ cot,
    const fa_chart* __restrict__ charts, const int4* __restrict__ chart_tex,
    int32_t* __restrict__ occ, ulonglong2* __restrict__ big, int4* __restrict__ big_fp,
    uint32_t big_cap, int small_texels,
    int lane_texels, unsigned long long* __restrict__ big_counter,
    const FrameState* __restrict__ stp, unsigned occ_blocks, int64_t V,
    const int32_t* __restrict__ cov, float2* __restrict__ uv) {
  __shared__ uint32_t wcnt[kOccSmallBlock / kWave], wtil[kOccSmallBlock / kWave];
  __shared__ uint32_t marks[kOccSmallBlock / kWave][kWave];
  __shared__ unsigned long long bbase;
  if (blockIdx.x >= occ_blocks) {
    uv_block<UV_PER>(blockIdx.x - occ_blocks, p, pos, cov, charts, uv, V, stp);
    return;
  }
  const FrameState st = *stp;
  if (st.status != FA_OK) return;
  const int nv = st.visible;
  const int lane = lane_id(), w = threadIdx.x / kWave;
  // the launch's block size, as a constant: a loop over a runtime wave count
  // is unrolled eight times with live temporaries (100 instead of 89 VGPRs:
  // four instead of five resident waves per SIMD)
  constexpr int nw = kOccSmallBlock / kWave;
  constexpr unsigned long long kLow = (1ull << kSlotShift) - 1;
  for (int i0 = blockIdx.x * blockDim.x; i0 < nv; i0 += occ_blocks * blockDim.x) {
    const int i = i0 + threadIdx.x;
    const bool valid = i < nv;
    SnapPoly sp;
    sp.n = 0;
    sp.chart = -1;
    const int t = valid ? vlist[i] : 0;
    if (valid) snap_polygon(t, idx, pos, cot, charts, p, st, sp);
    Footprint fa, fb;
    const int4 box = sp.n > 0 ? chart_tex[sp.chart] : make_int4(0, -1, 0, -1);
    const bool oka = sp.n > 0 && fan_footprint(sp, 0, box, p.omega, fa);
    const bool okb = sp.n > 3 && fan_footprint(sp, 1, box, p.omega, fb);
    const int na = oka ? (fa.tx1 - fa.tx0 + 1) * (fa.ty1 - fa.ty0 + 1) : 0;
    const int nb = okb ? (fb.tx1 - fb.tx0 + 1) * (fb.ty1 - fb.ty0 + 1) : 0;
    const bool wa = oka && na > small_texels, wb = okb && nb > small_texels;
    uint32_t txa = 0, txb = 0;
    const uint32_t nta = wa ? tiles_of(fa, &txa) : 0u, ntb = wb ? tiles_of(fb, &txb) : 0u;
    // queue order: wave-major, then lane, fan a before fan b
    const uint32_t mine = (uint32_t)wa + (uint32_t)wb, mine_t = nta + ntb;
    const uint32_t c_in = wave_incl_scan<uint32_t>(mine) - mine;
    const uint32_t t_in = wave_incl_scan<uint32_t>(mine_t) - mine_t;
    if (lane == kWave - 1) {
      wcnt[w] = c_in + mine;
      wtil[w] = t_in + mine_t;
    }
    __syncthreads();
    uint32_t c_before = 0, t_before = 0, c_all = 0, t_all = 0;
    for (int k = 0; k < nw; ++k) {
      const uint32_t c = wcnt[k], tl = wtil[k];
      if (k < w) {
        c_before += c;
        t_before += tl;
      }
      c_all += c;
      t_all += tl;
    }
    if (threadIdx.x == 0 && c_all)
      bbase = atomicAdd(big_counter, ((unsigned long long)c_all << kSlotShift) | t_all);
    __syncthreads();
    bool qa = false, qb = false;
    if (c_all) {
      const unsigned long long old = bbase;
      unsigned long long slot = (old >> kSlotShift) + c_before + c_in;
      unsigned long long tile = (old & kLow) + t_before + t_in;
      // x: footprint code | tiles across << 32; y: first tile | tiles << 40
      if (wa && slot < big_cap) {
        big[slot] = make_ulonglong2((unsigned long long)(2 * (int64_t)t) |
                                        ((unsigned long long)txa << 32),
                                    tile | ((unsigned long long)nta << kSlotShift));
        put_footprint(big_fp + 3 * slot, fa);
        qa = true;
      }
      slot += wa;
      tile += nta;
      if (wb && slot < big_cap) {
        big[slot] = make_ulonglong2((unsigned long long)(2 * (int64_t)t + 1) |
                                        ((unsigned long long)txb << 32),
                                    tile | ((unsigned long long)ntb << kSlotShift));
        put_footprint(big_fp + 3 * slot, fb);
        qb = true;
      }
    }
    const bool ca = oka && !qa && na > lane_texels, cb = okb && !qb && nb > lane_texels;
    if (oka && !qa && !ca) raster_lane(fa, occ, p.omega);
    if (okb && !qb && !cb) raster_lane(fb, occ, p.omega);
    raster_expand(fa, ca ? na : 0, occ, p.omega, marks[w]);
    if (__ballot(cb)) raster_expand(fb, cb ? nb : 0, occ, p.omega, marks[w]);
  }
}
__global__ __launch_bounds__(kOccSmallBlock) void k_occ_small(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ vlist, FrameParams p,
    const float* __restrict__ pos, const int32_t* __restrict__ cot,
    const fa_chart* __restrict__ charts, const int4* __restrict__ chart_tex,
    int32_t* __restrict__ occ, ulonglong2* __restrict__ big, int4* __restrict__ big_fp,
    uint32_t big_cap, int small_texels,
    int lane_texels, unsigned long long* __restrict__ big_counter,
    const FrameState* __restrict__ stp, unsigned occ_blocks, int64_t V,
    const int32_t* __restrict__ cov, float2* __restrict__ uv) {
  k_occ_small_body<kUvPerFrame>(idx, vlist, p, pos, cot, charts, chart_tex, occ, big, big_fp,
                                big_cap, small_texels, lane_texels, big_counter, stp, occ_blocks,
                                V, cov, uv);
}

// Queued footprints: their texel ranges cut into 16x16 tiles, concatenated,
// are split evenly over all waves of the grid; a wave finds its first
// footprint by a 64-way search over the (increasing) first-tile indices and
// walks forward, 4 texels per lane.
// Bound by the vector unit: a tile is 256 texels whose edge functions took
// about 150 instructions in 64 bits. In 32 bits, with one sign test for edges
// and range, the last rows left out where the range ends before them, and tiles
// outside an edge dropped by the scalar unit, it is about 36 (91k tiles of a
// 2.2M-triangle frame 31 -> 22 us, 158k tiles 42 -> 28; of the rest the search
// and the set-up take 7 and the footprints' broadcasts 4). Wider searches (256
// probes a round) read more lines and are 1 us slower.
__device__ __forceinline__ void k_occ_big_body(
    FrameParams p, int32_t* __restrict__ occ,
    const ulonglong2* __restrict__ big, const int4* __restrict__ big_fp, uint32_t big_cap,
    const unsigned long long* __restrict__ big_counter, const FrameState* __restrict__ stp) {
  const FrameState st = *stp;
  if (st.status != FA_OK) return;
  const unsigned long long ctr =
      __hip_atomic_load(big_counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t nent = (uint32_t)min<unsigned long long>(ctr >> kSlotShift, big_cap);
  if (nent == 0) return;
  constexpr unsigned long long kLow = (1ull << kSlotShift) - 1;
  // (all tiles counted are queued unless the queue was full)
  uint64_t total = ctr & kLow;
  if (ctr >> kSlotShift > big_cap) {
    const ulonglong2 lastv = big[nent - 1];
    total = (lastv.y & kLow) + (lastv.y >> kSlotShift);
  }
  const uint64_t nwaves = (uint64_t)gridDim.x * (kBlock / kWave);
  // the wave index through readfirstlane: the compiler then knows it (and all
  // loop bounds below) to be uniform and keeps the tile loop's control scalar
  const uint64_t wid = (uint64_t)blockIdx.x * (kBlock / kWave) +
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint64_t per = (total + nwaves - 1) / nwaves;
  const uint64_t k0 = wid * per, k1 = min<uint64_t>(total, k0 + per);
  if (k0 >= k1) return;
  const int lane = lane_id();
  // last entry whose first tile <= k0; entry 0 starts at tile 0
  uint32_t lo = 0, hi = nent;
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + kWave - 1) / kWave;
    const uint32_t probe = lo + (uint32_t)lane * step;
    const bool le = probe < hi && (big[probe].y & kLow) <= k0;
    const int cnt = __popcll(__ballot(le));
    lo += (uint32_t)(cnt - 1) * step;
    hi = min(hi, lo + step);
  }
  // The wave's footprints are set up 64 at a time, one per lane (their
  // dependent loads overlap), then rasterized one after another with the
  // footprint broadcast from its lane.
  const int lx = lane % kOccTile, ly = lane / kOccTile;
  constexpr int kRows = kWave / kOccTile;
  static_assert(kOccTile == 4 * kRows, "a tile is four rows of texels a lane");
  const uint32_t row_bytes = 4u * (uint32_t)p.omega;
  for (uint32_t e0 = lo; e0 < nent;) {
    const uint32_t my = e0 + (uint32_t)lane;
    uint64_t base = 0, nt = 0;
    uint32_t tiles_x = 1;
    bool mine = false;
    Footprint f;
    f.ax = f.ay = f.bx = f.by = f.cx = f.cy = 0;
    f.tx0 = f.tx1 = f.ty0 = f.ty1 = f.chart = f.neg = 0;
    if (my < nent) {
      const ulonglong2 ent = big[my];
      base = ent.y & kLow;
      nt = ent.y >> kSlotShift;
      tiles_x = (uint32_t)(ent.x >> 32);
      mine = base < k1;
      if (mine) f = get_footprint(big_fp + 3 * (int64_t)my);
    }
    const int cnt = __popcll(__ballot(mine));  // entries start in order: a prefix of lanes
    // this wave's tiles of the footprint (it has fewer than 2^32, at most
    // (omega / 16)^2)
    const uint32_t first = (uint32_t)((k0 > base ? k0 : base) - base);
    const uint32_t last = (uint32_t)((k1 < base + nt ? k1 : base + nt) - base);
    const unsigned long long small = __ballot(fits32(f));
    const Edges32 start = start32(f), fdx = dx32(f), fdy = dy32(f);
    for (int j = 0; j < cnt; ++j) {
      const uint32_t t0 = (uint32_t)rl((int)first, j), t1 = (uint32_t)rl((int)last, j);
      const uint32_t txj = (uint32_t)rl((int)tiles_x, j);
      const int fx0 = rl(f.tx0, j), fx1 = rl(f.tx1, j), fy0 = rl(f.ty0, j), fy1 = rl(f.ty1, j);
      const int chart = rl(f.chart, j);
      // tile column and row of the first tile, stepped below
      uint32_t ti = 0, tj = 0;
      if (t0) {
        ti = t0 % txj;
        tj = t0 / txj;
      }
      if (small >> j & 1ull) {
        const Edges32 dx{rl(fdx.e0, j), rl(fdx.e1, j), rl(fdx.e2, j)};
        const Edges32 dy{rl(fdy.e0, j), rl(fdy.e1, j), rl(fdy.e2, j)};
        // at the tile's first texel (uniform) and at that of its row of tiles;
        // the lane's offset; the most that a tile's texels have over its first
        constexpr int32_t kIn = kOccTile - 1;
        const int32_t ci = kOccTile * (int)ti, ri = kOccTile * (int)tj;
        Edges32 row{rl(start.e0, j) + ri * dy.e0, rl(start.e1, j) + ri * dy.e1,
                    rl(start.e2, j) + ri * dy.e2};
        Edges32 eo{row.e0 + ci * dx.e0, row.e1 + ci * dx.e1, row.e2 + ci * dx.e2};
        const Edges32 off{__mul24(lx, dx.e0) + __mul24(ly, dy.e0),
                          __mul24(lx, dx.e1) + __mul24(ly, dy.e1),
                          __mul24(lx, dx.e2) + __mul24(ly, dy.e2)};
        const Edges32 most{kIn * (max(dx.e0, 0) + max(dy.e0, 0)),
                           kIn * (max(dx.e1, 0) + max(dy.e1, 0)),
                           kIn * (max(dx.e2, 0) + max(dy.e2, 0))};
        const Edges32 dq{kRows * dy.e0, kRows * dy.e1, kRows * dy.e2};
        // texels to the range's last column and row from the lane's texel of
        // the first tile, and that texel's byte in the map (below 2^28)
        const int wide = fx1 - fx0 - lx, high = fy1 - fy0 - ly;
        const uint32_t lane_at = 4u * ((uint32_t)(fy0 + ly) * (uint32_t)p.omega +
                                       (uint32_t)(fx0 + lx));
        int i = ci, r = ri;
        for (uint32_t tt = t0; tt < t1; ++tt) {
          if (inside(Edges32{eo.e0 + most.e0, eo.e1 + most.e1, eo.e2 + most.e2})) {
            Edges32 ev{eo.e0 + off.e0, eo.e1 + off.e1, eo.e2 + off.e2};
            // negative where the lane's texel is past the last column or row,
            // or outside an edge
            const int left = wide - i, below = high - r;
            const uint32_t at =
                lane_at + 4u * ((uint32_t)r * (uint32_t)p.omega + (uint32_t)i);
            char* map = reinterpret_cast<char*>(occ);
            auto rows = [&](int q0) {
              int32_t out[2];
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                out[q] = ev.e0 | ev.e1 | ev.e2 | left | (below - (q0 + q) * kRows);
                add(ev, dq);
              }
#pragma unroll
              for (int q = 0; q < 2; ++q)
                if (out[q] >= 0)
                  *reinterpret_cast<int32_t*>(map + at + (q0 + q) * kRows * row_bytes) = chart;
            };
            rows(0);
            if (fy0 + r + 2 * kRows <= fy1) rows(2);
          }
          i += kOccTile;
          eo.e0 += kOccTile * dx.e0;
          eo.e1 += kOccTile * dx.e1;
          eo.e2 += kOccTile * dx.e2;
          if (++ti == txj) {
            ti = 0;
            i = 0;
            r += kOccTile;
            row.e0 += kOccTile * dy.e0;
            row.e1 += kOccTile * dy.e1;
            row.e2 += kOccTile * dy.e2;
            eo = row;
          }
        }
        continue;
      }
      Footprint fp;
      fp.ax = rl(f.ax, j); fp.ay = rl(f.ay, j);
      fp.bx = rl(f.bx, j); fp.by = rl(f.by, j);
      fp.cx = rl(f.cx, j); fp.cy = rl(f.cy, j);
      fp.neg = rl(f.neg, j);
      // The edge functions are linear in the texel: at the lane's texel they
      // are their value at the tile's first texel (uniform, scalar unit) plus
      // the lane's offset, fixed per footprint.
      const Edges dx = step_x(fp), dy = step_y(fp);
      const Edges off = madd(madd(Edges{0, 0, 0}, lx, dx), ly, dy);
      const Edges dq = madd(Edges{0, 0, 0}, kRows, dy);
      const int64_t row_step = (int64_t)kRows * p.omega;
      for (uint32_t tt = t0; tt < t1; ++tt) {
        const int ox = fx0 + kOccTile * (int)ti, oy = fy0 + kOccTile * (int)tj;
        const Edges eo = edges_at(fp, ox, oy);
        Edges ev{eo.e0 + off.e0, eo.e1 + off.e1, eo.e2 + off.e2};
        const int tx = ox + lx, ty0 = oy + ly;
        const bool col = tx <= fx1;
        int32_t* dst = occ + (int64_t)ty0 * p.omega + tx;
#pragma unroll
        for (int q = 0; q < kOccTile / kRows; ++q) {
          if (col && ty0 + q * kRows <= fy1 && inside(ev)) *dst = chart;
          add(ev, dq);
          dst += row_step;
        }
        if (++ti == txj) {
          ti = 0;
          ++tj;
        }
      }
    }
    if (cnt < kWave) break;
    e0 += kWave;
  }
}
__global__ __launch_bounds__(kBlock) void k_occ_big(
    FrameParams p, int32_t* __restrict__ occ,
    const ulonglong2* __restrict__ big, const int4* __restrict__ big_fp, uint32_t big_cap,
    const unsigned long long* __restrict__ big_counter, const FrameState* __restrict__ stp) {
  k_occ_big_body(p, occ, big, big_fp, big_cap, big_counter, stp);
}

__global__ void k_meta(FrameParams p, FrameState* stp,
                       const unsigned long long* __restrict__ big_counter,
                       fa_atlas_meta* __restrict__ meta) {
  if (threadIdx.x == 0) write_meta(p, stp, big_counter, false, 0ull, meta);
}

// Occupied texels and the frame record in one launch: every workgroup counts
// its share of the map and publishes the sum; the last one to finish (the
// one that draws the last ticket) adds them up and writes the record.
//
// Bound by reading the map back (about 5 TB/s), so only what a placed box
// reaches is read: each strip of kStripTexels columns up to the top of its
// highest box (above it the map holds the fill's -1). Every thread keeps its
// 16-byte column of the map and steps down the rows, kCountRows loads in
// flight. Against reading the whole map: 14.9 -> 11.7 us (4096^2, one view),
// 54.4 -> 15.1 (8192^2), 118 -> 47 (16 views); a map that the boxes fill
// (23.7k charts) stays at 14.8.
constexpr int kCountBlock = 1024;
constexpr int kCountRows = 8;
static_assert(kStripTexels % 4 == 0, "a 16-byte word lies in one strip");
__device__ __forceinline__ void k_occ_count_meta_body(
    FrameParams p, const int4* __restrict__ occ, unsigned long long* __restrict__ partial,
    FrameState* stp, const unsigned long long* __restrict__ big_counter,
    fa_atlas_meta* __restrict__ meta) {
  __shared__ unsigned long long sh[kCountBlock / kWave];
  __shared__ uint32_t last;
  const int row4 = p.omega / 4;  // 16-byte words per row (a power of two)
  static_assert(kCountBlock == 1 << 10, "columns and rows of a workgroup by shifts");
  const int lc = min(p.log2omega - 2, 10);  // log2 of the columns a workgroup covers at once
  const int step = (int)gridDim.x << (10 - lc);
  const int r_first = ((int)blockIdx.x << (10 - lc)) + ((int)threadIdx.x >> lc);
  uint32_t c32 = 0;
  for (int c = (int)threadIdx.x & ((1 << lc) - 1); c < row4; c += 1 << lc) {
    const int rows = (int)stp->strip_rows[4 * c / kStripTexels];
    const int4* __restrict__ col = occ + c;
    for (int r0 = r_first; r0 < rows; r0 += kCountRows * step) {
      int4 v[kCountRows];
#pragma unroll
      for (int u = 0; u < kCountRows; ++u) {
        const int r = r0 + u * step;
        v[u] = r < rows ? col[(int64_t)r * row4] : make_int4(-1, -1, -1, -1);
      }
#pragma unroll
      for (int u = 0; u < kCountRows; ++u)
        c32 += (v[u].x >= 0) + (v[u].y >= 0) + (v[u].z >= 0) + (v[u].w >= 0);
    }
  }
  // one thread counts at most 4 texels per 16-byte word it reads: far below 2^32
  const unsigned long long cnt = block_sum<unsigned long long>((unsigned long long)c32, sh);
  if (threadIdx.x == 0) {
    // the sum is stored at device scope and has completed (s_waitcnt on every
    // counter) before the ticket is taken, so whoever draws the last ticket
    // reads it with its device-scope load; no cache-wide release is needed
    __hip_atomic_store(&partial[blockIdx.x], cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    const uint32_t before = __hip_atomic_fetch_add(&stp->ticket, 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    last = before == gridDim.x - 1 ? 1u : 0u;
  }
  __syncthreads();
  if (!last) return;
  unsigned long long all = 0;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += blockDim.x)
    all += __hip_atomic_load(&partial[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  all = block_sum<unsigned long long>(all, sh);
  if (threadIdx.x == 0) write_meta(p, stp, big_counter, true, all, meta);
}
__global__ __launch_bounds__(kCountBlock) void k_occ_count_meta(
    FrameParams p, const int4* __restrict__ occ, unsigned long long* __restrict__ partial,
    FrameState* stp, const unsigned long long* __restrict__ big_counter,
    fa_atlas_meta* __restrict__ meta) {
  k_occ_count_meta_body(p, occ, partial, stp, big_counter, meta);
}

// ---- batched wrappers (view = blockIdx.y) --------------------------------
__global__ __launch_bounds__(kOccSmallBlock) void k_occ_small_b(
    const BatchView* __restrict__ bv, const int32_t* __restrict__ idx, uint32_t big_cap,
    int small_texels, int lane_texels, unsigned occ_blocks, int64_t V) {
  const BatchView& v = bv[blockIdx.y];
  k_occ_small_body<kUvPerBatch>(idx, in_global(v.w.vlist), v.p, in_global(v.w.pos), in_global(v.cot), in_global(v.charts), in_global(v.w.chart_tex), in_global(v.occ), in_global(v.w.big),
                   in_global(v.w.big_fp), big_cap, small_texels, lane_texels, in_global(v.w.big_counter), in_global(v.w.state),
                   occ_blocks, V, in_global(v.cov), reinterpret_cast<float2*>(in_global(v.uv)));
}
__global__ __launch_bounds__(kBlock) void k_occ_big_b(const BatchView* __restrict__ bv,
                                                      uint32_t big_cap) {
  const BatchView& v = bv[blockIdx.y];
  k_occ_big_body(v.p, in_global(v.occ), in_global(v.w.big), in_global(v.w.big_fp),
                 big_cap, in_global(v.w.big_counter), in_global(v.w.state));
}
__global__ __launch_bounds__(kCountBlock) void k_occ_count_meta_b(
    const BatchView* __restrict__ bv) {
  const BatchView& v = bv[blockIdx.y];
  k_occ_count_meta_body(v.p, reinterpret_cast<const int4*>(in_global(v.occ)), in_global(v.w.partial), in_global(v.w.state),
                        in_global(v.w.big_counter), in_global(v.meta));
}

}  // namespace

namespace {
// Workgroups of the count: every thread has its kCountRows loads (more
// workgroups than words keep a small map's count waiting for their launch: 10
// views of 512^2 took 26.5 us with kCountGrid each, 7.2 so).
unsigned count_grid(int omega) {
  const int64_t words = (int64_t)omega * omega / 4;
  return (unsigned)std::max<int64_t>(
      1, std::min<int64_t>(words / (kCountBlock * kCountRows), kCountGrid));
}
}  // namespace

hipError_t launch_uv(const int64_t V, const FrameParams& p, const Work& w, const int32_t* cov,
                     const fa_chart* charts, float* uv, hipStream_t st) {
  if (V > 0)
    k_uv<<<(unsigned)((V + kBlock * kUvPerFrame - 1) / (kBlock * kUvPerFrame)), kBlock, 0, st>>>(
        V, p, w.pos, cov, charts, reinterpret_cast<float2*>(uv), w.state);
  return hipGetLastError();
}

hipError_t launch_uv_corners(const int32_t* idx, int64_t T, const FrameParams& p, const Work& w,
                             const int32_t* cot, const fa_chart* charts, float* uv,
                             hipStream_t st) {
  if (T > 0)
    k_uv_corners<<<(unsigned)((T + kBlock - 1) / kBlock), kBlock, 0, st>>>(
        T, p, idx, w.pos, cot, charts, reinterpret_cast<float2*>(uv), w.state);
  return hipGetLastError();
}

hipError_t launch_occupancy(const int32_t* idx, int64_t T, const FrameParams& p, const Work& w,
                            const int32_t* cot, const fa_chart* charts, int32_t* occ,
                            int small_texels, int lane_texels, const OccExtras& x, Marker& mk,
                            hipStream_t st) {
  const int64_t n4 = (int64_t)p.omega * p.omega / 4;
  if (x.fill) {
    const unsigned fill_grid = (unsigned)std::min<int64_t>((n4 + kBlock - 1) / kBlock, 4096);
    k_occ_fill<<<fill_grid, kBlock, 0, st>>>(reinterpret_cast<int4*>(occ), n4);
  }
  mk(st);
  const uint32_t cap = (uint32_t)std::min<int64_t>(2 * std::max<int64_t>(T, 1), kBigCap);
  const int64_t V = x.uv ? x.V : 0;
  const unsigned occ_blocks = T > 0 ? visible_grid(T) : 0;
  const unsigned uv_blocks = (unsigned)((V + kOccSmallBlock * kUvPerFrame - 1) /
                                         (kOccSmallBlock * kUvPerFrame));
  if (occ_blocks + uv_blocks > 0)
    k_occ_small<<<occ_blocks + uv_blocks, kOccSmallBlock, 0, st>>>(
        idx, w.vlist, p, w.pos, cot, charts, w.chart_tex, occ, w.big, w.big_fp, cap, small_texels,
        lane_texels, w.big_counter, w.state, occ_blocks, V, x.cov,
        reinterpret_cast<float2*>(x.uv));
  mk(st);
  if (T > 0)
    k_occ_big<<<kOccBigGrid, kBlock, 0, st>>>(p, occ, w.big, w.big_fp, cap, w.big_counter,
                                              w.state);
  mk(st);
  if (x.meta)  // a scaled copy (no frame record) needs no count
    k_occ_count_meta<<<count_grid(p.omega), kCountBlock, 0, st>>>(p, reinterpret_cast<const int4*>(occ),
                                                         w.partial, w.state, w.big_counter, x.meta);
  mk(st);
  return hipGetLastError();
}

namespace {
// Texel range of every placed box for an atlas of side p.omega (the same exact
// integer membership test as at placement), and an empty large-footprint
// queue: the start of an occupancy pass at another atlas side.
__global__ void k_chart_tex(FrameParams p, const fa_chart* __restrict__ charts,
                            int4* __restrict__ chart_tex, unsigned long long* __restrict__ big_counter,
                            const FrameState* __restrict__ stp) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c == 0) *big_counter = 0ull;
  const FrameState st = *stp;
  if (st.status != FA_OK || c >= st.num_charts) return;
  const fa_chart& ch = charts[c];
  const int64_t om = p.omega, L = st.layout_w, L2 = 2 * L;
  chart_tex[c] = make_int4((int)ceil_div64(2 * (int64_t)ch.x * om - L, L2),
                           (int)ceil_div64(2 * ((int64_t)ch.x + ch.w) * om - L, L2) - 1,
                           (int)ceil_div64(2 * (int64_t)ch.y * om - L, L2),
                           (int)ceil_div64(2 * ((int64_t)ch.y + ch.h) * om - L, L2) - 1);
}
}  // namespace

hipError_t launch_occupancy_scaled(const int32_t* idx, int64_t T, const FrameParams& p,
                                   const Work& w, const int32_t* cot, const fa_chart* charts,
                                   int32_t* occ, int small_texels, int lane_texels,
                                   hipStream_t st) {
  k_chart_tex<<<(unsigned)((p.max_charts + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      p, charts, w.chart_tex, w.big_counter, w.state);
  Marker none;
  OccExtras x;
  return launch_occupancy(idx, T, p, w, cot, charts, occ, small_texels, lane_texels, x, none, st);
}

namespace {
// ---------------------------------------------------------------------------
// footprint push: full-scale profile of every chart
// ---------------------------------------------------------------------------
// Column u of chart c (prof[fp_off[c] + u], u < floor(oriented width) + 1)
// holds the first and last row, on the unit grid of the chart-local layout
// before scale and gutter, that the chart's snapped polygons reach inside the
// closed strip [u, u + 1] (first and last strips open outwards, rows clamped
// to the chart's floor(oriented height) + 1 rows). Exact integer arithmetic
// on the 1/256 snapped vertices: a side crossing's row is the floor of an
// exact rational. Empty column: (INT_MAX, -1).

// floor((py + (x0 - px) (qy - py) / (qx - px)) / 256), px != qx. Below 2^52
// the numerator and divisor are exact doubles: the rounded quotient is within
// one of the floor, and the exact integer remainder settles it.
__device__ __forceinline__ int32_t crossing_row(int64_t px, int64_t py, int64_t qx, int64_t qy,
                                                int64_t x0) {
  int64_t num = py * (qx - px) + (x0 - px) * (qy - py);
  int64_t den = qx - px;
  if (den < 0) {
    num = -num;
    den = -den;
  }
  const int64_t d = 256 * den;
  const int64_t lim = int64_t(1) << 52;
  if (num > -lim && num < lim) {
    int64_t q = (int64_t)floor((double)num / (double)d);
    const int64_t r = num - q * d;
    if (r < 0) --q;
    else if (r >= d) ++q;
    return (int32_t)q;
  }
  return (int32_t)floor_div64(num, d);
}

// The same for coordinates within 2^24, in doubles: products, sums and the
// remainder are whole numbers below 2^53 and so exact, the quotient is below
// 2^17 and comes from an approximate reciprocal (2^-20 or better) within one
// of the floor, and the remainder settles it.
constexpr int32_t kNearRow = 1 << 24;
__device__ __forceinline__ int32_t crossing_row_near(int32_t px, int32_t py, int32_t qx,
                                                     int32_t qy, int32_t x0) {
  const double run = (double)(qx - px), sg = run < 0.0 ? -1.0 : 1.0;
  const double num = sg * fma((double)py, run, (double)(x0 - px) * (double)(qy - py));
  const double d = 256.0 * sg * run;
  double q = floor(num * __builtin_amdgcn_rcp(d));
  const double r = fma(-q, d, num);
  if (r < 0.0) q -= 1.0;
  else if (r >= d) q += 1.0;
  return (int32_t)q;
}

// Setup of one visible-list entry for the profile raster: its near-clipped
// polygon snapped to the chart-local unit grid (1/256), the chart's column
// and row counts and first profile entry, and the columns [u0, u0 + cnt) it
// reaches (cnt = 0: nothing).
struct FpSetup {
  int32_t X[4], Y[4];
  int n, Uc, Rc, off, u0, cnt;
  bool near;  // every coordinate within kNearRow
};
__device__ __forceinline__ void fp_setup(int i, int nv, const int32_t* __restrict__ vlist,
                                         const int32_t* __restrict__ idx,
                                         const float* __restrict__ pos,
                                         const int32_t* __restrict__ cot,
                                         const fa_chart* __restrict__ charts,
                                         const int32_t* __restrict__ fp_off, const FrameParams& p,
                                         FpSetup& s) {
#pragma unroll
  for (int k = 0; k < 4; ++k) s.X[k] = s.Y[k] = 0;
  s.n = 0; s.Uc = 1; s.Rc = 1; s.off = 0; s.u0 = 0; s.cnt = 0; s.near = true;
  if (i >= nv) return;
  const float halfW = 0.5f * (float)p.W, halfH = 0.5f * (float)p.H;
  const int t = vlist[i];
  const int c = cot[t];
  const float4 a = clip_of(pos, idx[3 * (int64_t)t], p),
               b = clip_of(pos, idx[3 * (int64_t)t + 1], p),
               cc = clip_of(pos, idx[3 * (int64_t)t + 2], p);
  const bool out = c < 0 || outside<0>(a, b, cc) || outside<1>(a, b, cc) ||
                   outside<2>(a, b, cc) || outside<3>(a, b, cc) || outside<4>(a, b, cc) ||
                   outside<5>(a, b, cc);
  if (out) return;
  float4 poly[4];
  int n;
  if (pd<4>(a) < 0.0f || pd<4>(b) < 0.0f || pd<4>(cc) < 0.0f) {
    n = near_clip(a, b, cc, poly);
  } else {
    poly[0] = a; poly[1] = b; poly[2] = cc; poly[3] = cc; n = 3;
  }
  bool ok = n > 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) ok = ok && (k >= n || poly[k].w > 0.0f);
  if (!ok) return;
  const fa_chart& ch = charts[c];
  const float x0 = ch.ndc_box[0], y1 = ch.ndc_box[3], tw = ch.target_w;
  const int rot = ch.rotated;
  int32_t xmin = INT_MAX, xmax = INT_MIN;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < n) {
      const float nx = poly[k].x / poly[k].w, ny = poly[k].y / poly[k].w;
      const float px = ((nx - x0) * halfW) * p.rate;
      const float py = ((y1 - ny) * halfH) * p.rate;
      s.X[k] = snap(rot ? py : px);
      s.Y[k] = snap(rot ? (tw - px) : py);
      xmin = min(xmin, s.X[k]);
      xmax = max(xmax, s.X[k]);
      s.near = s.near && max(abs(s.X[k]), abs(s.Y[k])) <= kNearRow;
    }
  }
  s.n = n;
  s.Uc = (int)floorf(ch.oriented_w) + 1;
  s.Rc = (int)floorf(ch.oriented_h) + 1;
  s.off = fp_off[c];
  s.u0 = min(s.Uc - 1, max(0, xmin >> 8));
  s.cnt = min(s.Uc - 1, max(0, xmax >> 8)) - s.u0 + 1;
}

// What the raster needs of a set-up entry, 48 bytes: the polygon (a triangle's
// third vertex twice; 0 vertices: no columns) and `chart`: first profile entry,
// rows | vertices << 25 | near << 28, columns, columns reached. Rows past 2^20,
// which no snapped vertex reaches, are cut off.
struct FpRecord {
  int4 X, Y, chart;
};
__device__ __forceinline__ FpRecord fp_record(const FpSetup& s) {
  const bool four = s.n > 3;
  const int rows = min(s.Rc, 1 << 24);
  return FpRecord{make_int4(s.X[0], s.X[1], s.X[2], four ? s.X[3] : s.X[2]),
                  make_int4(s.Y[0], s.Y[1], s.Y[2], four ? s.Y[3] : s.Y[2]),
                  make_int4(s.off, rows | s.n << 25 | (int)s.near << 28, s.Uc, s.cnt)};
}

// Count: the (triangle, column) items of every group of 64 consecutive
// visible-list entries (group g = entries 64 g .. 64 g + 63), one wave per
// group; the blocks past the groups clear the profile. The entries' records go
// to `rec` (the large-footprint queue's memory, free until the occupancy),
// unless there are more than rec_cap of them.
__global__ __launch_bounds__(kBlock) void k_fp_count(
    const int32_t* __restrict__ vlist, const int32_t* __restrict__ idx,
    const float* __restrict__ pos, const int32_t* __restrict__ cot,
    const fa_chart* __restrict__ charts, const int32_t* __restrict__ fp_off,
    unsigned long long* __restrict__ group_items, int2* __restrict__ prof, unsigned count_blocks,
    int4* __restrict__ rec, int rec_cap, FrameParams p, const FrameState* __restrict__ stp) {
  if (stp->status != FA_OK) return;
  if (blockIdx.x >= count_blocks) {
    const int ncol = stp->fp_columns;
    const int64_t stride = (int64_t)(gridDim.x - count_blocks) * blockDim.x;
    for (int64_t e = (int64_t)(blockIdx.x - count_blocks) * blockDim.x + threadIdx.x; e < ncol;
         e += stride)
      prof[e] = make_int2(INT_MAX, -1);
    return;
  }
  const int nv = stp->visible;
  const int groups = (nv + kWave - 1) / kWave;
  const int nw = (int)(count_blocks * (blockDim.x / kWave));
  for (int g = (int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave); g < groups;
       g += nw) {
    FpSetup s;
    const int i = g * kWave + lane_id();
    fp_setup(i, nv, vlist, idx, pos, cot, charts, fp_off, p, s);
    if (i < nv && nv <= rec_cap) {
      const FpRecord r = fp_record(s);
      rec[3 * (int64_t)i] = r.X;
      rec[3 * (int64_t)i + 1] = r.Y;
      rec[3 * (int64_t)i + 2] = r.chart;
    }
    const int tot = wave_sum<int>(s.cnt);
    if (lane_id() == 0) group_items[g] = (unsigned long long)tot;
  }
}

// Scan: exclusive prefix of the groups' item counts in place, the total after
// the last group (one workgroup).
__global__ __launch_bounds__(1024) void k_fp_scan(unsigned long long* __restrict__ group_items,
                                                 const FrameState* __restrict__ stp) {
  __shared__ unsigned long long sh[1024 / kWave];
  if (stp->status != FA_OK) return;
  const int groups = (stp->visible + kWave - 1) / kWave;
  const int per = (groups + 1023) / 1024;
  const int b = min(groups, (int)threadIdx.x * per), e = min(groups, b + per);
  unsigned long long sum = 0;
  for (int g = b; g < e; ++g) sum += group_items[g];
  unsigned long long total = 0;
  unsigned long long run = block_incl_scan<unsigned long long>(sum, sh, &total) - sum;
  for (int g = b; g < e; ++g) {
    const unsigned long long v = group_items[g];
    group_items[g] = run;
    run += v;
  }
  if (threadIdx.x == 0) group_items[groups] = total;
}

// Raster: the frame's (triangle, column) items are split evenly over all
// waves (a wave's share is a contiguous range of the groups' items), so the
// columns of a few large triangles no longer load one wave. A wave finds the
// group holding its first item by a 64-way search over the group prefix and
// walks forward; of each group it touches, its lanes fetch the 64 records into
// LDS (first entry and column relative to the items) and the wave takes that
// group's items in its range 64 at a time. The owner of an item is the last one
// whose items start at or before it: a mark where each starts and a prefix
// maximum.
// An item looks for the sides that cross the left border of its column and
// takes those crossing the right one from the lane after it, which owns the
// next column.
// Neighbouring triangles share columns: the workgroup reduces kFpWin profile
// entries around those of its first items in LDS and flushes each touched one
// with one pair of global atomics; entries elsewhere (of other charts, mostly)
// take global atomics, after a look whether they would change anything (values
// only ever move one way, so an old one is safe to look at).
// Bound by the items' vector instructions and by the global atomics. Its
// workgroups are as many as the chip holds at once, whatever the mesh: few
// triangles may have many columns. With each item trying every side on both
// borders in 64-bit arithmetic, the set-up repeated, the owner's values fetched
// lane by lane and a window per wave and group, 2.2M-triangle frames (131k
// visible) took 85 us and one of 1500 triangles 28 or more; now 25 and 8, and
// the records add 4 to the count.
constexpr int kFpWin = 2048;
constexpr unsigned kFpGrid = 5 * 256;

__global__ __launch_bounds__(kBlock) void k_fp_raster(
    const int32_t* __restrict__ vlist, const int32_t* __restrict__ idx,
    const float* __restrict__ pos, const int32_t* __restrict__ cot,
    const fa_chart* __restrict__ charts, const int32_t* __restrict__ fp_off,
    const unsigned long long* __restrict__ group_first, int2* __restrict__ prof,
    const int4* __restrict__ rec, int rec_cap, FrameParams p,
    const FrameState* __restrict__ stp) {
  __shared__ int2 win[kFpWin];
  __shared__ int span_lo[kBlock / kWave], span_hi[kBlock / kWave];
  __shared__ int4 all_x[kBlock / kWave][kWave], all_y[kBlock / kWave][kWave];
  __shared__ int4 all_c[kBlock / kWave][kWave];
  __shared__ uint32_t all_mark[kBlock / kWave][kWave];
  if (stp->status != FA_OK) return;
  const int nv = stp->visible;
  const int groups = (nv + kWave - 1) / kWave;
  if (groups == 0) return;
  const unsigned long long total = group_first[groups];
  const int lane = lane_id();
  const unsigned long long nwaves = gridDim.x * (blockDim.x / kWave);
  const unsigned long long wave = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const unsigned long long per = max((total + nwaves - 1) / nwaves, (unsigned long long)kWave);
  if (blockIdx.x * (unsigned long long)(blockDim.x / kWave) * per >= total) return;  // (no items)
  const unsigned long long k0 = min(total, wave * per), k1 = min(total, k0 + per);
  const int w = threadIdx.x / kWave;
  int4* lds_x = all_x[w];
  int4* lds_y = all_y[w];
  int4* lds_c = all_c[w];
  uint32_t* mark = all_mark[w];
  auto settle = [] {  // LDS writes of the wave's lanes before its later reads
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  for (int e = threadIdx.x; e < kFpWin; e += kBlock) win[e] = make_int2(INT_MAX, -1);
  // this wave's items of a group: [ia, ib) in group-local numbering; a lane's
  // are [st0, st0 + cnt)
  int ia = 0, ib = 0, cnt = 0, st0 = 0;
  auto fetch = [&](int g, unsigned long long gfirst, int& elo, int& ehi) {
    FpRecord r{make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0)};
    const int i = g * kWave + lane;
    if (nv <= rec_cap) {
      if (i < nv)
        r = FpRecord{rec[3 * (int64_t)i], rec[3 * (int64_t)i + 1], rec[3 * (int64_t)i + 2]};
    } else {
      FpSetup s;
      fp_setup(i, nv, vlist, idx, pos, cot, charts, fp_off, p, s);
      r = fp_record(s);
    }
    cnt = r.chart.w;
    const int u0 = min(r.chart.z - 1, max(0, min(min(r.X.x, r.X.y), min(r.X.z, r.X.w)) >> 8));
    const int incl = (int)wave_incl_scan_dpp((uint32_t)cnt);
    const int gtot = __builtin_amdgcn_readlane(incl, kWave - 1);
    ia = (int)(k0 > gfirst ? k0 - gfirst : 0ull);
    ib = (int)min<unsigned long long>((unsigned long long)gtot, k1 - gfirst);
    st0 = incl - cnt;
    const int ja = max(st0, ia), jb = min(incl, ib) - 1;
    const bool mine = cnt > 0 && ja <= jb;
    elo = mine ? r.chart.x + u0 + (ja - st0) : INT_MAX;
    ehi = mine ? r.chart.x + u0 + (jb - st0) : INT_MIN;
    lds_x[lane] = r.X;
    lds_y[lane] = r.Y;
    lds_c[lane] = make_int4(r.chart.x + u0 - st0, u0 - st0, r.chart.y, r.chart.z - 1);
  };
  // last group whose first item <= k0 (group 0 starts at item 0)
  int g = 0, elo = INT_MAX, ehi = INT_MIN;
  if (k0 < k1) {
    int hi = groups;
    while (hi - g > 1) {
      const int step = (hi - g + kWave - 1) / kWave;
      const int probe = g + lane * step;
      const bool le = probe < hi && group_first[probe] <= k0;
      const int c = __popcll(__ballot(le));
      g += (c - 1) * step;
      hi = min(hi, g + step);
    }
    fetch(g, group_first[g], elo, ehi);
    elo = wave_min<int>(elo);
    ehi = wave_max<int>(ehi);
  }
  if (lane == 0) {
    span_lo[w] = elo;
    span_hi[w] = ehi;
  }
  __syncthreads();
  // the window: from the lowest entry of the waves' first items, or, if they
  // span more, around those of the first wave
  int from = span_lo[0], to = span_hi[0];
#pragma unroll
  for (int k = 1; k < kBlock / kWave; ++k) {
    from = min(from, span_lo[k]);
    to = max(to, span_hi[k]);
  }
  if (to - from >= kFpWin) from = span_lo[0] + (span_hi[0] - span_lo[0]) / 2 - kFpWin / 2;
  from = max(from - 1, 0);  // (an item may reach into the entry before its own)
  while (k0 < k1) {
    for (int w0 = ia; w0 < ib; w0 += kWave) {
      const int item = w0 + lane;
      mark[lane] = 0u;
      settle();
      if (cnt > 0 && st0 + cnt > w0 && st0 < w0 + kWave) mark[max(st0 - w0, 0)] = (uint32_t)lane + 1u;
      settle();
      const int o = (int)wave_incl_max_dpp(mark[lane]) - 1;  // (item w0 has an owner)
      const int4 vx = lds_x[o], vy = lds_y[o], vc = lds_c[o];
      const int32_t PX[4] = {vx.x, vx.y, vx.z, vx.w}, PY[4] = {vy.x, vy.y, vy.z, vy.w};
      const int u = vc.y + item, entry = vc.x + item;
      const int rows = vc.z & ((1 << 25) - 1), on = vc.z >> 25 & 7;
      const bool near = vc.z >> 28 & 1;
      const bool here = item < ib;
      const bool open_l = u == 0, open_r = u == vc.w;
      const int32_t sl = 256 * u, sr = sl + 256;
      // rows of the sides that cross the column's left border: a triangle has
      // at most two there, one going right and one going left; of a
      // near-clipped quadrilateral, which rounding may bend, all four are tried
      int32_t clo = INT_MAX, chi = INT_MIN;
      auto cross = [&](int32_t px, int32_t py, int32_t qx, int32_t qy) {
        const int32_t r = near ? crossing_row_near(px, py, qx, qy, sl)
                               : crossing_row(px, py, qx, qy, sl);
        clo = min(clo, r);
        chi = max(chi, r);
      };
      if (here && !open_l && on == 3) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          int32_t px = 0, py = 0, qx = 0, qy = 0;
          bool has = false;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const int m = k == 2 ? 0 : k + 1;
            if (h ? PX[m] < sl && sl < PX[k] : PX[k] < sl && sl < PX[m]) {
              px = PX[k]; py = PY[k];
              qx = PX[m]; qy = PY[m];
              has = true;
            }
          }
          if (has) cross(px, py, qx, qy);
        }
      } else if (here && !open_l) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int m = k == 3 ? 0 : k + 1;
          if (k < on && min(PX[k], PX[m]) < sl && sl < max(PX[k], PX[m]))
            cross(PX[k], PY[k], PX[m], PY[m]);
        }
      }
      // the column before takes them too (they cross its right border): it is
      // the lane before's, but for the first lane
      const int32_t nlo = __shfl_down(clo, 1, kWave), nhi = __shfl_down(chi, 1, kWave);
      const int no = __shfl_down(o, 1, kWave);
      const bool next = lane < kWave - 1 && item + 1 < ib && no == o;
      if (!here) continue;
      int32_t rlo = clo, rhi = chi;
      if (next) {
        rlo = min(rlo, nlo);
        rhi = max(rhi, nhi);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if ((open_l || PX[k] >= sl) && (open_r || PX[k] <= sr)) {
          rlo = min(rlo, PY[k] >> 8);
          rhi = max(rhi, PY[k] >> 8);
        }
      }
      auto put = [&](int e, int32_t lo_row, int32_t hi_row) {
        if (lo_row > hi_row) return;
        lo_row = min(rows - 1, max(0, lo_row));
        hi_row = min(rows - 1, max(0, hi_row));
        const int at = e - from;
        if (at >= 0 && at < kFpWin) {
          // (scoped to the workgroup, or the compiler joins them with the
          // global ones below into flat atomics)
          __hip_atomic_fetch_min(&win[at].x, lo_row, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_max(&win[at].y, hi_row, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
          const int32_t x = __hip_atomic_load(&prof[e].x, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
          const int32_t y = __hip_atomic_load(&prof[e].y, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
          if (lo_row < x) atomicMin(&prof[e].x, lo_row);
          if (hi_row > y) atomicMax(&prof[e].y, hi_row);
        }
      };
      put(entry, rlo, rhi);
      if (lane == 0) put(entry - 1, clo, chi);
    }
    settle();
    if (++g >= groups) break;
    const unsigned long long gfirst = group_first[g];
    if (gfirst >= k1) break;
    fetch(g, gfirst, elo, ehi);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kFpWin; e += kBlock) {
    const int2 v = win[e];
    if (v.y < 0) continue;
    atomicMin(&prof[from + e].x, v.x);
    atomicMax(&prof[from + e].y, v.y);
  }
}
}  // namespace

hipError_t launch_footprint(const int32_t* idx, int64_t T, const FrameParams& p, const Work& w,
                            const int32_t* cot, const fa_chart* charts, Marker& mk,
                            hipStream_t st) {
  const int rec_cap = (int)std::min<int64_t>(2 * T, kBigCap);  // (three int4 each)
  if (p.fp_cap > 0) {
    // one wave per group of 64 entries, then the blocks that clear the profile
    const unsigned cb = (unsigned)std::max<int64_t>(
        1, std::min<int64_t>((T + kBlock - 1) / kBlock, 2048));
    const unsigned clear = (unsigned)std::min<int64_t>(1024, (p.fp_cap + kBlock - 1) / kBlock);
    k_fp_count<<<cb + clear, kBlock, 0, st>>>(w.vlist, idx, w.pos, cot, charts, w.fp_off,
                                              w.fp_group, w.fp_prof, cb, w.big_fp, rec_cap, p,
                                              w.state);
  }
  mk(st);
  if (p.fp_cap > 0 && T > 0) {
    k_fp_scan<<<1, 1024, 0, st>>>(w.fp_group, w.state);
    k_fp_raster<<<kFpGrid, kBlock, 0, st>>>(w.vlist, idx, w.pos, cot, charts, w.fp_off,
                                                    w.fp_group, w.fp_prof, w.big_fp, rec_cap, p,
                                                    w.state);
  }
  mk(st);
  return hipGetLastError();
}

hipError_t launch_meta(const FrameParams& p, const Work& w, fa_atlas_meta* meta,
                       hipStream_t st) {
  k_meta<<<1, kWave, 0, st>>>(p, w.state, w.big_counter, meta);
  return hipGetLastError();
}

hipError_t launch_occupancy_batched(const BatchView* dev, int n, const int32_t* idx, int64_t T,
                                    int64_t V, int max_omega, int small_texels, int lane_texels,
                                    hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const uint32_t cap = (uint32_t)std::min<int64_t>(2 * std::max<int64_t>(T, 1), kBigCap);
  const unsigned occ_blocks = T > 0 ? view_groups(T, kOccSmallBlock, kOccSmallBlock, n) : 0;
  const unsigned uv_blocks = (unsigned)((V + kOccSmallBlock * kUvPerBatch - 1) /
                                         (kOccSmallBlock * kUvPerBatch));
  if (occ_blocks + uv_blocks > 0)
    k_occ_small_b<<<dim3(occ_blocks + uv_blocks, n), kOccSmallBlock, 0, st>>>(
        dev, idx, cap, small_texels, lane_texels, occ_blocks, V);
  if (T > 0)
    // (half as many: each wave starts with a search)
    k_occ_big_b<<<dim3(std::min<unsigned>(kOccBigGrid, kViewThreads / (2 * kBlock * n)), n),
                  kBlock, 0, st>>>(dev, cap);
  k_occ_count_meta_b<<<dim3(count_grid(max_omega), n), kCountBlock, 0, st>>>(dev);
  return hipGetLastError();
}

}  // namespace fa
