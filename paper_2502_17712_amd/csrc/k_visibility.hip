// Visible-triangle pass on gfx950 (App. "Detecting Visible Triangles": a depth
// pre-pass fills a depth buffer, a second pass tests each triangle's samples
// against it with "less or equal" and marks the triangles that pass).
//
// float64 throughout, fixed operation order, no contraction:
//   candidate  faces the eye ((b-a) x (c-a) . (eye-a) > 0) and no clip plane
//              has all three vertices outside;
//   occluder   candidate with every w > near (only these write and test depth);
//   depth      samples at the centres of a (W/k) x (H/k) grid; a covered
//              sample (edge functions all >= 0 or all <= 0, area != 0) gets the
//              NDC z interpolated with the edge-function weights; the buffer
//              keeps the minimum (64-bit order-preserving keys, atomicMin);
//   marking    an occluder stays visible iff it covers no sample (it cannot be
//              proven hidden) or some covered sample has z <= D + 1e-6;
//              candidates crossing the near plane stay visible.
#include <algorithm>
#include <cmath>

#include "fa_internal.h"

namespace fa {
namespace {

__device__ __forceinline__ double4 clip64(const VisParams& q, const double (&p)[3]) {
  const double x = p[0], y = p[1], z = p[2];
  double r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = ((q.M[4 * i] * x + q.M[4 * i + 1] * y) + q.M[4 * i + 2] * z) + q.M[4 * i + 3];
  return make_double4(r[0], r[1], r[2], r[3]);
}

// order-preserving key of a finite double (smaller value -> smaller key)
__device__ __forceinline__ unsigned long long dkey(double d) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(d);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double dval(unsigned long long k) {
  const unsigned long long b = (k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k;
  return __longlong_as_double((long long)b);
}

// the depth buffer is produced by atomics (possibly on other XCDs): read it
// with agent-scope loads
__device__ __forceinline__ unsigned long long dload(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Screen footprint of an occluder, from its clip-space vertices: vertices in
// coarse pixels (x right, y down) with their NDC z, and the range of sample
// centres inside its bounding box (all that the cull asks for).
struct Shot {
  double X[3], Y[3], Z[3];
  int ix0, ix1, iy0, iy1;
};

__device__ __forceinline__ void shot_of(const VisParams& q, const double4 (&c)[3], Shot& s) {
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    s.X[e] = ((c[e].x / c[e].w) * 0.5 + 0.5) * (double)q.Wc;
    s.Y[e] = (0.5 - (c[e].y / c[e].w) * 0.5) * (double)q.Hc;
    s.Z[e] = c[e].z / c[e].w;
  }
  const double xmin = fmin(fmin(s.X[0], s.X[1]), s.X[2]), xmax = fmax(fmax(s.X[0], s.X[1]), s.X[2]);
  const double ymin = fmin(fmin(s.Y[0], s.Y[1]), s.Y[2]), ymax = fmax(fmax(s.Y[0], s.Y[1]), s.Y[2]);
  s.ix0 = (int)fmin(fmax(ceil(xmin - 0.5), 0.0), (double)(q.Wc - 1));
  s.ix1 = (int)fmin(fmax(floor(xmax - 0.5), -1.0), (double)(q.Wc - 1));
  s.iy0 = (int)fmin(fmax(ceil(ymin - 0.5), 0.0), (double)(q.Hc - 1));
  s.iy1 = (int)fmin(fmax(floor(ymax - 0.5), -1.0), (double)(q.Hc - 1));
}

// Candidates, the list of occluders that have a sample in their bounding box
// (the others stay visible whatever the depth buffer holds), and the clearing
// of the depth buffer.
//
// Bound by the chain of index and position loads with about 200 float64
// instructions a triangle behind it: the next triangle's positions and the
// indices after those are in flight while one is computed, as whole 12-byte
// loads (nine single words a triangle kept the address units busy: 28 us on
// 2.2M triangles, 20 so). Each workgroup owns
// the chunks w, w + nseg, ... of kCullBlock triangles and a segment of the
// list as long as they are, so there is no counter to share or clear.
constexpr int kCullBlock = 512;
constexpr int kCullSegs = 512;  // most segments (workgroups with triangles)
static_assert(4 * kCullSegs <= 8 * kCountGrid, "the segments' counts use Work::partial");

__host__ __device__ inline int cull_segments(int64_t T) {
  const int64_t nc = (T + kCullBlock - 1) / kCullBlock;
  return (int)(nc < kCullSegs ? nc : kCullSegs);
}
// First entry of segment `w`: the triangles of the segments before it.
__device__ __forceinline__ int64_t segment_base(int64_t T, int nseg, int w) {
  const int64_t nc = (T + kCullBlock - 1) / kCullBlock;
  const int64_t each = nc / nseg, more = nc - each * nseg;
  const int64_t chunks = each * w + (w < more ? w : more);
  const int last = (int)((nc - 1) % nseg);  // owner of the last, perhaps partial, chunk
  return chunks * kCullBlock - (w > last ? nc * kCullBlock - T : 0);
}

__global__ __launch_bounds__(kCullBlock) void k_vis_cull(
    const float* __restrict__ pos, const int32_t* __restrict__ idx, int64_t T, int nseg,
    VisParams q, uint8_t* __restrict__ vis, int32_t* __restrict__ occl,
    uint32_t* __restrict__ counts, unsigned long long* __restrict__ depth, int64_t nd) {
  __shared__ uint32_t fill;
  const unsigned long long inf = 0xFFF0000000000000ull;  // dkey(+infinity)
  for (int64_t i = (int64_t)blockIdx.x * kCullBlock + threadIdx.x; i < nd;
       i += (int64_t)gridDim.x * kCullBlock)
    depth[i] = inf;
  if ((int)blockIdx.x >= nseg) return;
  if (threadIdx.x == 0) fill = 0u;
  __syncthreads();
  int32_t* seg = occl + segment_base(T, nseg, blockIdx.x);
  const int64_t step = (int64_t)nseg * kCullBlock;
  const int64_t first = (int64_t)blockIdx.x * kCullBlock + threadIdx.x;
  const float3* pos3 = reinterpret_cast<const float3*>(pos);
  const int3* idx3 = reinterpret_cast<const int3*>(idx);
  // (beyond the end: the last triangle, so that no load depends on a branch)
  int3 vn = idx3[min(first, T - 1)];  // indices of the triangle after next
  float3 pn[3] = {pos3[vn.x], pos3[vn.y], pos3[vn.z]};  // positions of the next triangle
  vn = idx3[min(first + step, T - 1)];
  // (whole waves: the appending below counts over the wave)
  for (int64_t t = first; t - lane_id() < T; t += step) {
    const double p[3][3] = {{pn[0].x, pn[0].y, pn[0].z},
                            {pn[1].x, pn[1].y, pn[1].z},
                            {pn[2].x, pn[2].y, pn[2].z}};
    pn[0] = pos3[vn.x];
    pn[1] = pos3[vn.y];
    pn[2] = pos3[vn.z];
    vn = idx3[min(t + 2 * step, T - 1)];
    double a[3], b[3], d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      a[k] = p[1][k] - p[0][k];
      b[k] = p[2][k] - p[0][k];
      d[k] = q.eye[k] - p[0][k];
    }
    const double n0 = a[1] * b[2] - a[2] * b[1];
    const double n1 = a[2] * b[0] - a[0] * b[2];
    const double n2 = a[0] * b[1] - a[1] * b[0];
    bool cand = t < T && ((n0 * d[0] + n1 * d[1]) + n2 * d[2]) > 0.0;
    bool listed = false;
    if (cand) {
      const double4 c[3] = {clip64(q, p[0]), clip64(q, p[1]), clip64(q, p[2])};
      const bool outside =
          (c[0].w + c[0].x < 0.0 && c[1].w + c[1].x < 0.0 && c[2].w + c[2].x < 0.0) ||
          (c[0].w - c[0].x < 0.0 && c[1].w - c[1].x < 0.0 && c[2].w - c[2].x < 0.0) ||
          (c[0].w + c[0].y < 0.0 && c[1].w + c[1].y < 0.0 && c[2].w + c[2].y < 0.0) ||
          (c[0].w - c[0].y < 0.0 && c[1].w - c[1].y < 0.0 && c[2].w - c[2].y < 0.0) ||
          (c[0].w + c[0].z < 0.0 && c[1].w + c[1].z < 0.0 && c[2].w + c[2].z < 0.0) ||
          (c[0].w - c[0].z < 0.0 && c[1].w - c[1].z < 0.0 && c[2].w - c[2].z < 0.0);
      cand = !outside;
      if (q.coarse > 0 && cand && c[0].w > q.near_w && c[1].w > q.near_w && c[2].w > q.near_w) {
        Shot s;
        shot_of(q, c, s);
        listed = s.ix0 <= s.ix1 && s.iy0 <= s.iy1;
      }
    }
    if (t < T) vis[t] = cand ? 1 : 0;
    const unsigned long long m = __ballot(listed);
    if (m) {
      uint32_t at = 0;
      if (lane_id() == 0) at = atomicAdd(&fill, (uint32_t)__popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      if (listed) seg[at + (uint32_t)__popcll(m & lanes_below())] = (int32_t)t;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = fill;
}

// Depth pre-pass and (MARK) the test against it. A workgroup sets up a batch
// of up to kVisBatch listed occluders and its threads share the samples of
// their bounding boxes, whichever triangle they belong to. Neighbours in the
// list are neighbours on the screen, and those under the camera have most of
// the samples (2.2M triangles: 569k occluders, 113k of them with samples, 325k
// samples), so a batch takes runs of kVisRun from all over the list; the work
// is then even and the passes wait for loads. The two passes on that scene,
// with the cull and the reuse flags: 133 us with a lane or a wave per occluder,
// 71 with consecutive batches of 64, 61 of 16, 45.2 in runs of 4 (runs of 8
// 47.2, single ones 46.5; 8 or 4 workgroups per CU 47, 3 52). Where samples are
// even all over the list, batches of 64 keep the lines of the depth buffer
// together: a heightfield of one million triangles at half resolution 52.7 us
// with them, 58.4 with runs of 4, but 119 and 70 on the scene above.
constexpr int kVisBatch = kWave;
constexpr int kVisRun = 4;
// Footprints of more samples than this are walked one after another, without
// looking for the owner of each sample, and short lists go one entry a
// workgroup (two triangles over all of 480 x 270 samples: 850 -> 121 us, forty
// over half of it 1550 -> 506; by one wave each they took 1040 and 17077).
// With 1024, 4096 and 16384: a 2.2M-triangle scene sampled at full resolution
// 180, 189 and 194 us, at half of it 69, 76 and 76; 1000 triangles of 50000
// samples 685 with each; only a list of 100000 triangles with 6000 samples each
// prefers to share them (7.06, 7.06 and 5.82 ms).
constexpr uint32_t kVisMany = 1024;
constexpr int kVisGrid = 6 * 256;  // most workgroups: what the chip holds at once

// edge functions of a footprint at the centre of sample (px, py); false: not
// covered
__device__ __forceinline__ bool covered(double X0, double X1, double X2, double Y0, double Y1,
                                        double Y2, int px, int py, double (&e)[3], double& area) {
  const double cx = (double)px + 0.5, cy = (double)py + 0.5;
  e[0] = (X2 - X1) * (cy - Y1) - (Y2 - Y1) * (cx - X1);
  e[1] = (X0 - X2) * (cy - Y2) - (Y0 - Y2) * (cx - X2);
  e[2] = (X1 - X0) * (cy - Y0) - (Y1 - Y0) * (cx - X0);
  area = (e[0] + e[1]) + e[2];
  return area != 0.0 && ((e[0] >= 0.0 && e[1] >= 0.0 && e[2] >= 0.0) ||
                         (e[0] <= 0.0 && e[1] <= 0.0 && e[2] <= 0.0));
}

template <bool MARK>
__global__ __launch_bounds__(kBlock, 6) void k_vis_depth(const float* __restrict__ pos,
                                                      const int32_t* __restrict__ idx, int64_t T,
                                                      int nseg, VisParams q,
                                                      const int32_t* __restrict__ occl,
                                                      const uint32_t* __restrict__ counts,
                                                      unsigned long long* __restrict__ depth,
                                                      uint8_t* __restrict__ vis) {
  static_assert(kCullSegs == 2 * kBlock, "two segments a thread");
  __shared__ uint32_t seg0[kCullSegs];  // listed occluders before each segment
  __shared__ uint32_t sh[kBlock / kWave];
  __shared__ double X[3][kVisBatch], Y[3][kVisBatch], Z[3][kVisBatch];
  __shared__ int ix0[kVisBatch], iy0[kVisBatch], nx[kVisBatch];
  __shared__ unsigned long long end[kVisBatch];  // samples of the batch up to and with each
  __shared__ uint32_t seen[kVisBatch];           // 1: covers a sample, 3: ... and passes at one
  __shared__ uint32_t many[kVisBatch];           // samples of a footprint that is walked alone
  __shared__ unsigned long long alone;           // ... and which those are
  const int tid = threadIdx.x, lane = lane_id();
  uint32_t n_occ;
  {
    const int g = 2 * tid;
    const uint32_t a = g < nseg ? counts[g] : 0u, b = g + 1 < nseg ? counts[g + 1] : 0u;
    const uint32_t incl = block_incl_scan<uint32_t>(a + b, sh, &n_occ);
    seg0[g] = incl - b - a;
    seg0[g + 1] = incl - b;
    __syncthreads();
  }
  // one batch a workgroup, smaller ones if that makes more workgroups
  const uint32_t run = n_occ > kVisRun * gridDim.x ? kVisRun : 1;
  const uint32_t batches =
      max((n_occ + kVisBatch - 1) / kVisBatch, min(gridDim.x, (n_occ + run - 1) / run));
  for (uint32_t b = blockIdx.x; b < batches; b += gridDim.x) {
    int32_t t = -1;
    if (tid < kVisBatch) {  // (the first wave)
      unsigned long long n = 0;
      const uint32_t i = run == 1 ? lane * batches + b
                                  : ((lane / kVisRun) * batches + b) * kVisRun + lane % kVisRun;
      if (i < n_occ) {
        int lo = 0, hi = nseg;  // last segment that starts at or before i
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (seg0[mid] <= i) lo = mid; else hi = mid;
        }
        t = occl[segment_base(T, nseg, lo) + (i - seg0[lo])];
        double p[3][3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const int64_t v = idx[3 * (int64_t)t + e];
#pragma unroll
          for (int k = 0; k < 3; ++k) p[e][k] = pos[3 * v + k];
        }
        const double4 c[3] = {clip64(q, p[0]), clip64(q, p[1]), clip64(q, p[2])};
        Shot s;
        shot_of(q, c, s);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          X[e][lane] = s.X[e];
          Y[e][lane] = s.Y[e];
          Z[e][lane] = s.Z[e];
        }
        const int w = max(s.ix1 - s.ix0 + 1, 0);
        ix0[lane] = s.ix0;
        iy0[lane] = s.iy0;
        nx[lane] = w;
        n = (unsigned long long)w * max(s.iy1 - s.iy0 + 1, 0);
      }
      const unsigned long long large = __ballot(n > kVisMany);
      many[lane] = (uint32_t)n;
      end[lane] = wave_incl_scan<unsigned long long>(n > kVisMany ? 0ull : n);
      if (MARK) seen[lane] = 0u;
      if (lane == 0) alone = large;
    }
    __syncthreads();
    const unsigned long long all = end[kVisBatch - 1];
    for (unsigned long long s = tid; s < all; s += kBlock) {
      int o = 0;  // first occluder whose samples end after s
#pragma unroll
      for (int h = kVisBatch / 2; h > 0; h >>= 1)
        if (end[o + h - 1] <= s) o += h;
      if (MARK && seen[o] == 3u) continue;
      const uint32_t k = (uint32_t)(s - (o ? end[o - 1] : 0ull));
      const uint32_t row = k / (uint32_t)nx[o];
      const int px = ix0[o] + (int)(k - row * (uint32_t)nx[o]), py = iy0[o] + (int)row;
      double e[3], area;
      if (!covered(X[0][o], X[1][o], X[2][o], Y[0][o], Y[1][o], Y[2][o], px, py, e, area))
        continue;
      const double z = ((e[0] * Z[0][o] + e[1] * Z[1][o]) + e[2] * Z[2][o]) / area;
      const int64_t pix = (int64_t)py * q.Wc + px;
      if (MARK)
        atomicOr(&seen[o], z <= dval(dload(&depth[pix])) + 1e-6 ? 3u : 1u);
      else
        atomicMin(&depth[pix], dkey(z));
    }
    for (unsigned long long left = alone; left; left &= left - 1) {
      const int o = __ffsll((long long)left) - 1;
      const double X0 = X[0][o], X1 = X[1][o], X2 = X[2][o];
      const double Y0 = Y[0][o], Y1 = Y[1][o], Y2 = Y[2][o];
      const double Z0 = Z[0][o], Z1 = Z[1][o], Z2 = Z[2][o];
      const uint32_t n = many[o], w = (uint32_t)nx[o];
      const int ox = ix0[o], oy = iy0[o];
      for (uint32_t k = tid; k < n; k += kBlock) {
        const uint32_t row = k / w;
        const int px = ox + (int)(k - row * w), py = oy + (int)row;
        double e[3], area;
        if (covered(X0, X1, X2, Y0, Y1, Y2, px, py, e, area)) {
          const double z = ((e[0] * Z0 + e[1] * Z1) + e[2] * Z2) / area;
          const int64_t pix = (int64_t)py * q.Wc + px;
          if (MARK)
            atomicOr(&seen[o], z <= dval(dload(&depth[pix])) + 1e-6 ? 3u : 1u);
          else
            atomicMin(&depth[pix], dkey(z));
        }
        if (MARK && seen[o] == 3u) break;
      }
    }
    __syncthreads();
    if (MARK && t >= 0) vis[t] = seen[lane] != 1u ? 1 : 0;
  }
}

// Temporal reuse classification (Sec. "Temporal Reuse"): 0 not visible now,
// 1 reuse the key frame's shading, 2 shade (newly visible, or some vertex had
// max(|x|, |y|) >= w in the key frame's clip space, float32 as the atlas path
// computes it).
//
// Bound by the dependent loads of the visible triangles (visible byte,
// indices, positions), so every thread issues kReusePer triangles level by
// level. The reused triangles are counted per workgroup; the last one to
// finish adds the sums (stored at device scope and completed before the
// ticket is drawn) and sets the ticket back to 0. One atomic per wave on a
// single counter, which serializes at about 3 ns each, took 102 us on a
// 2.2M-triangle scene and its clearing launch 5; the count per workgroup takes
// 18 us in all, and 12 with indices and positions in 12-byte loads.
constexpr int kReuseBlock = 1024;
constexpr int kReusePer = 4;
constexpr int kReuseGrid = 256;  // workgroups
static_assert(kReuseGrid <= kCountGrid, "the reuse count's sums use Work::partial");

__global__ __launch_bounds__(kReuseBlock) void k_reuse_flags(
    const float* __restrict__ pos, const int32_t* __restrict__ idx, int64_t T, KeyClip kc,
    const uint8_t* __restrict__ key_vis, const uint8_t* __restrict__ vis,
    uint8_t* __restrict__ flags, unsigned long long* __restrict__ reused,
    unsigned long long* __restrict__ partial, unsigned long long* __restrict__ ticket) {
  __shared__ uint32_t sh[kReuseBlock / kWave];
  __shared__ uint32_t last;
  uint32_t count = 0;
  const float3* pos3 = reinterpret_cast<const float3*>(pos);
  const int3* idx3 = reinterpret_cast<const int3*>(idx);
  const int64_t step = (int64_t)gridDim.x * kReuseBlock;
  for (int64_t t0 = (int64_t)blockIdx.x * kReuseBlock + threadIdx.x; t0 < T;
       t0 += kReusePer * step) {
    bool on[kReusePer], key[kReusePer];
    int3 vi[kReusePer];
    float3 q[kReusePer][3];
#pragma unroll
    for (int k = 0; k < kReusePer; ++k) {
      const int64_t t = t0 + k * step;
      on[k] = t < T && vis[t];
      key[k] = t < T && key_vis[t] != 0;
    }
#pragma unroll
    for (int k = 0; k < kReusePer; ++k) {
      vi[k] = make_int3(0, 0, 0);
      if (on[k]) vi[k] = idx3[t0 + k * step];
    }
#pragma unroll
    for (int k = 0; k < kReusePer; ++k) {
      q[k][0] = q[k][1] = q[k][2] = make_float3(0.0f, 0.0f, 0.0f);
      if (on[k]) {
        q[k][0] = pos3[vi[k].x];
        q[k][1] = pos3[vi[k].y];
        q[k][2] = pos3[vi[k].z];
      }
    }
#pragma unroll
    for (int k = 0; k < kReusePer; ++k) {
      const int64_t t = t0 + k * step;
      bool partly = false;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (i == 2) continue;  // z is not needed
          float acc = kc.M[4 * i] * q[k][e].x;
          acc = acc + kc.M[4 * i + 1] * q[k][e].y;
          acc = acc + kc.M[4 * i + 2] * q[k][e].z;
          r[i] = acc + kc.M[4 * i + 3];
        }
        if (fmaxf(fabsf(r[0]), fabsf(r[1])) >= r[3]) partly = true;
      }
      const bool reuse = on[k] && key[k] && !partly;
      count += reuse;
      if (t < T) flags[t] = on[k] ? (reuse ? 1 : 2) : 0;
    }
  }
  if (!reused) return;
  count = block_sum<uint32_t>(count, sh);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&partial[blockIdx.x], (unsigned long long)count, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    last = __hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  // at most 2^30 triangles: the total fits 32 bits
  uint32_t all = 0;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += kReuseBlock)
    all += (uint32_t)__hip_atomic_load(&partial[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  all = block_sum<uint32_t>(all, sh);
  if (threadIdx.x == 0) {
    *reused = all;
    __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

hipError_t launch_reuse_flags(const float* pos, const int32_t* idx, int64_t T, const KeyClip& kc,
                              const uint8_t* key_vis, const uint8_t* vis, uint8_t* flags,
                              unsigned long long* reused, const Work& w, hipStream_t st) {
  // (one workgroup even without triangles: it writes the count)
  const unsigned g = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>((T + kReuseBlock - 1) / kReuseBlock, kReuseGrid));
  k_reuse_flags<<<g, kReuseBlock, 0, st>>>(pos, idx, T, kc, key_vis, vis, flags, reused, w.partial,
                                           w.big_counter + 1);
  return hipGetLastError();
}

hipError_t launch_visibility(const float* pos, const int32_t* idx, int64_t T, const VisParams& q,
                             int32_t* occl, unsigned long long* depth, uint8_t* vis,
                             const Work& w, hipStream_t st) {
  if (T == 0) return hipSuccess;
  const int64_t nd = q.coarse > 0 ? (int64_t)q.Wc * q.Hc : 0;
  uint32_t* counts = reinterpret_cast<uint32_t*>(w.partial);
  const int nseg = cull_segments(T);
  // (a depth buffer of many samples is cleared by more workgroups than few triangles need)
  const int64_t clear = std::min<int64_t>(nd / (8 * kCullBlock), 1024);
  const unsigned g = (unsigned)std::max<int64_t>(nseg, clear);
  k_vis_cull<<<g, kCullBlock, 0, st>>>(pos, idx, T, nseg, q, vis, occl, counts, depth, nd);
  if (q.coarse > 0) {
    const unsigned og =
        (unsigned)std::min<int64_t>(T, kVisGrid);
    k_vis_depth<false><<<og, kBlock, 0, st>>>(pos, idx, T, nseg, q, occl, counts, depth, vis);
    k_vis_depth<true><<<og, kBlock, 0, st>>>(pos, idx, T, nseg, q, occl, counts, depth, vis);
  }
  return hipGetLastError();
}

}  // namespace fa
