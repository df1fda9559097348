// FastAtlas packing on gfx950 (Secs. "Parallel Atlas and Scale Factor
// Computation" and "Box Packing").
//
// One workgroup evaluates one candidate scale j/J:
//   sizes   a = max(m_min, ceil(w * j/J)) + 2g, b likewise for the height;
//   fold    exclusive prefix sum X of the widths (64-bit), row = X >> log2(omega),
//           offset = X & (omega - 1), overflow m = max(offset + a - omega);
//           layout width L = omega + m (the rows are later rescaled by omega/L);
//   mirror  rows with row % 3 != 0 run right to left;
//   push    row by row, a box rises to the top of the frontline under its span
//           and raises that span by its height. The frontline (L <= 2 omega
//           columns) lives in LDS; the boxes of a row have disjoint spans, so
//           each wave takes whole boxes and one barrier per row orders rows.
// A candidate fits iff m <= omega and the layout height H <= L. Selection takes
// the largest effective scale (j/J) * omega / L, compared exactly.
//
// Footprint push (a generalization of the push to non-rectangular charts):
// a box meets the frontline with its footprint profile instead of its full
// height. The profile of content column k (box column k + g) at scale j/J is
// pooled from the chart's full-scale profile: the fine columns whose scaled
// cells touch k give top row T = floor(min top * j / J) and bottom row B =
// floor((max bottom + 1) * j / J) (inclusive), or the box bottom when they
// reach the chart's last row; the gutter then widens it by g columns and
// rows. With top[d] / bottom[d] = min(b - 1, 2g + B) the widened profile of
// box column d:
//   y = max(0, max_d F[x+d] - top[d]),  F[x+d] = y + bottom[d] + 1,
// computed per content column k (its widened window is d in [k, k + 2g]):
// y = max over k of (max F over the window) - T_k, and, since the new
// frontline value only grows, F[x+d] = max over the k covering d of
// min(y + b, y + 2g + B_k + 1), applied with LDS atomic max.
#include <algorithm>
#include <climits>
#include <cstddef>

#include "fa_internal.h"

namespace fa {
namespace {

// Footprint push: candidates of frames with at most kPackLds charts keep
// their prefix sums and sizes in LDS next to the frontline.
constexpr int kPackLds = 4096;

constexpr uint32_t kEmpty = 0xFFFFFFFFu;  // no texel in the box's column
constexpr int kAllCols = 768;  // wider boxes are pushed by the whole workgroup
constexpr int kAllList = 256;  // ... as many of them

// Content column kk (pooled value q) of a box of a columns whose first column
// is F[0]: the height that it needs, and the frontline raised over it by a box
// of b rows at y (its new top).
// (The gutter's columns are read four at a time, and without a branch, so that
// the reads of several columns are in flight together; past the box they read
// its last column.)
__device__ __forceinline__ int rise_of(const int32_t* F, int kk, uint32_t q, int g, int a) {
  const int dend = min(kk + 2 * g, a - 1);
  int fm = 0;
  for (int h = 0; h <= 2 * g; h += 4) {
    const int f0 = F[min(kk + h, dend)], f1 = F[min(kk + h + 1, dend)];
    const int f2 = F[min(kk + h + 2, dend)], f3 = F[min(kk + h + 3, dend)];
    fm = max(fm, max(max(f0, f1), max(f2, f3)));
  }
  return q == kEmpty ? 0 : fm - (int)(q & 0xFFFFu);
}
__device__ __forceinline__ int raise_by(int32_t* F, int kk, uint32_t q, int g, int a, int b,
                                        int y) {
  if (q == kEmpty) return 0;
  const int Bk = (int)(q >> 16);
  const int v = Bk == 0x7FFF ? y + b : min(y + b, y + 2 * g + Bk + 1);
  const int dend = min(kk + 2 * g, a - 1);
  atomicMax(&F[kk], v);
  for (int h = 1; h <= 2 * g; ++h) atomicMax(&F[min(kk + h, dend)], v);
  return v;
}

// Footprint push in three launches: MODE 1 sizes, fold, overflow and row
// starts (to global memory; tab[3] = -1 marks a rejected candidate, tab[5]
// the number of rows with boxes), then k_fp_pool, then MODE 2 the push. (The
// box push is k_pack_box.)
// LDS: at most kPackLds charts (a body of its own, so that the compiler knows
// these accesses for LDS ones: flat loads are waited for together with the
// prefetched pool values).
// The push is bound by the chain of LDS accesses from box to box. Boxes over
// kAllCols columns by the whole workgroup, maxima by DPP, the columns of a
// gutter read together and two (not four) columns a lane prefetched took it
// from 44 to 28 us on a 2.2M-triangle frame (144 charts) and from 58 to 37 on
// one of 86k (234 charts).
template <int NT, int MODE, bool LDS>
__device__ __forceinline__ void pack_body(const float2* __restrict__ wh,
                                          const FrameState* __restrict__ st, const FrameParams& p,
                                          long long* __restrict__ cand_x,
                                          uint32_t* __restrict__ cand_ab,
                                          int32_t* __restrict__ cand_y,
                                          int32_t* __restrict__ cand_rs,
                                          int32_t* __restrict__ cand_tab, int64_t stride,
                                          const uint32_t* __restrict__ fp_pool,
                                          int64_t pool_stride, int32_t* F, long long* sh64,
                                          int32_t* sh32, int32_t* Hsh, int32_t* all_box) {
  constexpr int NW = NT / kWave;
  const int j = blockIdx.x + 1;
  const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
  const int C = st->num_charts;
  const int omega = p.omega, lg = p.log2omega;
  long long* Xg = cand_x + (int64_t)(j - 1) * stride;
  uint32_t* ABg = cand_ab + (int64_t)(j - 1) * stride;
  int32_t* RSg = cand_rs + (int64_t)(j - 1) * (stride + 1);
  long long* X = LDS ? reinterpret_cast<long long*>(F + 2 * omega) : Xg;
  uint32_t* AB = LDS ? reinterpret_cast<uint32_t*>(F + 2 * omega + 2 * kPackLds) : ABg;
  int32_t* RS = (LDS && MODE != 1) ? F + 2 * omega + 3 * kPackLds : RSg;
  int32_t* Y = cand_y + (int64_t)(j - 1) * stride;
  int32_t* tab = cand_tab + (j - 1) * kCandStride;
  long long m, rows;
  int nr;

  if constexpr (MODE != 2) {
    const float s = (float)j / (float)p.J;
    const int pad = 2 * p.gutter;
    // ---- sizes, fold and overflow -----------------------------------------
    long long run = 0, mloc = 0;
    int bad = 0;
    for (int base = 0; base < C; base += NT) {
      const int i = base + tid;
      int a = 0, b = 0;
      if (i < C) {
        const float2 v = wh[i];
        const int wi = (int)ceilf(v.x * s);
        const int hi = (int)ceilf(v.y * s);
        a = max(p.min_box, wi) + pad;
        b = max(p.min_box, hi) + pad;
      }
      long long tot;
      const long long incl = block_incl_scan<long long>((long long)a, sh64, &tot);
      const long long Xi = run + incl - a;
      run += tot;
      if (i < C) {
        Xg[i] = Xi;
        if (a > 2 * omega || b > 2 * omega) bad = 1;  // cannot fit: m > omega or H > L
        const uint32_t ca = (uint32_t)min(a, 2 * omega + 1), cb = (uint32_t)min(b, 2 * omega + 1);
        ABg[i] = ca | (cb << 16);
        if (LDS) {
          X[i] = Xi;
          AB[i] = ca | (cb << 16);
        }
        mloc = max(mloc, (Xi & (long long)(omega - 1)) + a - omega);
      }
    }
    m = block_max<long long>(mloc, sh64);
    bad = block_max<int>(bad, sh32);
    rows = C > 0 ? (X[C - 1] >> lg) + 1 : 0;
    if (m > omega || bad) {
      if (tid == 0) {
        tab[0] = 0;
        tab[1] = (int32_t)min(m, (long long)INT_MAX);
        tab[2] = (int32_t)min(m + omega, (long long)INT_MAX);
        tab[3] = -1;
        tab[4] = (int32_t)min(rows, (long long)INT_MAX);
      }
      return;
    }
    // ---- row starts: first box of every non-empty row, in order ------------
    nr = 0;
    for (int base = 0; base < C; base += NT) {
      const int i = base + tid;
      const int first = (i < C && (i == 0 || (X[i] >> lg) != (X[i - 1] >> lg))) ? 1 : 0;
      int tot;
      const int incl = block_incl_scan<int>(first, sh32, &tot);
      if (first) RS[nr + incl - 1] = i;
      nr += tot;
    }
    if (tid == 0) RS[nr] = C;
    if constexpr (MODE == 1) {
      if (tid == 0) {
        tab[0] = 0;
        tab[1] = (int32_t)m;
        tab[2] = omega + (int)m;
        tab[3] = 0;
        tab[4] = (int32_t)min(rows, (long long)INT_MAX);
        tab[5] = nr;
      }
      return;
    }
  } else {
    if (tab[3] < 0) return;  // rejected by its fold
    m = tab[1];
    rows = tab[4];
    nr = tab[5];
    if (LDS) {
      for (int i = tid; i < C; i += NT) {
        X[i] = Xg[i];
        AB[i] = ABg[i];
      }
      for (int i = tid; i <= nr; i += NT) RS[i] = RSg[i];
    }
  }
  const int L = omega + (int)m;
  for (int c = tid; c < L; c += NT) F[c] = 0;
  if (tid < 2) Hsh[tid] = 0;
  const uint32_t* pool = fp_pool + (int64_t)(j - 1) * pool_stride;
  __syncthreads();

  // ---- push: row by row; the boxes of a row have disjoint spans, so each
  // wave takes whole boxes (a strided read-max, then a strided write) and
  // one barrier per row orders the rows. The height test reads a slot that
  // no wave can touch again before every wave has read it.
  int Hw = 0;
  // boxes of more than kAllCols columns are pushed by the whole workgroup
  // (list of the first kAllList of them, in order)
  int n_all = 0;
  for (int base = 0; base < C && n_all < kAllList; base += NT) {
    const int i = base + tid;
    const int one = i < C && (int)(AB[i] & 0xFFFFu) - p.gutter > kAllCols ? 1 : 0;
    int tot;
    const int at = n_all + block_incl_scan<int>(one, sh32, &tot) - one;
    if (one && at < kAllList) all_box[at] = i;
    n_all += tot;
  }
  n_all = min(n_all, kAllList);
  __syncthreads();
  const int last_all = n_all > 0 ? all_box[n_all - 1] : -1;
  int next_all = 0;
  // footprint push: the pooled values do not depend on the frontline, so each
  // wave loads its next box's first R x 64 columns while it pushes the current
  constexpr int R = 2;
  uint32_t nxt[R];
  int prr = 0, pk = 0;
  auto advance = [&](bool first) {
    if (!first) pk += NW;
    else pk = nr > 0 ? RS[0] + w : 0;
    while (prr < nr && pk >= RS[prr + 1]) {
      ++prr;
      if (prr < nr) pk = RS[prr] + w;
    }
  };
  auto prefetch = [&]() {
    if (prr >= nr) return;
    const uint32_t* src = pool + X[pk];
    const int ncol = (int)(AB[pk] & 0xFFFFu) - p.gutter;
#pragma unroll
    for (int rk = 0; rk < R; ++rk) {
      const int kk = lane + rk * kWave;
      nxt[rk] = kk < ncol ? src[kk] : kEmpty;
    }
  };
  if constexpr (MODE == 2) {
    advance(true);
    prefetch();
  }
  for (int rr = 0; rr < nr; ++rr) {
    const int s0 = RS[rr], s1 = RS[rr + 1];
    const long long r = X[s0] >> lg;
    const bool right = (r % 3) != 0;
    {
      // the row's widest boxes, column by column over the workgroup (the
      // boxes of a row do not touch each other's columns)
      for (; next_all < n_all && all_box[next_all] < s1; ++next_all) {
        const int k = all_box[next_all];
        const uint32_t ab = AB[k];
        const int a = (int)(ab & 0xFFFFu), b = (int)(ab >> 16);
        const int o = (int)(X[k] - (r << lg));
        const int x = right ? L - o - a : o;
        const int g = p.gutter, ncol = a - g;
        const uint32_t* src = pool + X[k];
        int mx = 0;
        for (int k0 = tid; k0 < ncol; k0 += R * NT) {
          uint32_t q[R];
#pragma unroll
          for (int h = 0; h < R; ++h) q[h] = k0 + h * NT < ncol ? src[k0 + h * NT] : kEmpty;
#pragma unroll
          for (int h = 0; h < R; ++h) mx = max(mx, rise_of(F + x, k0 + h * NT, q[h], g, a));
        }
        const int y = block_max<int>(mx, sh32);
        for (int k0 = tid; k0 < ncol; k0 += R * NT) {
          uint32_t q[R];
#pragma unroll
          for (int h = 0; h < R; ++h) q[h] = k0 + h * NT < ncol ? src[k0 + h * NT] : kEmpty;
#pragma unroll
          for (int h = 0; h < R; ++h)
            Hw = max(Hw, raise_by(F + x, k0 + h * NT, q[h], g, a, b, y));
        }
        if (tid == 0) Y[k] = y;
      }
      for (int k = s0 + w; k < s1; k += NW) {
        const long long Xk = X[k];
        const uint32_t ab = AB[k];
        const int a = (int)(ab & 0xFFFFu), b = (int)(ab >> 16);
        const int o = (int)(Xk - (r << lg));
        const int x = right ? L - o - a : o;
        {
          // one lane per content column; the pooled values come from k_fp_pool
          const int g = p.gutter, ncol = a - g;
          const uint32_t* src = pool + Xk;
          uint32_t keep[R];
  #pragma unroll
          for (int rk = 0; rk < R; ++rk) keep[rk] = nxt[rk];
          advance(false);
          prefetch();
          if (ncol > kAllCols && k <= last_all) continue;  // (done above)
          int mx = 0;
#pragma unroll
          for (int rk = 0; rk < R; ++rk)
            mx = max(mx, rise_of(F + x, lane + rk * kWave, keep[rk], g, a));
          for (int k0 = lane + R * kWave; k0 < ncol; k0 += R * kWave) {
            uint32_t q[R];
#pragma unroll
            for (int h = 0; h < R; ++h)
              q[h] = k0 + h * kWave < ncol ? src[k0 + h * kWave] : kEmpty;
#pragma unroll
            for (int h = 0; h < R; ++h)
              mx = max(mx, rise_of(F + x, k0 + h * kWave, q[h], g, a));
          }
          const int y = wave_max_dpp(mx);
#pragma unroll
          for (int rk = 0; rk < R; ++rk)
            Hw = max(Hw, raise_by(F + x, lane + rk * kWave, keep[rk], g, a, b, y));
          for (int k0 = lane + R * kWave; k0 < ncol; k0 += R * kWave) {
            uint32_t q[R];
#pragma unroll
            for (int h = 0; h < R; ++h)
              q[h] = k0 + h * kWave < ncol ? src[k0 + h * kWave] : kEmpty;
#pragma unroll
            for (int h = 0; h < R; ++h)
              Hw = max(Hw, raise_by(F + x, k0 + h * kWave, q[h], g, a, b, y));
          }
          if (lane == 0) Y[k] = y;
        }
      }
    }
    Hw = wave_max_dpp(Hw);  // lane 0 publishes the wave's height
    if (lane == 0) atomicMax(&Hsh[rr & 1], Hw);
    __syncthreads();
    if (Hsh[rr & 1] > L) break;
  }
  if (tid == 0) {
    const int H = nr > 0 ? max(Hsh[0], Hsh[1]) : 0;
    tab[0] = H <= L ? 1 : 0;
    tab[1] = (int32_t)m;
    tab[2] = L;
    tab[3] = H;
    tab[4] = (int32_t)min(rows, (long long)INT_MAX);
  }
}

template <int NT, int MODE>
__global__ __launch_bounds__(NT) void k_pack(const float2* __restrict__ wh,
                                             const FrameState* __restrict__ st, FrameParams p,
                                             long long* __restrict__ cand_x,
                                             uint32_t* __restrict__ cand_ab,
                                             int32_t* __restrict__ cand_y,
                                             int32_t* __restrict__ cand_rs,
                                             int32_t* __restrict__ cand_tab, int64_t stride,
                                             const uint32_t* __restrict__ fp_pool,
                                             int64_t pool_stride) {
  // [2 * omega] frontline, then the LDS copies of X, AB and the row starts
  extern __shared__ int32_t F[];
  __shared__ long long sh64[NT / kWave];
  __shared__ int32_t sh32[NT / kWave];
  __shared__ int32_t Hsh[2];
  __shared__ int32_t all_box[kAllList];
  if (st->status != FA_OK) return;
  if (st->num_charts <= kPackLds)
    pack_body<NT, MODE, true>(wh, st, p, cand_x, cand_ab, cand_y, cand_rs, cand_tab, stride,
                              fp_pool, pool_stride, F, sh64, sh32, Hsh, all_box);
  else
    pack_body<NT, MODE, false>(wh, st, p, cand_x, cand_ab, cand_y, cand_rs, cand_tab, stride,
                               fp_pool, pool_stride, F, sh64, sh32, Hsh, all_box);
}

// Box push of one candidate per workgroup (the default packing). Everything
// the row loop reads is in LDS, so its only global accesses are the stores of
// the box positions, which no later instruction of the workgroup waits for.
// Dynamic LDS, in 32-bit words (box_lds):
//   [kcap]     fold position of each box of the current chunk, relative to
//              the chunk's first box (kcap boxes of at most 2 omega + 1 columns
//              span less than 2^31)
//   [kcap]     a | b << 16 of each box of the chunk
//   [kcap + 4] by rows: the boxes under each box, then its top; by columns:
//              chunk-local starts of the chunk's row segments
//   by rows: the frontline's edge columns, the tables of shared boxes, the
//   cells (16 bits: box at every 2^g-th fold position) and the row starts (16
//   bits); by columns: the whole frontline, then the lists of mid and wide
//   boxes.
// Frames with more than kcap charts are pushed in chunks, reloaded from the
// fold written to global memory. Cross-lane maxima and scans use DPP lane
// moves.
//
// By rows (push_rows). A row's boxes follow each other without holes, so all
// columns but the at most m on either side of it are covered by the row
// before, and what a box rises to is the highest top among the few boxes of
// that row under it. Those are found for all boxes of a chunk at once, before
// the push; a row then costs two dependent LDS accesses and one barrier,
// however wide its boxes are. Only the m edge columns on each side, which a
// row may leave to an older one, keep a frontline value each. Reading and
// raising every column of every box (push_columns) took about 2.4 us a row of
// 4096 columns: 273 us for 23.7k charts and 64 us for 3000 boxes of 33
// columns; by rows, at about 1 us a row, they take 179 and 34 us.
// By columns: candidates with a wide overflow m (a few boxes nearly as wide as
// the atlas), where the edges are most of the frontline, rows so long that two
// of them do not fit a chunk, frames of up to kFewBoxes charts, whose few
// columns walks take less than finding what lies under each box (one chart:
// 7.6 us by columns, 8.5 by rows), and candidates whose boxes are narrow or lie
// many to an edge (columns_cheaper).
constexpr int kFoldItems = 4;   // consecutive boxes per thread in the fold
constexpr int kNarrow = 8;      // by columns: boxes up to this wide are pushed by one lane
constexpr int kMidList = 2048, kWideList = 256;  // by columns: entries of the box lists
// (9 to 16 boxes take 0.5 to 1 us less by columns too, which columns_cheaper finds)
constexpr int kFewBoxes = 8;
// By rows: most edge columns on either side. With half as many, 1000 boxes with
// an overflow of 642 columns take 73 us in place of 50, 4000 with one of 532 125
// in place of 98; with twice as many nothing is faster and 200 boxes with one of
// 1142 take 39 in place of 35.
constexpr int kEdgeMax = 1024;
constexpr int kUnderLane = 8;   // by rows: boxes under a box that one lane looks at
// By rows: the mark of a box that 16 lanes push together, in its a | b << 16
// (a and b are below 2^15), which the push leaves as it is.
constexpr uint32_t kShared16 = 1u << 31;

constexpr int kCellBits = 12;   // by rows: 2^12 cells index a chunk's fold positions
constexpr int kCells = 1 << kCellBits;
// By rows: rows of a chunk with a table of their shared boxes, and boxes in it
// (32 rows: 16000 boxes in 110 rows 176 -> 186 us; 4 boxes: 60000 boxes in 156
// rows 373 -> 413; 16 boxes do not fit the LDS at 4096 columns).
constexpr int kTabRows = 128;
constexpr int kTabBoxes = 8;

// Boxes per chunk by columns (by rows: the multiples of it end a segment too,
// so that both stop at the same box) and by rows, and the dynamic LDS of a
// push.
__host__ __device__ inline int box_kcap(int omega) {
  return ((131072 - 8 * omega - 4) / 12) & ~63;
}
__host__ __device__ inline int row_kcap(int omega) {
  return box_kcap(omega) < 8128 ? box_kcap(omega) : 8128;
}
__host__ inline size_t box_lds(int omega) {
  const size_t kc = (size_t)box_kcap(omega), kr = (size_t)row_kcap(omega);
  const size_t rows = 4 * kc + 8 * kr + 16 + 8 * (size_t)std::min(omega, kEdgeMax) +
                      (16 * kTabBoxes + 4) * kTabRows + 2 * (kCells + 8) + 2 * (kr + 2);
  const size_t columns = 12 * kc + 16 + 8 * (size_t)omega + 4 * (kMidList + kWideList);
  return (std::max(rows, columns) + 15) & ~size_t(15);
}
// ... at any atlas side
__host__ inline size_t box_lds_max() {
  size_t most = 0;
  for (int om = 16; om <= kMaxAtlas; om *= 2) most = std::max(most, box_lds(om));
  return most;
}

// What both pushes work on.
struct PushArgs {
  const long long* Xg;     // the candidate's fold in global memory
  const uint32_t* ABg;
  int32_t* Y;              // positions out
  int C, omega, lg, m, kcap;
};

// Whether the push by columns takes less, from what both depend on, in ns: by
// rows a row, a box and a box over edge columns (about m C / omega of them a row
// and side; they are pushed by 16 lanes each and, above kTabBoxes a row, looked
// up one by one); by columns a column, a row and a box of at most kNarrow, at
// most 64 and more columns. Fitted to 810 sets of 9 to 60000 boxes in one
// candidate each, alike and with a share of boxes 3 to 30 times as large, at
// atlases of 512 to 8192 and every block size (1.03 and 500: rows where the two
// are level); within 4 us or 15% of the faster way for all but 11 of them. Boxes
// of 4 to 6 columns with a few of 130 took 538, 450 and 206 us by rows (261, 269
// and 145 by columns), most sets of wider boxes 1.3 to 2 times as long by columns
// as by rows; 64 candidates of 60000 such boxes 475 us by rows, 311 so.
template <int NT>
__device__ __forceinline__ bool columns_cheaper(const PushArgs& q, float rows, float narrow,
                                                float wide) {
  constexpr int k = NT == 1024 ? 0 : NT == 512 ? 1 : 2;
  constexpr float kStart[3] = {2540.f, 2100.f, 2150.f}, kRow[3] = {972.f, 850.f, 766.f};
  constexpr float kBox[3] = {2.0f, 2.95f, 5.8f}, kBoxColumn[3] = {2.4e-4f, 2.6e-4f, 3.5e-4f};
  constexpr float kEdge[3] = {100.f, 114.f, 127.f};
  constexpr float kColumn[3] = {0.35f, 0.43f, 0.70f}, kColumnRow[3] = {1341.f, 1250.f, 1106.f};
  constexpr float kUpTo8[3] = {2.24f, 2.7f, 4.6f}, kUpTo64[3] = {8.6f, 13.2f, 27.f};
  constexpr float kAbove64[3] = {30.f, 53.f, 101.f};
  const float boxes = (float)q.C, omega = (float)q.omega;
  const float by_rows = kStart[k] + kRow[k] * rows + (kBox[k] + kBoxColumn[k] * omega) * boxes +
                        kEdge[k] * (float)q.m * boxes / omega;
  const float by_columns = kColumn[k] * omega + kColumnRow[k] * rows + kUpTo8[k] * narrow +
                           kUpTo64[k] * (boxes - narrow - wide) + kAbove64[k] * wide;
  return 1.03f * by_columns + 500.f < by_rows;
}

// The next chunk [c0, c0 + cn) from the fold in global memory.
template <int NT>
__device__ __forceinline__ long long load_chunk(const PushArgs& q, int c0, int cn, uint32_t* Xr,
                                                uint32_t* AB) {
  const long long xbase = q.Xg[c0];
  constexpr int U = 4;  // loads in flight per thread
  for (int i0 = threadIdx.x; i0 < cn; i0 += U * NT) {
    long long xv[U];
    uint32_t abv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT;
      xv[u] = i < cn ? q.Xg[c0 + i] : 0;
      abv[u] = i < cn ? q.ABg[c0 + i] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT;
      if (i < cn) {
        Xr[i] = (uint32_t)(xv[u] - xbase);
        AB[i] = abv[u];
      }
    }
  }
  __syncthreads();
  return xbase;
}

// First box of every row among the cn boxes of a chunk, in order, into RS
// (ROW_OF: also each box's number of rows started up to it, less one, into
// row_of). Returns the number of rows; ends before a barrier.
template <int NT, bool ROW_OF, typename R>
__device__ __forceinline__ int row_starts(const PushArgs& q, long long xbase, int cn,
                                          const uint32_t* Xr, R* RS, uint32_t* row_of,
                                          uint32_t (*shs)[NT / kWave], int& pass) {
  int nr = 0;
  for (int base = 0; base < cn; base += kFoldItems * NT, ++pass) {
    const int i0 = base + kFoldItems * threadIdx.x;
    uint32_t fl = 0, own = 0;
    if (i0 < cn) {
      const uint4 v = *reinterpret_cast<const uint4*>(Xr + i0);
      const uint32_t xv[kFoldItems + 1] = {i0 > 0 ? Xr[i0 - 1] : 0u, v.x, v.y, v.z, v.w};
#pragma unroll
      for (int u = 0; u < kFoldItems; ++u) {
        const int i = i0 + u;
        const bool f = i < cn && (i == 0 || ((xbase + xv[u + 1]) >> q.lg) !=
                                                ((xbase + xv[u]) >> q.lg));
        fl |= (uint32_t)f << u;
        own += f;
      }
    }
    uint32_t tot;
    int at = nr + (int)(block_incl_scan_dpp<NT>(own, shs[pass & 1], &tot) - own);
#pragma unroll
    for (int u = 0; u < kFoldItems; ++u) {
      if (fl >> u & 1u) RS[at++] = (R)(i0 + u);
      if (ROW_OF && i0 + u < cn) row_of[i0 + u] = (uint32_t)(at - 1);
    }
    nr += (int)tot;
  }
  return nr;
}

// A row in a chunk: its base (fold position of column 0, relative to the
// chunk) and whether it runs right to left.
struct Row {
  int base;
  bool right;
};
__device__ __forceinline__ Row row_at(const PushArgs& q, long long xbase, uint32_t x) {
  const long long r = (xbase + x) >> q.lg;
  return Row{(int)((r << q.lg) - xbase), (uint32_t)r % 3u != 0u};
}

// A zero that the compiler takes to differ between lanes: a uniform LDS word
// loaded at an index with it added stays in a vector register until its own
// readfirstlane, instead of being waited for at once.
__device__ __forceinline__ int lane_zero() {
  int z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  return z;
}

// The edge value of column u counted from a row's start is E[base + step u],
// with the base of the row's own low (u < m) or high (u >= omega) side.
__device__ __forceinline__ int edge_step(bool right) { return right ? -1 : 1; }
__device__ __forceinline__ int edge_low(const PushArgs& q, bool right) {
  return right ? 2 * q.m - 1 : 0;
}
__device__ __forceinline__ int edge_high(const PushArgs& q, bool right) {
  return right ? q.omega + q.m - 1 : q.m - q.omega;
}

// What the push of a shared box needs: the box and its height, the boxes under
// it, and the edge words under it on either side (first and count each, the
// height or count in the upper half).
__device__ __forceinline__ uint4 shared_box(const PushArgs& q, int k, uint32_t ab, int first, int n,
                                            int u, bool right, int pf, int pe) {
  const int a = (int)(ab & 0xFFFFu), step = edge_step(right);
  const int l1 = min(u + a, pf), h0 = max(u, pe);  // columns [u, l1) and [h0, u + a)
  const int nl = max(l1 - u, 0), nh = max(u + a - h0, 0);
  const int l = edge_low(q, right) + step * (right ? l1 - 1 : u);
  const int h = edge_high(q, right) + step * (right ? u + a - 1 : h0);
  return make_uint4((uint32_t)k | (ab & 0xFFFF0000u), (uint32_t)first | ((uint32_t)n << 16),
                    nl ? (uint32_t)l | ((uint32_t)nl << 16) : 0u,
                    nh ? (uint32_t)h | ((uint32_t)nh << 16) : 0u);
}

// Push a shared box by the 16 lanes of a row of the wave (sl: the lane's place
// among them); v: its words, wanted or not. Returns the box's top in every
// lane; every lane of the wave calls it.
__device__ __forceinline__ int push_shared(const uint4 v, bool wanted, int sl, const uint32_t* PT,
                                           const int32_t* E) {
  const uint32_t vy = wanted ? v.y : 0u, vz = wanted ? v.z : 0u, vw = wanted ? v.w : 0u;
  const int first = (int)(vy & 0xFFFFu), n = (int)(vy >> 16);
  const int l = (int)(vz & 0xFFFFu), nl = (int)(vz >> 16);
  const int h = (int)(vw & 0xFFFFu), nh = (int)(vw >> 16);
  // the first 16 boxes and 32 columns of either edge load together (a word
  // that is not wanted reads another)
  const int v0 = (int)PT[first + min(sl, max(n - 1, 0))];
  const int v1 = E[l + min(sl, max(nl - 1, 0))], v2 = E[l + min(sl + 16, max(nl - 1, 0))];
  const int v3 = E[h + min(sl, max(nh - 1, 0))], v4 = E[h + min(sl + 16, max(nh - 1, 0))];
  int y = n ? v0 : 0;
  y = max(y, nl ? max(v1, v2) : 0);
  y = max(y, nh ? max(v3, v4) : 0);
  if (__ballot(n > 16 || nl > 32 || nh > 32)) {
    for (int i = sl + 16; i < n; i += 16) y = max(y, (int)PT[first + i]);
    for (int i = sl + 32; i < nl; i += 16) y = max(y, E[l + i]);
    for (int i = sl + 32; i < nh; i += 16) y = max(y, E[h + i]);
  }
  return row16_max(y);
}

// cell[c]: the box of the chunk that holds fold position c << g (boxes follow
// each other without holes from position 0); returns g, the least with the
// whole chunk in kCells cells and in one to four cells a box. The entry past
// the last position's holds the last box. Ends before a barrier.
template <int NT>
__device__ __forceinline__ int fill_cells(int cn, const uint32_t* Xr, const uint32_t* AB,
                                          uint16_t* cell) {
  const int span = (int)Xr[cn - 1] + (int)(AB[cn - 1] & 0xFFFFu);
  // (cells a power of two: the span's bit length less the cells')
  const int bits = min(kCellBits, 33 - __clz(cn));
  const int g = max(0, 32 - __clz(span - 1) - bits);
  const int last = (span - 1) >> g;
  const int lane = lane_id();
  for (int ib = (int)(threadIdx.x & ~(kWave - 1)); ib < cn; ib += NT) {
    const int i = ib + lane;
    int c = 0, e = 0;  // cells [c, e) start inside box i
    if (i < cn) {
      const int x = (int)Xr[i];
      c = (x + (1 << g) - 1) >> g;
      e = i == cn - 1 ? last + 2 : (x + (int)(AB[i] & 0xFFFFu) + (1 << g) - 1) >> g;
    }
    const bool wide = e - c > 8;
    if (!wide)
      for (; c < e; ++c) cell[c] = (uint16_t)i;
    for (unsigned long long todo = __ballot(wide); todo; todo &= todo - 1) {
      const int l = __ffsll((long long)todo) - 1;
      const int c0 = __builtin_amdgcn_readlane(c, l), c1 = __builtin_amdgcn_readlane(e, l);
      for (int k = c0 + lane; k < c1; k += kWave) cell[k] = (uint16_t)(ib + l);
    }
  }
  return g;
}

// The boxes of the row before under each box of a chunk, into PT: first |
// count << 14; kShared16 in AB where they are more than kUnderLane or some
// columns are the edge's. On entry PT holds each box's row. A box under an end of the
// span is looked up through its cell: a search over the boxes of that cell
// (one or two steps; over the whole row, eight). The shared boxes of the first
// kTabRows rows also go to their row's table, with all that their push needs
// (tab_n counts them, past kTabBoxes too).
template <int NT>
__device__ __forceinline__ void boxes_under(const PushArgs& q, long long xbase, int c0, int cn,
                                            const uint32_t* Xr, uint32_t* AB, const uint16_t* RS,
                                            const uint16_t* cell, int g, uint32_t* PT, uint4* tab, uint32_t* tab_n) {
  const int L = q.omega + q.m;
  for (int i = threadIdx.x; i < cn; i += NT) {
    const int ri = (int)PT[i];
    const uint32_t ab = AB[i];
    if (ri == 0) {
      // the first row of the frame rests on nothing; that of a later chunk is
      // pushed already: its top
      PT[i] = c0 > 0 ? (uint32_t)q.Y[c0 + i] + (ab >> 16) : 0u;
      continue;
    }
    const int rs = RS[ri], ps = RS[ri - 1];
    const int a = (int)(ab & 0xFFFFu), x = (int)Xr[i], xr = (int)Xr[rs], xp = (int)Xr[ps];
    const Row cur = row_at(q, xbase, xr), prv = row_at(q, xbase, xp);
    const int o = x - cur.base;
    const int u = cur.right != prv.right ? L - o - a : o;  // from the start of the row before
    const int b0 = prv.base + u, b1 = b0 + a;              // ... as fold positions
    // the boxes that hold the first and the last position in that row
    const int p0 = min(max(b0, xp), xr - 1), p1 = min(max(b1 - 1, xp), xr - 1);
    int lo = cell[p0 >> g], hi = cell[(p0 >> g) + 1];
    int lo2 = cell[p1 >> g], hi2 = cell[(p1 >> g) + 1];
    while (lo < hi || lo2 < hi2) {
      const int mid = (lo + hi + 1) >> 1, mid2 = (lo2 + hi2 + 1) >> 1;
      const int v = (int)Xr[mid], v2 = (int)Xr[mid2];
      if (lo < hi) {
        if (v <= p0) lo = mid;
        else hi = mid - 1;
      }
      if (lo2 < hi2) {
        if (v2 <= p1) lo2 = mid2;
        else hi2 = mid2 - 1;
      }
    }
    const bool none = b0 >= xr || b1 <= xp;  // all of it over edge columns
    const int n = none ? 0 : lo2 - lo + 1;
    const bool shared = n > kUnderLane || b0 < xp || b1 > xr;
    PT[i] = (uint32_t)lo | ((uint32_t)n << 14);
    if (shared) AB[i] = ab | kShared16;
    if (shared && ri < kTabRows) {
      const uint32_t slot = atomicAdd(&tab_n[ri], 1u);
      if (slot < kTabBoxes)
        tab[ri * kTabBoxes + slot] = shared_box(q, i, ab, lo, n, u, prv.right, xp - prv.base,
                                                xr - prv.base);
    }
  }
}

// Push by rows; over[0] receives the height. The push stops one segment after
// the first one whose top lies above L, a segment being a row or, where a
// multiple of kcap boxes falls inside it, its part on either side.
//
// A segment is one step between two barriers, bound by the latency of its
// instructions, so its parts run in different waves: half of them push the
// plain boxes, one a lane; a quarter the shared ones, 16 lanes each; the last
// quarter stores the tops of the row before in its edge columns. Everything of
// a step that the step before cannot change (the boxes' words, row bounds) is
// loaded before the barrier.
template <int NT>
__device__ __forceinline__ void push_rows(const PushArgs& q, int32_t* S, int& pass,
                                          uint32_t (*shs)[NT / kWave], int32_t* over) {
  int Hw = 0;  // the thread's highest top
  constexpr int NW = NT / kWave;
  constexpr int NP = NW / 2, NS = NW / 4, NE = NW - NP - NS;  // plain, shared, edge waves
  static_assert(NW % 4 == 0, "every part has a wave");
  const int kr = row_kcap(q.omega);
  uint32_t* Xr = reinterpret_cast<uint32_t*>(S);
  uint32_t* AB = Xr + q.kcap;  // (where the fold put the first chunk)
  uint32_t* PT = AB + kr;
  int32_t* E = reinterpret_cast<int32_t*>(PT + kr + 4);  // [m] left, [m] right edge columns
  uint4* tab = reinterpret_cast<uint4*>(E + 2 * min(q.omega, kEdgeMax));
  uint32_t* tab_n = reinterpret_cast<uint32_t*>(tab + kTabRows * kTabBoxes);
  uint16_t* cell = reinterpret_cast<uint16_t*>(tab_n + kTabRows);
  uint16_t* RS = cell + kCells + 8;
  const int tid = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int sub = lane >> 4, sl = lane & 15;
  const int m = q.m, L = q.omega + m, C = q.C;
  const int zero = lane_zero();
  for (int c = tid; c < 2 * m; c += NT) E[c] = 0;
  if (tid < 3) over[tid] = 0;

  int o_prev = 2, o_cur = 0;  // slots of `over`: the segment before, this one
  int rbegin = 0;             // rows at the chunk's start that are pushed already
  long long xbase = 0;
  for (int c0 = 0;;) {
    const int cn = min(kr, C - c0);
    if (c0 > 0) xbase = load_chunk<NT>(q, c0, cn, Xr, AB);
    const int g = fill_cells<NT>(cn, Xr, AB, cell);
    if (tid < kTabRows) tab_n[tid] = 0u;
    const int nr = row_starts<NT, true>(q, xbase, cn, Xr, RS, PT, shs, pass);
    if (tid < 2) RS[nr + tid] = (uint16_t)cn;
    __syncthreads();
    boxes_under<NT>(q, xbase, c0, cn, Xr, AB, RS, cell, g, PT, tab, tab_n);
    __syncthreads();

    // ---- push (a row that the chunk cuts waits for the next chunk)
    const int full = c0 + cn == C ? nr : nr - 1;
    int ri = rbegin;
    int s0 = RS[ri], s1 = RS[ri + 1];
    int ps = ri > 0 ? (int)RS[ri - 1] : 0;
    uint32_t x0 = Xr[s0];
    Row cur = row_at(q, xbase, x0), prv = row_at(q, xbase, Xr[ps]);
    int pf = (int)Xr[ps] - prv.base, pe = (int)x0 - prv.base;
    int cut = ((c0 + s0) / q.kcap + 1) * q.kcap - c0;  // the next multiple of kcap
    int e0 = s0;
    bool stop = false;
    // this lane's first box of the segment (plain waves), the 16 lanes' first
    // table entry of the row (shared waves)
    const int at = w * kWave + lane, slot0 = 4 * (w - NP) + sub;
    const bool tabled = w >= NP && w < NP + NS && slot0 < kTabBoxes;
    uint32_t pt_nxt = 0u, ab_nxt = 0u, n_nxt = 0u;
    uint4 t_nxt = make_uint4(0u, 0u, 0u, 0u);
    if (w < NP) {
      pt_nxt = PT[min(e0 + at, cn - 1)];
      ab_nxt = AB[min(e0 + at, cn - 1)];
    } else if (w < NP + NS) {
      n_nxt = tab_n[min(ri, kTabRows - 1) + zero];
      if (tabled) t_nxt = tab[min(ri, kTabRows - 1) * kTabBoxes + slot0];
    }
    while (ri < full) {
      const int e1 = min(s1, cut);
      const int32_t was_over = over[o_prev + zero];
      const int rs2_v = RS[ri + 2 + zero];
      const uint32_t x1_v = Xr[min(s1, cn - 1) + zero];
      bool above = false;

      if (w < NP) {
        // plain boxes (the next segment starts at e1)
        const uint32_t pt_seg = PT[min(e1 + at, cn - 1)], ab_seg = AB[min(e1 + at, cn - 1)];
        for (int k0 = e0 + w * kWave; k0 < e1; k0 += NP * kWave) {
          const int k = k0 + lane;
          const bool mine = k < e1 && !(ab_nxt & kShared16);
          const uint32_t pt = mine ? pt_nxt : 0u;
          const int b = (int)(ab_nxt >> 16);
          if (k0 + NP * kWave < e1) {
            pt_nxt = PT[min(k + NP * kWave, cn - 1)];
            ab_nxt = AB[min(k + NP * kWave, cn - 1)];
          }
          const int first = (int)(pt & 0x3FFFu), n = (int)(pt >> 14);
          int v[kUnderLane / 2];
#pragma unroll
          for (int u = 0; u < kUnderLane / 2; ++u) v[u] = (int)PT[first + max(0, min(u, n - 1))];
          int y = max(max(v[0], v[1]), max(v[2], v[3]));
          if (__ballot(n > kUnderLane / 2)) {
#pragma unroll
            for (int u = 0; u < kUnderLane / 2; ++u)
              v[u] = (int)PT[first + max(0, min(u + kUnderLane / 2, n - 1))];
            y = max(y, max(max(v[0], v[1]), max(v[2], v[3])));
          }
          if (n == 0) y = 0;
          if (mine) {
            PT[k] = (uint32_t)(y + b);
            q.Y[c0 + k] = y;
            Hw = max(Hw, y + b);
            above = above || y + b > L;
          }
        }
        pt_nxt = pt_seg;
        ab_nxt = ab_seg;
      } else if (w < NP + NS) {
        // shared boxes: 16 lanes each, four at a time
        const int rn = min(e1 == s1 ? ri + 1 : ri, kTabRows - 1);
        const uint32_t n_seg = tab_n[rn + zero];
        uint4 t_seg = make_uint4(0u, 0u, 0u, 0u);
        if (tabled) t_seg = tab[rn * kTabBoxes + slot0];
        auto put = [&](int k, int b, int y, bool wanted) {
          if (wanted && sl == 0) {
            PT[k] = (uint32_t)(y + b);
            q.Y[c0 + k] = y;
            Hw = max(Hw, y + b);
            above = above || y + b > L;
          }
        };
        const int ns = __builtin_amdgcn_readfirstlane((int)n_nxt);
        if (ri < kTabRows && ns <= kTabBoxes) {
          // from the row's table, 4 NS entries at a time
          for (int t0 = 4 * (w - NP); t0 < ns; t0 += 4 * NS) {
            if (t0 != 4 * (w - NP)) t_nxt = tab[ri * kTabBoxes + min(t0 + sub, kTabBoxes - 1)];
            const int k = (int)(t_nxt.x & 0xFFFFu);
            const bool wanted = t0 + sub < ns && k >= e0 && k < e1;
            put(k, (int)(t_nxt.x >> 16), push_shared(t_nxt, wanted, sl, PT, E), wanted);
          }
        } else {
          // found among the row's boxes
          for (int k0 = e0 + (w - NP) * kWave; k0 < e1; k0 += NS * kWave) {
            const int ko = k0 + lane;
            unsigned long long todo = __ballot(ko < e1 && (AB[min(ko, cn - 1)] & kShared16));
            while (todo) {
              int src = -1;
#pragma unroll
              for (int g4 = 0; g4 < 4; ++g4) {
                if (todo) {
                  const int l = __ffsll((long long)todo) - 1;
                  todo &= todo - 1;
                  if (sub == g4) src = l;
                }
              }
              const int k = k0 + max(src, 0);
              const uint32_t pt = PT[k], ab = AB[k] & ~kShared16;
              const int a = (int)(ab & 0xFFFFu), o = (int)Xr[k] - cur.base;
              const int u = cur.right != prv.right ? L - o - a : o;
              const uint4 v = shared_box(q, k, ab, (int)(pt & 0x3FFFu), (int)(pt >> 14), u,
                                         prv.right, pf, pe);
              put(k, (int)(ab >> 16), push_shared(v, src >= 0, sl, PT, E), src >= 0);
            }
          }
        }
        n_nxt = n_seg;
        t_nxt = t_seg;
      } else if (e0 == s0 && ri > 0) {
        // the tops of the row before into its edge columns (boxes read only
        // the columns it left): the even waves on the low side, the odd ones
        // (or the same one) on the high side, four boxes at a time
        const int we = w - NP - NS;
        constexpr int NH = NE > 1 ? NE / 2 : 1;  // waves per side
        const int p_step = edge_step(prv.right);
        const int p_low = edge_low(q, prv.right), p_high = edge_high(q, prv.right);
        if (NE == 1 || we % 2 == 0) {
          for (int kb = ps + 4 * (we / 2); kb < s0; kb += 4 * NH) {
            const int k = min(kb + sub, s0 - 1);
            const uint32_t ab = AB[k], x = Xr[k];
            const int top = (int)PT[k];
            const int o = (int)x - prv.base;
            if (!__ballot(o < m)) break;
            const int e = min(o + (int)(ab & 0xFFFFu), m);
            for (int c = o + sl; c < e; c += 16) E[p_low + p_step * c] = top;
            if (__ballot(e == m)) break;  // the boxes after it start past the edge
          }
        }
        if (NE == 1 || we % 2 == 1) {
          for (int kb = s0 - 1 - 4 * (we / 2); kb >= ps; kb -= 4 * NH) {
            const int k = max(kb - sub, ps);
            const uint32_t ab = AB[k], x = Xr[k];
            const int top = (int)PT[k];
            const int o = (int)x - prv.base, e = o + (int)(ab & 0xFFFFu);
            if (!__ballot(e > q.omega)) break;
            for (int c = max(o, q.omega) + sl; c < e; c += 16) E[p_high + p_step * c] = top;
            if (__ballot(o <= q.omega)) break;  // the boxes before it end before the edge
          }
        }
      }
      if (above) over[o_cur] = 1;
      const uint32_t x1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)x1_v);
      const int s2 = __builtin_amdgcn_readfirstlane(rs2_v);
      const Row nxt = row_at(q, xbase, x1);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(was_over)) {
        stop = true;
        break;
      }
      o_prev = o_cur;
      o_cur = o_cur == 2 ? 0 : o_cur + 1;
      if (e1 == cut) cut += q.kcap;
      e0 = e1;
      if (e1 == s1) {
        ++ri;
        ps = s0;
        prv = cur;
        pf = (int)x0 - prv.base;
        pe = (int)x1 - prv.base;
        s0 = s1;
        s1 = s2;
        x0 = x1;
        cur = nxt;
      }
    }
    if (stop || c0 + cn == C) break;
    // the next chunk starts with the last row pushed
    c0 += ps;
    rbegin = 1;
    __syncthreads();  // (every thread has read its words of this chunk)
  }
  // the height in over[0] (which every thread has read)
  if (tid < 3) over[tid] = 0;
  __syncthreads();
  const int hw = wave_max_dpp(Hw);
  if (lane == 0) atomicMax(&over[0], hw);
  __syncthreads();
}

// The start of a push by columns (the frontline at its widest).
template <int NT>
__device__ __forceinline__ void columns_clear(int omega, int32_t* F, int32_t* Hsh,
                                              int32_t (*LC)[2]) {
  const int tid = threadIdx.x;
  for (int c = tid; c < 2 * omega; c += NT) F[c] = 0;
  if (tid < 3) Hsh[tid] = 0;
  if (tid < 4) LC[tid >> 1][tid & 1] = 0;
}

// Push by columns: the boxes of a chunk segment by segment in two phases. A:
// the threads take the segment's boxes in order; a box at most kNarrow columns
// wide is pushed by its own lane, the others go to a list of mid boxes (up to
// 64 columns) or of wide ones. B (after a barrier): the mid boxes four per
// wave step, 16 lanes each; the wide boxes one per wave. Boxes of a row have
// disjoint spans, so the order inside a segment changes nothing. A row that
// straddles two chunks is pushed as two segments. Bounds of the lists: a row's
// boxes lie in L <= 2 omega <= 16384 columns, so at most 1820 are wider than 8
// and 252 wider than 64.
template <int NT>
__device__ __forceinline__ void push_columns(const PushArgs& q, int32_t* S, int& pass,
                                             uint32_t (*shs)[NT / kWave], int32_t* Hsh,
                                             int32_t (*LC)[2]) {
  constexpr int NW = NT / kWave;
  uint32_t* Xr = reinterpret_cast<uint32_t*>(S);
  uint32_t* AB = Xr + q.kcap;
  int32_t* RS = reinterpret_cast<int32_t*>(AB + q.kcap);
  int32_t* F = RS + q.kcap + 4;
  int32_t* WM = F + 2 * q.omega;
  int32_t* WW = WM + kMidList;
  const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
  const int sub = lane >> 4, sl = lane & 15;
  const int L = q.omega + q.m, C = q.C;
  if (C > kFewBoxes) {  // (cleared beside the fold otherwise)
    columns_clear<NT>(q.omega, F, Hsh, LC);
    __syncthreads();
  }

  int seg = 0, Hw = 0;
  bool over = false;
  for (int c0 = 0; c0 < C && !over; c0 += q.kcap) {
    const int cn = min(q.kcap, C - c0);
    long long xbase = 0;
    if (c0 > 0) xbase = load_chunk<NT>(q, c0, cn, Xr, AB);
    const int nr = row_starts<NT, false>(q, xbase, cn, Xr, RS, nullptr, shs, pass);
    if (tid == 0) RS[nr] = cn;
    __syncthreads();

    int s0 = 0, s1 = nr > 0 ? RS[1] : 0;
    Row row = row_at(q, xbase, Xr[0]);
    for (int rr = 0; rr < nr; ++rr, ++seg) {
      // next segment: its end and its row
      const int s1n = rr + 2 <= nr ? RS[rr + 2] : cn;
      const uint32_t xfirst = rr + 1 < nr ? Xr[s1] : 0u;
      const int hprev = Hsh[(seg + 2) % 3];  // the height after segment seg - 1
      int* cnt = LC[seg & 1];
      for (int k = s0 + tid; k < s1; k += NT) {
        const uint32_t ab = AB[k];
        const int a = (int)(ab & 0xFFFFu), b = (int)(ab >> 16);
        const int o = (int)Xr[k] - row.base;
        const int x = row.right ? L - o - a : o;
        const bool narrow = a <= kNarrow;
        if (narrow) {
          int v[kNarrow];
#pragma unroll
          for (int c = 0; c < kNarrow; ++c) v[c] = c < a ? F[x + c] : 0;
          int mx = 0;
#pragma unroll
          for (int c = 0; c < kNarrow; ++c) mx = max(mx, v[c]);
#pragma unroll
          for (int c = 0; c < kNarrow; ++c)
            if (c < a) F[x + c] = mx + b;
          q.Y[c0 + k] = mx;
          Hw = max(Hw, mx + b);
        }
        const bool wide = a > kWave;
        const unsigned long long mm = __ballot(!narrow && !wide), mw = __ballot(wide);
        const unsigned long long below = lanes_below();
        int bm = 0, bw = 0;
        if (lane == __ffsll((long long)__ballot(true)) - 1) {
          if (mm) bm = atomicAdd(&cnt[0], __popcll(mm));
          if (mw) bw = atomicAdd(&cnt[1], __popcll(mw));
        }
        bm = __builtin_amdgcn_readfirstlane(bm);
        bw = __builtin_amdgcn_readfirstlane(bw);
        if (!narrow && !wide) WM[bm + __popcll(mm & below)] = k;
        if (wide) WW[bw + __popcll(mw & below)] = k;
      }
      __syncthreads();
      const int nm = cnt[0], nwd = cnt[1];
      if (tid == 0) {
        LC[(seg + 1) & 1][0] = 0;
        LC[(seg + 1) & 1][1] = 0;
      }
      for (int e0 = 4 * w; e0 < nm; e0 += 4 * NW) {
        const int e = e0 + sub;
        int a = 0, b = 0, x = 0, k = 0;
        if (e < nm) {
          k = WM[e];
          const uint32_t ab = AB[k];
          a = (int)(ab & 0xFFFFu);
          b = (int)(ab >> 16);
          const int o = (int)Xr[k] - row.base;
          x = row.right ? L - o - a : o;
        }
        int mx = 0;
        for (int c = x + sl; c < x + a; c += 16) mx = max(mx, F[c]);
        mx = row16_max(mx);
        for (int c = x + sl; c < x + a; c += 16) F[c] = mx + b;
        if (e < nm && sl == 0) q.Y[c0 + k] = mx;
        if (e < nm) Hw = max(Hw, mx + b);
      }
      for (int e = w; e < nwd; e += NW) {
        const int k = WW[e];
        const uint32_t ab = AB[k];
        const int a = (int)(ab & 0xFFFFu), b = (int)(ab >> 16);
        const int o = (int)Xr[k] - row.base;
        const int x = row.right ? L - o - a : o;
        int mx = 0;
        for (int c = x + lane; c < x + a; c += kWave) mx = max(mx, F[c]);
        const int y = wave_max_dpp(mx);
        for (int c = x + lane; c < x + a; c += kWave) F[c] = y + b;
        if (lane == 0) q.Y[c0 + k] = y;
        Hw = max(Hw, y + b);
      }
      const int hw = wave_max_dpp(Hw);
      if (lane == 0) atomicMax(&Hsh[seg % 3], hw);
      __syncthreads();
      // every wave read the same settled value: all leave at the same segment
      if (hprev > L) {
        over = true;
        break;
      }
      s0 = s1;
      s1 = s1n;
      row = row_at(q, xbase, xfirst);
    }
  }
}

template <int NT>
__device__ __forceinline__ void k_pack_box_body(const float2* __restrict__ wh,
                                                 const FrameState* __restrict__ st, FrameParams p,
                                                 long long* __restrict__ cand_x,
                                                 uint32_t* __restrict__ cand_ab,
                                                 int32_t* __restrict__ cand_y,
                                                 int32_t* __restrict__ cand_tab, int64_t stride,
                                                 int kcap) {
  extern __shared__ __align__(16) int32_t S[];
  constexpr int NW = NT / kWave;
  __shared__ uint32_t shs[2][NW];
  __shared__ int32_t shm[NW], shb[NW];
  __shared__ uint2 shn[NW];
  __shared__ int32_t Hsh[3];
  __shared__ long long last_x;
  __shared__ long long sh64[NW];
  __shared__ int32_t LC[2][2];  // by columns: boxes in the mid and the wide list

  if (st->status != FA_OK) return;
  const int j = blockIdx.x + 1;
  const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
  const int C = st->num_charts;
  const int omega = p.omega, lg = p.log2omega;
  long long* Xg = cand_x + (int64_t)(j - 1) * stride;
  uint32_t* ABg = cand_ab + (int64_t)(j - 1) * stride;
  int32_t* Y = cand_y + (int64_t)(j - 1) * stride;
  int32_t* tab = cand_tab + (j - 1) * kCandStride;
  uint32_t* Xr = reinterpret_cast<uint32_t*>(S);
  uint32_t* AB = Xr + kcap;

  // ---- sizes, fold and overflow: kFoldItems consecutive boxes per thread, a
  // thread-local prefix, then one block scan of the thread sums; the first
  // chunk goes straight to LDS
  const float s = (float)j / (float)p.J;
  const int pad = 2 * p.gutter;
  long long run = 0;
  int mloc = INT_MIN, bad = 0;
  uint32_t narrow = 0, wide = 0;  // boxes of at most kNarrow and of more than 64 columns
  if (tid == 0) last_x = 0;
  if (C <= kFewBoxes) columns_clear<NT>(omega, S + 3 * kcap + 4, Hsh, LC);
  int pass = 0;
  for (int base = 0; base < C; base += kFoldItems * NT, ++pass) {
    const int i0 = base + kFoldItems * tid;
    int a[kFoldItems], b[kFoldItems];
    uint32_t own = 0;
#pragma unroll
    for (int u = 0; u < kFoldItems; ++u) {
      a[u] = b[u] = 0;
      if (i0 + u < C) {
        const float2 v = wh[i0 + u];
        a[u] = max(p.min_box, (int)ceilf(v.x * s)) + pad;
        b[u] = max(p.min_box, (int)ceilf(v.y * s)) + pad;
        if (a[u] > 2 * omega || b[u] > 2 * omega) bad = 1;  // cannot fit: m > omega or H > L
        a[u] = min(a[u], 2 * omega + 1);  // (the clamp only touches rejected candidates)
        b[u] = min(b[u], 2 * omega + 1);
      }
      own += (uint32_t)a[u];
    }
    uint32_t tot;
    const uint32_t incl = block_incl_scan_dpp<NT>(own, shs[pass & 1], &tot);
    long long Xi = run + (long long)(incl - own);
    run += tot;
    uint32_t xs[kFoldItems], abs_[kFoldItems];
#pragma unroll
    for (int u = 0; u < kFoldItems; ++u) {
      const int i = i0 + u;
      xs[u] = (uint32_t)Xi;
      abs_[u] = (uint32_t)a[u] | ((uint32_t)b[u] << 16);
      if (i < C) {
        Xg[i] = Xi;
        ABg[i] = abs_[u];
        if (i == C - 1) last_x = Xi;
        mloc = max(mloc, (int)(Xi & (long long)(omega - 1)) + a[u] - omega);
        narrow += a[u] <= kNarrow;
        wide += a[u] > kWave;
        Xi += a[u];
      }
    }
    // the first chunk to LDS, one 16-byte store per array (i0 is a multiple
    // of 4 and kcap of 64; entries past C are never read)
    if (i0 < kcap) {
      *reinterpret_cast<uint4*>(Xr + i0) = make_uint4(xs[0], xs[1], xs[2], xs[3]);
      *reinterpret_cast<uint4*>(AB + i0) = make_uint4(abs_[0], abs_[1], abs_[2], abs_[3]);
    }
  }
  {
    const int wm = wave_max_dpp(mloc), wb = wave_max_dpp(bad);
    const uint32_t wn = wave_incl_scan_dpp(narrow), ww = wave_incl_scan_dpp(wide);
    if (lane == kWave - 1) {
      shm[w] = wm;
      shb[w] = wb;
      shn[w] = make_uint2(wn, ww);
    }
  }
  __syncthreads();
  int m = 0;
  bad = 0;
  narrow = wide = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    m = max(m, shm[k]);
    bad = max(bad, shb[k]);
    narrow += shn[k].x;
    wide += shn[k].y;
  }
  if (bad) {
    // a box side above 2 omega rejects the candidate; its overflow m and row
    // count are still reported exactly, from the unclamped widths in 64 bits
    long long run2 = 0, ml = 0, lx = 0;
    for (int base = 0; base < C; base += NT) {
      const int i = base + tid;
      long long a = 0;
      if (i < C) a = max(p.min_box, (int)ceilf(wh[i].x * s)) + pad;
      long long tot;
      const long long incl = block_incl_scan<long long>(a, sh64, &tot);
      const long long Xi = run2 + incl - a;
      run2 += tot;
      if (i < C) {
        ml = max(ml, (Xi & (long long)(omega - 1)) + a - omega);
        if (i == C - 1) lx = Xi;
      }
    }
    ml = block_max<long long>(ml, sh64);
    lx = block_max<long long>(lx, sh64);
    if (tid == 0) {
      tab[0] = 0;
      tab[1] = (int32_t)min(ml, (long long)INT_MAX);
      tab[2] = (int32_t)min(ml + omega, (long long)INT_MAX);
      tab[3] = -1;
      tab[4] = (int32_t)min((lx >> lg) + 1, (long long)INT_MAX);
    }
    return;
  }
  const long long rows = C > 0 ? (last_x >> lg) + 1 : 0;
  if (m > omega) {
    if (tid == 0) {
      tab[0] = 0;
      tab[1] = m;
      tab[2] = m + omega;
      tab[3] = -1;
      tab[4] = (int32_t)min(rows, (long long)INT_MAX);
    }
    return;
  }
  const int L = omega + m;

  const PushArgs q{Xg, ABg, Y, C, omega, lg, m, kcap};
  // two rows have to fit a chunk (a row holds boxes at least min_box + 2
  // gutter wide that start in omega columns)
  const bool by_rows = C > kFewBoxes && m <= kEdgeMax &&
                       2 * (omega / (p.min_box + pad) + 2) <= row_kcap(omega) &&
                       !columns_cheaper<NT>(q, (float)rows, (float)narrow, (float)wide);
  if (__builtin_amdgcn_readfirstlane(by_rows)) {
    push_rows<NT>(q, S, pass, shs, Hsh);
  } else {
    push_columns<NT>(q, S, pass, shs, Hsh, LC);
  }
  if (tid == 0) {
    const int H = C > 0 ? max(Hsh[0], max(Hsh[1], Hsh[2])) : 0;
    tab[0] = H <= L ? 1 : 0;
    tab[1] = m;
    tab[2] = L;
    tab[3] = H;
    tab[4] = (int32_t)min(rows, (long long)INT_MAX);
  }
}
template <int NT>
__global__ __launch_bounds__(NT) void k_pack_box(const float2* __restrict__ wh,
                                                 const FrameState* __restrict__ st, FrameParams p,
                                                 long long* __restrict__ cand_x,
                                                 uint32_t* __restrict__ cand_ab,
                                                 int32_t* __restrict__ cand_y,
                                                 int32_t* __restrict__ cand_tab, int64_t stride,
                                                 int kcap) {
  k_pack_box_body<NT>(wh, st, p, cand_x, cand_ab, cand_y, cand_tab, stride, kcap);
}

// Footprint push: pooled profile of every box of every candidate that its
// fold did not reject, content column k of box i at pool[X_i + k] as
// T | B << 16 (B = 0x7FFF: the box bottom; 0xFFFFFFFF: empty). One lane per
// fold position of candidate blockIdx.y + 1: the box is the last one starting
// at or before it, positions in the box's right gutter are skipped.
// Bound by dependent loads: a wave searches the fold 64 ways for its first
// position, fetches the boxes from there on, one a lane (each has a column at
// least), and a lane finds its own from marks where they start; the profile
// columns under a position are loaded four or sixteen at a time (144 charts, 64
// candidates: 21 -> 12 us).
template <int N>
__device__ __forceinline__ void rows_of(const int2* pr, int u0, int u1, int& tmin, int& bmax) {
  for (int u = u0; u <= u1; u += N) {
    int2 v[N];
#pragma unroll
    for (int h = 0; h < N; ++h) v[h] = pr[min(u + h, u1)];
#pragma unroll
    for (int h = 0; h < N; ++h) {
      if (v[h].y < 0) continue;
      tmin = min(tmin, v[h].x);
      bmax = max(bmax, v[h].y);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_fp_pool(
    const float2* __restrict__ wh, const FrameState* __restrict__ st, FrameParams p,
    const long long* __restrict__ cand_x, const uint32_t* __restrict__ cand_ab,
    const int32_t* __restrict__ cand_tab, int64_t stride, const int32_t* __restrict__ order,
    const int32_t* __restrict__ fp_off, const int2* __restrict__ fp_prof,
    uint32_t* __restrict__ fp_pool, int64_t pool_stride) {
  if (st->status != FA_OK) return;
  const int j = blockIdx.y + 1;
  if (cand_tab[(j - 1) * kCandStride + 3] < 0) return;
  const int C = st->num_charts;
  if (C == 0) return;
  const int J = p.J;
  const long long* X = cand_x + (int64_t)(j - 1) * stride;
  const uint32_t* AB = cand_ab + (int64_t)(j - 1) * stride;
  uint32_t* pool = fp_pool + (int64_t)(j - 1) * pool_stride;
  const long long end = X[C - 1] + (long long)(AB[C - 1] & 0xFFFFu);
  __shared__ uint32_t marks[kBlock / kWave][kWave];
  const int lane = lane_id();
  uint32_t* mark = marks[threadIdx.x / kWave];
  for (long long pos0 = (long long)blockIdx.x * kBlock + (threadIdx.x & ~(kWave - 1)); pos0 < end;
       pos0 += (long long)gridDim.x * kBlock) {
    int lo = 0, hi = C;  // the last box starting at or before pos0
    while (hi - lo > 1) {
      const int step = (hi - lo + kWave - 1) / kWave;
      const int probe = lo + lane * step;
      const int n = __popcll(__ballot(probe < hi && X[probe] <= pos0));
      lo += (n - 1) * step;
      hi = min(hi, lo + step);
    }
    // starts relative to pos0 (the first one's at most 2^15 before it)
    const int rel = lo + lane < C ? (int)min(X[lo + lane] - pos0, (long long)kWave) : kWave;
    mark[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (rel < kWave) mark[max(rel, 0)] = (uint32_t)lane + 1u;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int own = (int)wave_incl_max_dpp(mark[lane]) - 1;
    const int i = lo + own;
    const int kk = lane - __shfl(rel, own, kWave);
    const long long pos = pos0 + lane;
    if (pos >= end || kk >= (int)(AB[i] & 0xFFFFu) - p.gutter) continue;
    const float2 sz = wh[i];
    const int Uc = (int)floorf(sz.x) + 1, Rc = (int)floorf(sz.y) + 1;
    const int2* pr = fp_prof + fp_off[order[i]];
    const int u0 = min(Uc - 1, max(0, (kk * J + j - 1) / j - 1));
    const int u1 = min(Uc - 1, ((kk + 1) * J + j - 1) / j - 1);
    int tmin = INT_MAX, bmax = -1;
    if (J < 4 * j) rows_of<4>(pr, u0, u1, tmin, bmax);  // (uniform)
    else rows_of<16>(pr, u0, u1, tmin, bmax);
    uint32_t q = 0xFFFFFFFFu;
    if (bmax >= 0) {
      const int T = tmin * j / J;
      const int B = bmax == Rc - 1 ? 0x7FFF : min((bmax + 1) * j / J, 0x7FFF);
      q = (uint32_t)T | ((uint32_t)B << 16);
    }
    pool[pos] = q;
  }
}

// Selection and placement in one kernel: every workgroup reduces the J
// candidate records (one lane per candidate) to the largest effective scale
// j/L_j among fitting candidates (ties -> larger j), workgroup 0 publishes it,
// then every thread places one chart from the chosen candidate.
__device__ __forceinline__ bool sel_better(int j1, int L1, int j2, int L2) {
  if (j1 == 0) return false;
  if (j2 == 0) return true;
  const long long a = (long long)j1 * L2, b = (long long)j2 * L1;
  return a > b || (a == b && j1 > j2);
}

// Box i of the packing order at its place in candidate jm + 1; its texel range
// and the rows it reaches in the strips of the occupancy count.
__device__ __forceinline__ void place_box(const FrameParams& p, int jm, int L, int i,
                                          const int32_t* __restrict__ order,
                                          const long long* __restrict__ cand_x,
                                          const uint32_t* __restrict__ cand_ab,
                                          const int32_t* __restrict__ cand_y, int64_t stride,
                                          fa_chart* __restrict__ charts,
                                          int4* __restrict__ chart_tex, uint32_t* strips,
                                          int32_t* __restrict__ placements) {
  const long long Xi = cand_x[(int64_t)jm * stride + i];
  const uint32_t ab = cand_ab[(int64_t)jm * stride + i];
  const int a = (int)(ab & 0xFFFFu), b = (int)(ab >> 16);
  const long long r = Xi >> p.log2omega;
  const int o = (int)(Xi - (r << p.log2omega));
  fa_chart& ch = charts[order[i]];
  const int x = (r % 3 == 0) ? o : L - o - a, y = cand_y[(int64_t)jm * stride + i];
  ch.x = x;
  ch.y = y;
  ch.w = a;
  ch.h = b;
  if (placements) {
    int32_t* o = placements + 5 * (int64_t)order[i];
    o[0] = x;
    o[1] = y;
    o[2] = a;
    o[3] = b;
    o[4] = ch.rotated;
    return;  // (no occupancy map follows)
  }
  if (chart_tex) {
    // texels t whose centre lies in the box: 2 x omega <= (2t+1) L < 2 (x+w) omega
    const int64_t om = p.omega, L2 = 2 * (int64_t)L;
    const int4 r = make_int4((int)ceil_div64(2 * (int64_t)x * om - L, L2),
                             (int)ceil_div64(2 * ((int64_t)x + a) * om - L, L2) - 1,
                             (int)ceil_div64(2 * (int64_t)y * om - L, L2),
                             (int)ceil_div64(2 * ((int64_t)y + b) * om - L, L2) - 1);
    chart_tex[order[i]] = r;
    const int c0 = max(r.x, 0) / kStripTexels, c1 = min(r.y, p.omega - 1) / kStripTexels;
    const int top = min(r.w + 1, p.omega);  // (box sides may lie past the map's edge)
    if (top > 0 && r.y >= 0)
      for (int c = c0; c <= c1; ++c) atomicMax(&strips[c], (uint32_t)top);
  }
}

__device__ __forceinline__ void k_select_place_body(
    FrameParams p, const int32_t* __restrict__ cand_tab, FrameState* st,
    int32_t* __restrict__ cand_out, const int32_t* __restrict__ order,
    const long long* __restrict__ cand_x, const uint32_t* __restrict__ cand_ab,
    const int32_t* __restrict__ cand_y, int64_t stride, fa_chart* __restrict__ charts,
    int4* __restrict__ chart_tex, int32_t* __restrict__ placements = nullptr,
    fa_atlas_meta* __restrict__ meta = nullptr,
    const unsigned long long* __restrict__ big_counter = nullptr) {
  __shared__ int sj, sL;
  __shared__ uint32_t strips[kMaxStrips];
  const int C = st->num_charts;
  const int tid = threadIdx.x;
  if (blockIdx.x > 0 && (int64_t)blockIdx.x * kBlock >= C) return;
  if (tid < kMaxStrips) strips[tid] = 0u;
  if (tid < kWave) {
    // the first wave alone reads the status, which workgroup 0 may set below
    // while others start: were every wave to read it, some of a workgroup's
    // might leave and the rest place boxes by a winner that nobody wrote
    const bool ok = st->status == FA_OK;
    if (blockIdx.x == 0 && tid < p.J && cand_out) {
      const int32_t* t = cand_tab + tid * kCandStride;
      int32_t* o = cand_out + 4 * tid;
      o[0] = ok ? t[0] : 0; o[1] = ok ? t[1] : 0; o[2] = ok ? t[2] : 0; o[3] = ok ? t[3] : 0;
    }
    int j = 0, L = 1, H0 = 0, rows0 = 0;
    if (ok && tid < p.J) {
      const int32_t* t = cand_tab + tid * kCandStride;
      if (t[0]) { j = tid + 1; L = t[2]; H0 = t[3]; rows0 = t[4]; }
    }
    // over the rows of 16 lanes by DPP (pairs, quads, half rows, rows), then
    // over the rows
    auto better = [&](int oj, int oL) {
      if (sel_better(oj, oL, j, L)) { j = oj; L = oL; }
    };
    better(dpp_keep<0xB1>(j), dpp_keep<0xB1>(L));
    better(dpp_keep<0x4E>(j), dpp_keep<0x4E>(L));
    better(dpp_keep<0x141>(j), dpp_keep<0x141>(L));
    better(dpp_keep<0x140>(j), dpp_keep<0x140>(L));
#pragma unroll
    for (int r = 0; r < kWave; r += 16)
      better(__builtin_amdgcn_readlane(j, r), __builtin_amdgcn_readlane(L, r));
    j = __builtin_amdgcn_readfirstlane(j);
    L = __builtin_amdgcn_readfirstlane(L);
    // (the winner's record is in lane j - 1)
    const int H = __builtin_amdgcn_readlane(H0, max(j - 1, 0));
    const int rows = __builtin_amdgcn_readlane(rows0, max(j - 1, 0));
    if (tid == 0) {
      sj = j;
      sL = L;
      if (blockIdx.x == 0) {
        if (ok) {
          st->jstar = j;
          if (!j) {
            st->status = FA_ERR_NOFIT;
          } else {
            st->layout_w = L;
            st->layout_h = H;
            st->rows = rows;
            st->s_star = (float)j / (float)p.J;
            st->q_star = (float)p.omega / (float)L;
          }
        }
        if (meta) write_meta(p, st, big_counter, false, 0ull, meta);
      }
    }
  }
  __syncthreads();
  const int jm = sj - 1, L = sL;
  if (jm < 0) return;
  const int i = blockIdx.x * kBlock + tid;
  if (i < C) place_box(p, jm, L, i, order, cand_x, cand_ab, cand_y, stride, charts, chart_tex, strips,
                       placements);
  __syncthreads();
  if (chart_tex && tid < kMaxStrips && strips[tid]) atomicMax(&st->strip_rows[tid], strips[tid]);
}
__global__ __launch_bounds__(kBlock) void k_select_place(
    FrameParams p, const int32_t* __restrict__ cand_tab, FrameState* st,
    int32_t* __restrict__ cand_out, const int32_t* __restrict__ order,
    const long long* __restrict__ cand_x, const uint32_t* __restrict__ cand_ab,
    const int32_t* __restrict__ cand_y, int64_t stride, fa_chart* __restrict__ charts,
    int4* __restrict__ chart_tex) {
  k_select_place_body(p, cand_tab, st, cand_out, order, cand_x, cand_ab, cand_y, stride, charts, chart_tex);
}

// ... of the packer-only entry: placements and the frame record with it
__global__ __launch_bounds__(kBlock) void k_select_emit(
    FrameParams p, const int32_t* __restrict__ cand_tab, FrameState* st,
    int32_t* __restrict__ cand_out, const int32_t* __restrict__ order,
    const long long* __restrict__ cand_x, const uint32_t* __restrict__ cand_ab,
    const int32_t* __restrict__ cand_y, int64_t stride, fa_chart* __restrict__ charts,
    int32_t* __restrict__ placements, fa_atlas_meta* __restrict__ meta,
    const unsigned long long* __restrict__ big_counter) {
  k_select_place_body(p, cand_tab, st, cand_out, order, cand_x, cand_ab, cand_y, stride, charts,
                      nullptr, placements, meta, big_counter);
}

// ---- batched wrappers (view = blockIdx.y) --------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void k_pack_box_b(const BatchView* __restrict__ bv,
                                                   int64_t stride) {
  const BatchView& v = bv[blockIdx.y];
  k_pack_box_body<NT>(in_global(v.w.sorted_wh), in_global(v.w.state), v.p, in_global(v.w.cand_x), in_global(v.w.cand_ab), in_global(v.w.cand_y),
                      in_global(v.w.cand_tab), stride, box_kcap(v.p.omega));
}
__global__ __launch_bounds__(kBlock) void k_select_place_b(const BatchView* __restrict__ bv,
                                                           int64_t stride) {
  const BatchView& v = bv[blockIdx.y];
  k_select_place_body(v.p, in_global(v.w.cand_tab), in_global(v.w.state), in_global(v.cand_out), in_global(v.w.vals_a), in_global(v.w.cand_x),
                      in_global(v.w.cand_ab), in_global(v.w.cand_y), stride, in_global(v.charts), in_global(v.w.chart_tex));
}

// ---- packer-only entry: box sizes in, placements out ---------------------
__global__ void k_pack_state(FrameState* st, int32_t n) {
  constexpr unsigned kCharts = offsetof(FrameState, num_charts) / 4;
  for (unsigned i = threadIdx.x; i < sizeof(FrameState) / 4; i += blockDim.x)
    reinterpret_cast<uint32_t*>(st)[i] = i == kCharts ? (uint32_t)n : 0u;  // (FA_OK is 0)
}

}  // namespace

namespace {

hipError_t box_attributes() {
  const void* ks[6] = {(const void*)k_pack_box<256>,    (const void*)k_pack_box<512>,
                       (const void*)k_pack_box<1024>,   (const void*)k_pack_box_b<256>,
                       (const void*)k_pack_box_b<512>, (const void*)k_pack_box_b<1024>};
  for (const void* k : ks) {
    const hipError_t e =
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)box_lds_max());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

void box_launch(const FrameParams& p, const Work& w, int block, hipStream_t st) {
  const int64_t stride = p.max_charts;
  const int kcap = box_kcap(p.omega);
  const size_t dyn = box_lds(p.omega);
  if (block == 1024)
    k_pack_box<1024><<<p.J, 1024, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                             w.cand_y, w.cand_tab, stride, kcap);
  else if (block == 512)
    k_pack_box<512><<<p.J, 512, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                           w.cand_y, w.cand_tab, stride, kcap);
  else
    k_pack_box<256><<<p.J, 256, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                           w.cand_y, w.cand_tab, stride, kcap);
}

template <int MODE>
hipError_t pack_attributes(int max_dyn_bytes) {
  hipError_t e = hipFuncSetAttribute((const void*)k_pack<256, MODE>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, max_dyn_bytes);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_pack<512, MODE>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, max_dyn_bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_pack<1024, MODE>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, max_dyn_bytes);
}

template <int MODE>
void pack_launch(const FrameParams& p, const Work& w, int block, size_t dyn, hipStream_t st) {
  const int64_t stride = p.max_charts;
  if (block == 1024)
    k_pack<1024, MODE><<<p.J, 1024, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                               w.cand_y, w.cand_rs, w.cand_tab, stride,
                                               w.fp_pool, p.pool_stride);
  else if (block == 512)
    k_pack<512, MODE><<<p.J, 512, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                             w.cand_y, w.cand_rs, w.cand_tab, stride, w.fp_pool,
                                             p.pool_stride);
  else
    k_pack<256, MODE><<<p.J, 256, dyn, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                             w.cand_y, w.cand_rs, w.cand_tab, stride, w.fp_pool,
                                             p.pool_stride);
}
}  // namespace

hipError_t pack_kernel_attributes(int max_frontline_bytes) {
  const int max_dyn_bytes = max_frontline_bytes + kPackLds * 16 + 4;
  hipError_t e = box_attributes();
  if (e == hipSuccess) e = pack_attributes<1>(max_dyn_bytes);
  if (e == hipSuccess) e = pack_attributes<2>(max_dyn_bytes);
  return e;
}

hipError_t launch_pack(const FrameParams& p, const Work& w, int block, bool footprint,
                       hipStream_t st) {
  const size_t dyn = (size_t)2 * p.omega * sizeof(int32_t) + (size_t)kPackLds * 16 + 4;
  if (!footprint) {
    box_launch(p, w, block, st);
    return hipGetLastError();
  }
  pack_launch<1>(p, w, block, dyn, st);
  k_fp_pool<<<dim3(32, p.J), kBlock, 0, st>>>(w.sorted_wh, w.state, p, w.cand_x, w.cand_ab,
                                              w.cand_tab, p.max_charts, w.vals_a, w.fp_off,
                                              w.fp_prof, w.fp_pool, p.pool_stride);
  pack_launch<2>(p, w, block, dyn, st);
  return hipGetLastError();
}

hipError_t launch_select_place(const FrameParams& p, const Work& w, fa_chart* charts,
                               int32_t* cand_out, hipStream_t st) {
  k_select_place<<<(unsigned)((p.max_charts + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      p, w.cand_tab, w.state, cand_out, w.vals_a, w.cand_x, w.cand_ab, w.cand_y, p.max_charts,
      charts, w.chart_tex);
  return hipGetLastError();
}

hipError_t launch_pack_state(int32_t n, const Work& w, hipStream_t st) {
  k_pack_state<<<1, 256, 0, st>>>(w.state, n);
  return hipGetLastError();
}

hipError_t launch_select_emit(const FrameParams& p, const Work& w, int32_t n, fa_chart* charts,
                              int32_t* cand_out, int32_t* placements, fa_atlas_meta* meta,
                              hipStream_t st) {
  k_select_emit<<<(unsigned)std::max(1, (n + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      p, w.cand_tab, w.state, cand_out, w.vals_a, w.cand_x, w.cand_ab, w.cand_y, p.max_charts,
      charts, placements, meta, w.big_counter);
  return hipGetLastError();
}

hipError_t launch_pack_batched(const BatchView* dev, int n, int J, int64_t max_charts, int block,
                               hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const size_t dyn = box_lds_max();  // each view sizes its chunks from its own omega
  if (block == 1024)
    k_pack_box_b<1024><<<dim3(J, n), 1024, dyn, st>>>(dev, max_charts);
  else if (block == 512)
    k_pack_box_b<512><<<dim3(J, n), 512, dyn, st>>>(dev, max_charts);
  else
    k_pack_box_b<256><<<dim3(J, n), 256, dyn, st>>>(dev, max_charts);
  k_select_place_b<<<dim3((unsigned)((max_charts + kBlock - 1) / kBlock), n), kBlock, 0, st>>>(
      dev, max_charts);
  return hipGetLastError();
}

}  // namespace fa
