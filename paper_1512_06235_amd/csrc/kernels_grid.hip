// Grid-based approximate candidate search (Section 6.2.1, eqs. 4-9, and the
// GPU steps 1, 3 and 4 of Appendix A).
//
// The paper bins b's features into four grids of 2d x 2d cells, shifted by
// (0,0), (d,0), (0,d) and (d,d).  A query's line is cut by b's keypoint box at
// A and B; K + 1 equidistant points are taken between them (K the smallest
// integer with K d >= |AB|), and each point selects the centre-most of the
// four cells that contain it.  C' is the union of the features of the selected
// cells; the two nearest of C' by exact squared L2 and the ratio test decide
// the match.  C' approximates the band of eq. (2): it can hold features up to
// 2d (per axis) from a sample point and miss band members near a cell corner.
//
// Here b is binned once, into d x d cells: a cell of any of the four grids is a
// block of 2 x 2 of them, and the centre-most cell of a point is the block
// around its nearest multiple of d in x and y.  Along a line the blocks move
// monotonically in x and in y, so the samples whose block holds a given cell
// follow each other, and a cell is new to C' exactly when the sample before
// did not hold it: no set needs to be kept.  (Rounding can make a line that
// runs along a boundary between two blocks step back and forth; a query where
// that happens compares with eight samples instead of one, see walk_robust.)
//
// Every floating-point decision (crossings, sample points, cells, centre
// distances) has the result of IEEE double with no contraction, in a fixed
// order, so the result is reproducible bit for bit by a plain implementation
// of the same steps.  Cells and samples are first placed by one multiplication
// with 1 / d; where that lands within 1e-5 of a cell boundary (its error is
// below 1e-6: coordinates are at most 2^31 cells from the origin) the steps
// are evaluated as written.
#include <algorithm>
#include <cmath>


#include "line.h"
#include "sfm_internal.h"

#pragma clang fp contract(off)

namespace sfm {
namespace {

constexpr int kBinThreads = 1024;
constexpr double kNearEdge = 1e-5;   // cells: nearer than this to an edge, decide as written

// d x d cell of coordinate x: the two 2d-wide cells (shift 0 and d) that hold x
// are floor(x / 2d) and floor((x - d) / 2d), and these two name it.
__device__ __forceinline__ int32_t fine_cell(double x, double d, double inv_d) {
  const double t = x * inv_d, m = floor(t), f = t - m;
  if (f > kNearEdge && f < 1.0 - kNearEdge) return int32_t(m);
  const double two_d = 2.0 * d;
  return int32_t(floor(x / two_d) + floor((x - d) / two_d) + 1.0);
}

// Cells are stored in strips of four rows, column by column within a strip:
// cell (x, y) is 4 x + cell_row(y).  A line in any direction then touches few
// lines of the start table (read column by column over the whole height, nearly
// every sample was a line of its own).
__device__ __forceinline__ int32_t cell_row(int32_t strip, int32_t y) {
  return (y >> 2) * strip + (y & 3);
}
// cell_row(y + 1) from r = cell_row(y).
__device__ __forceinline__ int32_t next_row(int32_t strip, int32_t y, int32_t r) {
  return r + ((y & 3) == 3 ? strip - 3 : 1);
}

// One workgroup per (pair, strip of kGridLdsCells cells in storage order):
// counts per cell in LDS, a scan, then a scatter of the features of the strip;
// the features of earlier strips are only counted.  Features of one cell land
// in any order; C' is a set, so the order never matters.
__global__ __launch_bounds__(kBinThreads) void grid_bin_kernel(GridView v) {
  extern __shared__ int32_t cnt[];
  __shared__ int32_t wsum[kBinThreads / 64], wbelow[kBinThreads / 64];
  const int32_t p = blockIdx.x;
  const GridPair* P = v.pairs + p;
  const int64_t ncell = P->ncell;
  const int64_t c0 = int64_t(blockIdx.y) * v.strip_cells;
  if (c0 >= ncell) return;   // uniform
  const int32_t nc = int32_t(min(ncell - c0, int64_t(v.strip_cells)));
  const ImageDev B = v.images[P->b];
  const int32_t nb = P->nb, fx0 = P->fx0, fy0 = P->fy0, nfx = P->nfx, nfy = P->nfy;
  const int32_t strip = P->strip;
  const double d = P->d, inv_d = 1.0 / d;
  int32_t* start = v.cell_start + P->cell_off + c0;
  int32_t* items = v.items + P->item_off;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int32_t c = t; c < nc; c += kBinThreads) cnt[c] = 0;
  __syncthreads();
  // The strip's cell of feature j: negative before the strip, nc or more after
  // it (or outside the grid).
  auto cell_of = [&](int32_t j) -> int64_t {
    const float2 xy = ldg_xy(B.xy, j);
    const int32_t cx = fine_cell(double(xy.x), d, inv_d) - fx0;
    const int32_t cy = fine_cell(double(xy.y), d, inv_d) - fy0;
    if (cx < 0 || cx >= nfx || cy < 0 || cy >= nfy) {
      *v.err = 1;
      return nc;
    }
    return int64_t(4 * cx) + cell_row(strip, cy) - c0;
  };
  int32_t below = 0;
  for (int32_t j = t; j < nb; j += kBinThreads) {
    const int64_t c = cell_of(j);
    if (c < 0)
      ++below;
    else if (c < nc)
      atomicAdd(&cnt[c], 1);
  }
  __syncthreads();
  // Exclusive scan: each thread owns a contiguous run of cells.
  const int32_t chunk = (nc + kBinThreads - 1) / kBinThreads;
  const int32_t r0 = min(nc, chunk * t), r1 = min(nc, r0 + chunk);
  int32_t sum = 0;
  for (int32_t c = r0; c < r1; ++c) sum += cnt[c];
  int32_t inc = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o, 64);
  if (lane == 63) wsum[wave] = inc;
  if (lane == 0) wbelow[wave] = below;
  __syncthreads();
  int32_t run = inc - sum;
  for (int w = 0; w < kBinThreads / 64; ++w) run += wbelow[w] + (w < wave ? wsum[w] : 0);
  for (int32_t c = r0; c < r1; ++c) {
    const int32_t n = cnt[c];
    start[c] = run;
    cnt[c] = run;
    run += n;
  }
  if (t == kBinThreads - 1 && c0 + nc == ncell) start[nc] = run;
  __syncthreads();
  for (int32_t j = t; j < nb; j += kBinThreads) {
    const int64_t c = cell_of(j);
    if (c >= 0 && c < nc) items[atomicAdd(&cnt[c], 1)] = j;
  }
}

__device__ __forceinline__ unsigned long long wave_min(unsigned long long x) {
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long y = __shfl_xor(x, o, 64);
    x = y < x ? y : x;
  }
  return x;
}

// The line of query i of pair pr cut by b's keypoint box: crossings on the
// edges x = x0, x = x1, y = y0, y = y1 in that order; A is the first, B the
// first of those farthest from A.  False without a crossing.
__device__ __forceinline__ bool line_crossings(const GridView& v, const GridPair* P, int32_t pr,
                                               const ImageDev& A, int32_t i, double& xA,
                                               double& yA, double& xB, double& yB) {
  const double xa = double(A.xy[2 * i]), ya = double(A.xy[2 * i + 1]);
  const double* F = v.F + 9 * int64_t(pr);
  const double la = F[0] * xa + F[1] * ya + F[2];
  const double lb = F[3] * xa + F[4] * ya + F[5];
  const double lc = F[6] * xa + F[7] * ya + F[8];
  const double x0 = P->box[0], y0 = P->box[1], x1 = P->box[2], y1 = P->box[3];
  int nh = 0;
  double far = -1.0;
  auto hit = [&](double x, double y) {
    if (nh++ == 0) { xA = x; yA = y; }
    const double dx = x - xA, dy = y - yA;
    const double r = dx * dx + dy * dy;
    if (r > far) { xB = x; yB = y; far = r; }
  };
  if (lb != 0.0) {
    const double ya0 = -(la * x0 + lc) / lb;
    if (y0 <= ya0 && ya0 <= y1) hit(x0, ya0);
    const double ya1 = -(la * x1 + lc) / lb;
    if (y0 <= ya1 && ya1 <= y1) hit(x1, ya1);
  }
  if (la != 0.0) {
    const double xb0 = -(lb * y0 + lc) / la;
    if (x0 <= xb0 && xb0 <= x1) hit(xb0, y0);
    const double xb1 = -(lb * y1 + lc) / la;
    if (x0 <= xb1 && xb1 <= x1) hit(xb1, y1);
  }
  return nh > 0;
}

// A query's line between its crossings: A, B and K (K < 0: no crossing, or
// no features of b).
struct Segment {
  double xA, yA, xB, yB;
  int32_t K;
};

__device__ __forceinline__ Segment query_segment(const GridView& v, const GridPair* P, int32_t pr,
                                                 const ImageDev& A, int32_t i) {
  Segment s = {0.0, 0.0, 0.0, 0.0, -1};
  if (!line_crossings(v, P, pr, A, i, s.xA, s.yA, s.xB, s.yB) || P->nb == 0) return s;
  const double dx = s.xB - s.xA, dy = s.yB - s.yA;
  const double len2 = dx * dx + dy * dy;
  const double d2 = P->d * P->d;
  int64_t K = int64_t(ceil(sqrt(len2) / P->d));
  while (K > 0 && double((K - 1) * (K - 1)) * d2 >= len2) --K;
  while (double(K * K) * d2 < len2) ++K;
  s.K = int32_t(K);
  return s;
}

// Samples of one segment.  at(k): the lower corner of the block of 2 x 2 cells
// that sample k selects, relative to the pair's first cell.
struct Sampler {
  const Segment* seg;   // in LDS
  int32_t K;
  double d, inv_d, tx, ty, dtx, dty;
  int32_t fx0, fy0, xmax, ymax;   // first cell; last lower corner of a block

  __device__ __forceinline__ Sampler(const Segment& s, bool live, const GridPair* P)
      : seg(&s), K(live ? s.K : -1), d(P->d), inv_d(1.0 / P->d), fx0(P->fx0), fy0(P->fy0), xmax(P->nfx - 2),
        ymax(P->nfy - 2) {
    const double step = K > 0 ? inv_d / double(K) : 0.0;
    // Of a sample at m d (m an integer) the block's lower corner is cell m - 1.
    tx = s.xB * inv_d - double(fx0 + 1);
    ty = s.yB * inv_d - double(fy0 + 1);
    dtx = (s.xA - s.xB) * step;
    dty = (s.yA - s.yB) * step;
  }

  // Relative to the first cell.  (Samples lie in b's box, whose cells have a
  // margin on every side: the clamp never changes one.)
  __device__ __forceinline__ int2 corner(int32_t x, int32_t y) const {
    return make_int2(min(max(x - fx0, 0), xmax), min(max(y - fy0, 0), ymax));
  }

  // As written: the sample point, and the centre-most of the four cells that
  // hold it (lower grid on ties).
  __device__ __forceinline__ int2 exact(int32_t k) const {
    const Segment s = *seg;
    const double two_d = 2.0 * d;
    double px = s.xA, py = s.yA;
    if (s.K > 0) {
      const double kd = double(k), rd = double(s.K - k), Kd = double(s.K);
      px = (kd * s.xA + rd * s.xB) / Kd;
      py = (kd * s.yA + rd * s.yB) / Kd;
    }
    double best = INFINITY, fx = 0.0, fy = 0.0;
    for (int g = 0; g < 4; ++g) {
      const double sx = (g & 1) ? d : 0.0, sy = (g & 2) ? d : 0.0;
      const double cx = floor((px - sx) / two_d), cy = floor((py - sy) / two_d);
      const double ex = px - (cx * two_d + sx + d);
      const double ey = py - (cy * two_d + sy + d);
      const double r = ex * ex + ey * ey;
      if (r < best) {
        best = r;
        fx = 2.0 * cx + double(g & 1);
        fy = 2.0 * cy + double(g >> 1);
      }
    }
    return corner(int32_t(fx), int32_t(fy));
  }

  // Relative to the first cell, from one multiplication; false where that is
  // too near an edge to tell.  (Adding 1.5 * 2^52 rounds to an integer in the
  // low bits.  Samples lie in b's box, which the grid's margin encloses, so no
  // clamp is needed.)
  __device__ __forceinline__ bool quick(int32_t k, int32_t& x, int32_t& y) const {
    constexpr double kRound = 6755399441055744.0;
    const double kd = double(k);
    const double ax = __builtin_fma(kd, dtx, tx), ay = __builtin_fma(kd, dty, ty);
    const double rx = ax + kRound, ry = ay + kRound;
    const double ex = ax - (rx - kRound), ey = ay - (ry - kRound);
    x = int32_t(uint32_t(__double_as_longlong(rx)));
    y = int32_t(uint32_t(__double_as_longlong(ry)));
    return fmax(fabs(ex), fabs(ey)) < 0.5 - kNearEdge;
  }
};

constexpr int kListCap = 256;   // found features a query lists in LDS before they are consumed

// The item range of a cell by its index (one 8-byte load; starts are 4-byte
// aligned, which global loads allow).
typedef int32_t int2u __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ int2 cell_range(const int32_t* start, int32_t c) {
  const int2u r = *reinterpret_cast<const __attribute__((address_space(1))) int2u*>(
      (const __attribute__((address_space(1))) int32_t*)(start + c));
  return make_int2(r.x, r.y);
}

// The cells that are new to C' at samples kb .. kb + kPer - 1: those of each
// sample's block that the sample before did not hold, three at most, a fourth
// for sample 0.  (The new column, then, where the block moved in y, the new
// row's cells of the columns that are not new.)  Samples past the last one
// repeat it, so nothing moves and nothing is new.  Cell 0 is in the empty
// margin of the grid.  Selections only: as branches these took most of the
// kernel's instructions.  step: the smallest and largest moves in x and y.
constexpr int kPer = 6;   // 96 samples a query and chunk: three chunks for the usual 260
constexpr int kRanges = 3 * kPer + 1;
struct Steps {
  int32_t lo_x, hi_x, lo_y, hi_y;
};
__device__ __forceinline__ void new_cells(const Sampler& S, int32_t strip, int32_t kb,
                                          int32_t (&cell)[kRanges], Steps& step) {
  const int32_t Kc = max(S.K, 0);
  int32_t cx[kPer + 1], cy[kPer + 1];   // samples kb - 1 .. kb + kPer - 1
  uint32_t edge = 0u;
#pragma unroll
  for (int u = 0; u <= kPer; ++u)
    if (!S.quick(min(u ? kb - 1 + u : max(kb - 1, 0), Kc), cx[u], cy[u])) edge |= 1u << u;
  while (edge) {
    const int u = __builtin_ctz(edge);
    edge &= edge - 1;
    const int2 e = S.exact(min(max(kb - 1 + u, 0), Kc));
#pragma unroll
    for (int n = 0; n <= kPer; ++n) {
      cx[n] = n == u ? e.x : cx[n];
      cy[n] = n == u ? e.y : cy[n];
    }
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int32_t x = cx[u + 1], y = cy[u + 1];
    const int32_t my = y - cy[u];
    int32_t mx = x - cx[u];
    step.lo_x = min(step.lo_x, mx);
    step.hi_x = max(step.hi_x, mx);
    step.lo_y = min(step.lo_y, my);
    step.hi_y = max(step.hi_y, my);
    const bool first = u == 0 && kb == 0 && S.K >= 0;
    if (u == 0) mx = first ? 1 : mx;
    const int32_t X0 = 4 * x, Y0 = cell_row(strip, y), Y1 = next_row(strip, y, Y0);
    const int32_t XN = mx > 0 ? X0 + 4 : X0, YN = my > 0 ? Y1 : Y0;
    const int32_t rowA = my != 0 ? X0 + YN : 0, rowB = my != 0 ? X0 + 4 + YN : 0;
    cell[3 * u] = mx != 0 ? XN + Y0 : rowA;
    cell[3 * u + 1] = mx != 0 ? XN + Y1 : rowB;
    int32_t corner = mx != 0 ? (mx > 0 ? rowA : rowB) : 0;
    if (u == 0) {
      corner = first ? X0 + Y0 : corner;
      cell[3 * kPer] = first ? X0 + Y1 : 0;
    }
    cell[3 * u + 2] = corner;
  }
}

// The same for one sample k, where blocks step back and forth or by two: a
// cell is new when none of the eight samples before holds it.  (Samples more
// than six steps apart share no cell: a cell lies within 1.5 d of its sample
// in x and y, and K >= 2 steps are longer than d / 2.)
__device__ __forceinline__ void new_cells_robust(const Sampler& S, int32_t strip, int32_t k,
                                                 int32_t (&cell)[kRanges]) {
#pragma unroll
  for (int n = 0; n < kRanges; ++n) cell[n] = 0;
  if (k > S.K) return;
  int2 c = make_int2(0, 0);
  uint32_t held = 0u;   // bit 2 a + b: cell (x + a, y + b) is not new
  for (int32_t q = k; q >= max(0, k - 8); --q) {
    const int2 e = S.exact(q);
    if (q == k) {
      c = e;
      continue;
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int32_t x = c.x + (n >> 1) - e.x, y = c.y + (n & 1) - e.y;
      if (x >= 0 && x <= 1 && y >= 0 && y <= 1) held |= 1u << n;
    }
  }
#pragma unroll
  for (int n = 0; n < 4; ++n)
    if (!((held >> n) & 1u))
      cell[n] = 4 * (c.x + (n >> 1)) + cell_row(strip, c.y + (n & 1));
}

// Walks the samples of a query's segment with W lanes and lists every feature
// of C' once in LDS, as its position in the item array; consume(count) takes
// a list of up to kListCap of them, when it is full and at the end (a chunk
// that does not fit is worked out again after the list was taken).  Several
// queries walk side by side in one wave, so lists are taken when one of them
// is full.  Sets `back` when the blocks did not move monotonically (what was
// listed is then not C', and `robust` is to be used).  Returns the number listed.
template <int W, class Consume>
__device__ __forceinline__ int32_t walk(const GridView& v, const GridPair* P, const Sampler& S,
                                        int32_t* list, int sub, bool robust, bool& back,
                                        Consume&& consume) {
  const int32_t* start = v.cell_start + P->cell_off;
  const int32_t strip = P->strip;
  Steps step = {0, 0, 0, 0};
  int32_t found = 0, count = 0, w0 = 0;
  const int32_t stride = robust ? W : W * kPer;
  for (int32_t k0 = 0;;) {
    const bool more = __any(k0 <= S.K);
    bool take = !more;
    if (more) {
      int32_t cell[kRanges];
      if (robust)
        new_cells_robust(S, strip, k0 + sub, cell);
      else
        new_cells(S, strip, k0 + kPer * sub, cell, step);
      int2 r[kRanges];
#pragma unroll
      for (int n = 0; n < kRanges; ++n) r[n] = cell_range(start, cell[n]);
      int32_t own = 0;
#pragma unroll
      for (int n = 0; n < kRanges; ++n) own += r[n].y - r[n].x;
      int32_t inc = own;
#pragma unroll
      for (int o = 1; o < W; o <<= 1) {
        const int32_t y = __shfl_up(inc, o, W);
        if (sub >= o) inc += y;
      }
      const int32_t total = __shfl(inc, W - 1, W);
      const int32_t left = max(total - w0, 0);
      int32_t n_list = 0;   // how many of the chunk's features are listed now
      if (!__any(count + left > kListCap)) {
        n_list = left;
      } else {
        take = true;
        if (!__any(count > 0)) n_list = min(left, kListCap);
      }
      // Positions w0 .. w0 + n_list - 1 of the chunk go to count ...
      int32_t pos = inc - own - w0;
      if (!__any(n_list != total)) {
        pos += count;
        if (own > 0) {
#pragma unroll
          for (int n = 0; n < kRanges; ++n)
            for (int32_t s = r[n].x; s < r[n].y; ++s) list[pos++] = s;
        }
      } else if (n_list > 0 && pos < n_list && pos + own > 0) {
#pragma unroll
        for (int n = 0; n < kRanges; ++n)
          for (int32_t s = r[n].x; s < r[n].y; ++s, ++pos)
            if (pos >= 0 && pos < n_list) list[count + pos] = s;
      }
      const bool whole = !take;
      if (whole) {
        found += total;
        k0 += stride;
        w0 = 0;
      } else if (!__any(count > 0)) {
        w0 += kListCap;
      }
      count += n_list;
    }
    if (take) {
      wave_lds_fence();
      consume(count);
      wave_lds_fence();
      count = 0;
      if (!more) break;
    }
  }
  const bool odd = (step.lo_x < 0 && step.hi_x > 0) || (step.lo_y < 0 && step.hi_y > 0) ||
                   step.lo_x < -1 || step.hi_x > 1 || step.lo_y < -1 || step.hi_y > 1;
  // A lane sees its own samples: also steps of opposite signs on two lanes.
  uint32_t signs = (step.lo_x < 0 ? 1u : 0u) | (step.hi_x > 0 ? 2u : 0u) |
                   (step.lo_y < 0 ? 4u : 0u) | (step.hi_y > 0 ? 8u : 0u) | (odd ? 16u : 0u);
#pragma unroll
  for (int o = 1; o < W; o <<= 1) signs |= uint32_t(__shfl_xor(int32_t(signs), o, 64));
  back = (signs & 3u) == 3u || (signs & 12u) == 12u || (signs & 16u) != 0u;
  return found;
}

// The query's 128 descriptor bytes as 32 words, and its exact squared
// distance to feature j of b: |q|^2 + |b_j|^2 - 2 q.b_j.
__device__ __forceinline__ void query_words(const ImageDev& A, int32_t i, uint32_t q[32]) {
  const uint4* qd = reinterpret_cast<const uint4*>(A.desc + 128 * int64_t(i));
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const uint4 u = qd[w];
    q[4 * w] = u.x; q[4 * w + 1] = u.y; q[4 * w + 2] = u.z; q[4 * w + 3] = u.w;
  }
}

__device__ __forceinline__ unsigned long long dist_key(const uint32_t q[32], int32_t qn,
                                                       const ImageDev& B, int32_t j) {
  const uint4* bd = reinterpret_cast<const uint4*>(B.desc + 128 * int64_t(j));
  uint32_t dot = 0;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const uint4 u = bd[w];
    dot = __builtin_amdgcn_udot4(q[4 * w], u.x, dot, false);
    dot = __builtin_amdgcn_udot4(q[4 * w + 1], u.y, dot, false);
    dot = __builtin_amdgcn_udot4(q[4 * w + 2], u.z, dot, false);
    dot = __builtin_amdgcn_udot4(q[4 * w + 3], u.w, dot, false);
  }
  const int32_t D = qn + B.norm2[j] - 2 * int32_t(dot);
  // Packed keys (D << 32 | j) order by distance, then index.
  return (static_cast<unsigned long long>(uint32_t(D)) << 32) | uint32_t(j);
}

// Branch-free, so the two stay in registers (a conditional store to one of
// the two references made the compiler keep them in scratch).
__device__ __forceinline__ void push_two(unsigned long long key, unsigned long long& b1,
                                         unsigned long long& b2) {
  const bool lt1 = key < b1;
  const unsigned long long n2 = lt1 ? b1 : (key < b2 ? key : b2);
  b1 = lt1 ? key : b1;
  b2 = n2;
}

// Wave-wide two nearest of the lanes' pairs and the ratio test; lane 0
// writes the query's result and adds to its pair's counters.
__device__ __forceinline__ void grid_finish(const GridView& v, int64_t q_off, int32_t pr,
                                            int32_t i, unsigned long long b1,
                                            unsigned long long b2, int32_t n) {
  const unsigned long long m1 = wave_min(b1);
  const unsigned long long m2 = wave_min(b1 == m1 ? b2 : b1);
  if (threadIdx.x == 0) {
    QueryResult r;
    r.match = n > 0 ? int32_t(uint32_t(m1)) : -1;
    r.d1 = n > 0 ? int32_t(m1 >> 32) : kDistInf;
    r.d2 = n > 1 ? int32_t(m2 >> 32) : kDistInf;
    bool accept = false;
    if (n >= 2)
      accept = int64_t(v.ratio_den) * r.d1 < int64_t(v.ratio_num) * r.d2;
    else if (n == 1)
      accept = v.accept_single != 0;
    r.flags = (accept ? 1 : 0) | (v.keep_counts ? (n << 1) : 0);
    v.res[q_off + i] = r;
    atomicAdd(&v.counters[pr].comparisons, static_cast<unsigned long long>(n));
    if (accept) atomicAdd(&v.counters[pr].accepted, 1u);
  }
}

// Two nearest of the listed C' and the ratio test for query i of pair pr.
__device__ __forceinline__ void grid_decide(const GridView& v, int64_t q_off, int32_t pr,
                                            const ImageDev& A, const ImageDev& B, int32_t i,
                                            const int32_t* cand, int32_t n) {
  uint32_t q[32];
  query_words(A, i, q);
  const int32_t qn = A.norm2[i];
  unsigned long long b1 = ~0ull, b2 = ~0ull;
  for (int32_t s = threadIdx.x; s < n; s += 64) push_two(dist_key(q, qn, B, cand[s]), b1, b2);
  grid_finish(v, q_off, pr, i, b1, b2, n);
}

// One wave per workgroup and kGridQueriesPerBlock consecutive queries of one
// pair (an entry of the host's block table).  Lane q first cuts query q's
// line; then each 16 lanes take one query at a time, four queries side by
// side: they walk its samples, list the new features in LDS and compute the
// listed features' distances.
// C' has 30 to 300 features at the usual sizes, so 16 lanes are mostly in use
// where 64 were half idle.  Bound by the VALU: about 45 instructions a sample
// and lane (placing it, its new cells and their lists) and 75 for 16
// candidates.  60 pairs (0.43 M queries, d = 4, 257 samples and about 110
// candidates a query): 0.70 ms.  With four grids, ten FP64 divisions a sample
// and a bitmap per query it took 2.31 ms; on the way here, lanes that read
// whole rows (1.87 ms, every line of a row asked of the L2 eight times) and
// pairs dealt to all XCDs at once (1.17 ms, 5 GB of L2 misses).
constexpr int kGroupLanes = 16;

__global__ __launch_bounds__(64, 4) void grid_query_kernel(GridView v) {
  __shared__ Segment segs[kGridQueriesPerBlock];
  __shared__ int32_t lists[64 / kGroupLanes][kListCap];
  const int2 blk = read_uniform(v.blocks, int32_t(blockIdx.x));
  const int32_t pr = blk.x;
  if (pr < 0) return;   // padding of the table
  const GridPair pair = read_uniform(v.pairs, pr);
  const GridPair* P = &pair;
  const ImageDev A = read_uniform(v.images, pair.a), B = read_uniform(v.images, pair.b);
  const int64_t q_off = P->q_off;
  const int32_t n_here = min(kGridQueriesPerBlock, P->na - blk.y);
  const int lane = threadIdx.x, sub = lane & (kGroupLanes - 1), grp = lane / kGroupLanes;
  if (lane < n_here) segs[lane] = query_segment(v, P, pr, A, blk.y + lane);
  __syncthreads();
  int32_t* list = lists[grp];
  const int32_t* items = v.items + P->item_off;
  unsigned long long comparisons = 0;
  uint32_t accepted = 0;
  for (int32_t q0 = 0; q0 < n_here; q0 += 64 / kGroupLanes) {
    const bool live = q0 + grp < n_here;
    const int32_t q = min(q0 + grp, n_here - 1), i = blk.y + q;
    // The lane's two 16-byte chunks of the query's row.
    const int quad = sub & 3;
    const RowPart qr = row_part(A.desc, i, quad);
    const int32_t qn = A.norm2[i];
    int32_t d1 = kDistInf, j1 = 0x7FFFFFFF, d2 = kDistInf, taken = 0;
    auto consume = [&](int32_t count) {
      // Past the limit on |C'| the first found are kept (the error flag says so).
      count = min(count, kGridMaxCand - taken);
      // Sixteen candidates at a time, one a lane.
      if (count <= 0) return;
      int32_t jn = items[list[min(sub, count - 1)]];
      for (int32_t e0 = 0; e0 < count; e0 += kGroupLanes) {
        const int32_t j = jn;   // the next sixteen load meanwhile
        jn = items[list[min(e0 + kGroupLanes + sub, count - 1)]];
        const int32_t nb2 = B.norm2[j];
        const int32_t dot = quad_dots(qr, quad_rows(B.desc, j, quad), quad);
        const int32_t D = e0 + sub < count ? qn + nb2 - 2 * dot : kDistInf;
        const bool first = D < d1 || (D == d1 && j < j1);
        d2 = min(d2, first ? d1 : D);
        j1 = first ? j : j1;
        d1 = first ? D : d1;
      }
      taken += count;
    };
    int32_t found = 0;
    bool again = live;   // this query is to be walked (again)
    Sampler S(segs[q], live, P);
    for (int pass = 0; pass < 2; ++pass) {
      bool back;
      const int32_t n = walk<kGroupLanes>(v, P, S, list, sub, pass != 0, back, consume);
      if (again) found = n;
      again = again && pass == 0 && back;
      if (!__any(again)) break;
      S.K = again ? S.K : -1;
      if (again) {
        d1 = d2 = kDistInf;
        j1 = 0x7FFFFFFF;
        taken = 0;
      }
    }
    // The two smallest over the query's lanes, lowest index on ties.
#pragma unroll
    for (int o = 1; o < kGroupLanes; o <<= 1) {
      const int32_t e1 = __shfl_xor(d1, o, 64), ej = __shfl_xor(j1, o, 64);
      const int32_t e2 = __shfl_xor(d2, o, 64);
      const bool other = e1 < d1 || (e1 == d1 && ej < j1);
      d2 = min(min(d2, e2), max(d1, e1));
      j1 = other ? ej : j1;
      d1 = min(d1, e1);
    }
    if (sub == 0 && live) {
      if (found > kGridMaxCand) *v.err = 1;
      const int32_t n = taken;
      QueryResult r;
      r.match = n > 0 ? j1 : -1;
      r.d1 = n > 0 ? d1 : kDistInf;
      r.d2 = n > 1 ? d2 : kDistInf;
      bool accept = false;
      if (n >= 2)
        accept = int64_t(v.ratio_den) * r.d1 < int64_t(v.ratio_num) * r.d2;
      else if (n == 1)
        accept = v.accept_single != 0;
      r.flags = (accept ? 1 : 0) | (v.keep_counts ? (n << 1) : 0);
      v.res[q_off + i] = r;
      comparisons += uint32_t(n);
      accepted += accept ? 1u : 0u;
    }
  }
  for (int o = kGroupLanes; o < 64; o <<= 1) {
    comparisons += (unsigned long long)__shfl_xor((long long)comparisons, o, 64);
    accepted += uint32_t(__shfl_xor(int32_t(accepted), o, 64));
  }
  if (lane == 0) {
    if (comparisons) atomicAdd(&v.counters[pr].comparisons, comparisons);
    if (accepted) atomicAdd(&v.counters[pr].accepted, accepted);
  }
}

// ---------------------------------------------------------------------------
// Query grouping: queries whose lines cross b's box within tol of the
// previous line's crossings (in sorted order) share the first line's C'.
// ---------------------------------------------------------------------------

__device__ __forceinline__ int32_t pair_of(const int32_t* seg_begin, int32_t n_pairs, int32_t t) {
  int32_t lo = 0, hi = n_pairs - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (seg_begin[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Unsigned key with the order of the double (-0 first made +0).
__device__ __forceinline__ unsigned long long sortable(double x) {
  x = x + 0.0;
  const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(x));
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ __launch_bounds__(256) void grid_cross_kernel(GridView v, GroupView g) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.n) return;
  const int32_t pr = pair_of(g.seg_begin, v.n_pairs, t);
  const GridPair* P = v.pairs + pr;
  const ImageDev A = v.images[P->a];
  double xA = 0.0, yA = 0.0, xB = 0.0, yB = 0.0;
  const bool crosses = line_crossings(v, P, pr, A, int32_t(t - P->q_off), xA, yA, xB, yB);
  g.cross[4 * int64_t(t)] = xA;
  g.cross[4 * int64_t(t) + 1] = yA;
  g.cross[4 * int64_t(t) + 2] = xB;
  g.cross[4 * int64_t(t) + 3] = yB;
  g.hit[t] = crosses ? 1 : 0;
  g.val[0][t] = t;
}

// ---------------------------------------------------------------------------
// Least-significant-digit radix sort of the positions by (pair, A.x, A.y,
// B.x, B.y), the crossing components as 64-bit order-preserving keys (lines
// without a crossing sort last) and the pair index as the most significant
// key: 8-bit digits, least significant first, each pass a stable counting
// sort, so equal keys keep position order.  A pass counts the digits of each
// 2048-position tile, scans the counts (digit-major, so each digit's tiles
// follow each other), then sorts every tile by the digit in LDS (eight
// stable one-bit splits) and scatters it.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortPer = 8;                              // positions per thread
constexpr int kSortTile = kSortThreads * kSortPer;       // positions per tile
constexpr int kRadix = 256;

// Digit `byte` of the sort key `comp` (0..3: crossing component, 4: pair) of
// original position s.
__device__ __forceinline__ uint32_t sort_digit(const GridView& v, const GroupView& g, int32_t s,
                                               int comp, int byte) {
  unsigned long long key;
  if (comp < 4)
    key = g.hit[s] ? sortable(g.cross[4 * int64_t(s) + comp]) : ~0ull;
  else
    key = static_cast<unsigned long long>(pair_of(g.seg_begin, v.n_pairs, s));
  return uint32_t(key >> (8 * byte)) & (kRadix - 1);
}

// counts[d * ntiles + tile]: positions of the tile with digit d.
__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(GridView v, GroupView g,
                                                                  const int32_t* val, int comp,
                                                                  int byte, int32_t* counts,
                                                                  int32_t ntiles) {
  __shared__ int32_t h[kRadix];
  const int t = threadIdx.x;
  h[t] = 0;
  __syncthreads();
  const int32_t base = blockIdx.x * kSortTile;
  for (int k = 0; k < kSortPer; ++k) {
    const int32_t i = base + k * kSortThreads + t;
    if (i < g.n) atomicAdd(&h[sort_digit(v, g, val[i], comp, byte)], 1);
  }
  __syncthreads();
  counts[int64_t(t) * ntiles + blockIdx.x] = h[t];
}

// Exclusive scan of one value per thread over the block; returns the total.
__device__ __forceinline__ int32_t block_excl_scan(int32_t x, int32_t& total, int32_t* wsum) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int32_t inc = x;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  int32_t before = 0;
  total = 0;
  for (int w = 0; w < kSortThreads / 64; ++w) {
    before += w < wv ? wsum[w] : 0;
    total += wsum[w];
  }
  __syncthreads();
  return before + inc - x;
}

// One pass: the tile sorted stably by the digit, then every position written
// at (scanned count of its digit and tile) + (its rank among the tile's
// positions with that digit).
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(
    GridView v, GroupView g, const int32_t* val_in, int32_t* val_out, int comp, int byte,
    const int32_t* offsets, int32_t ntiles) {
  __shared__ int32_t sval[kSortTile];
  __shared__ uint8_t sdig[kSortTile];
  __shared__ int32_t dstart[kRadix];
  __shared__ int32_t wsum[kSortThreads / 64];
  const int t = threadIdx.x;
  const int32_t base = blockIdx.x * kSortTile;
  const int32_t cnt = min(kSortTile, g.n - base);
  // Thread t holds tile positions kSortPer t .. kSortPer t + kSortPer - 1.
  // Past the end: digit 255 and last in order, so they stay behind every
  // real position and are never written.
  int32_t vals[kSortPer];
  uint32_t dig[kSortPer];
#pragma unroll
  for (int k = 0; k < kSortPer; ++k) {
    const int32_t i = kSortPer * t + k;
    vals[k] = i < cnt ? val_in[base + i] : 0;
    dig[k] = i < cnt ? sort_digit(v, g, vals[k], comp, byte) : kRadix - 1;
  }
  for (int bit = 0; bit < 8; ++bit) {
    int32_t zeros = 0;
#pragma unroll
    for (int k = 0; k < kSortPer; ++k) zeros += ((dig[k] >> bit) & 1) ? 0 : 1;
    int32_t total_zeros;
    int32_t zb = block_excl_scan(zeros, total_zeros, wsum);   // zeros before this thread
    const int32_t first = kSortPer * t;
#pragma unroll
    for (int k = 0; k < kSortPer; ++k) {
      const bool one = (dig[k] >> bit) & 1;
      const int32_t pos = one ? total_zeros + (first + k - zb) : zb;
      zb += one ? 0 : 1;
      sval[pos] = vals[k];
      sdig[pos] = uint8_t(dig[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortPer; ++k) {
      vals[k] = sval[kSortPer * t + k];
      dig[k] = sdig[kSortPer * t + k];
    }
    __syncthreads();
  }
  // First tile position of each digit among the real positions.
  dstart[t] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortPer; ++k)
    if (kSortPer * t + k < cnt) atomicAdd(&dstart[dig[k]], 1);
  __syncthreads();
  int32_t total;
  const int32_t start = block_excl_scan(dstart[t], total, wsum);
  dstart[t] = start;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortPer; ++k) {
    const int32_t i = kSortPer * t + k;
    if (i < cnt)
      val_out[offsets[int64_t(dig[k]) * ntiles + blockIdx.x] + (i - dstart[dig[k]])] = vals[k];
  }
}

__global__ __launch_bounds__(256) void copy_i32_kernel(const int32_t* src, int32_t* dst,
                                                       int32_t n) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) dst[t] = src[t];
}

__global__ __launch_bounds__(256) void grid_stencil_kernel(GridView v, GroupView g) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.n) return;
  const int32_t pr = pair_of(g.seg_begin, v.n_pairs, t);
  int32_t start = 1;
  if (t > g.seg_begin[pr]) {
    const int32_t s = g.val[0][t], q = g.val[0][t - 1];
    if (g.hit[s] && g.hit[q]) {
      const double* a = g.cross + 4 * int64_t(s);
      const double* b = g.cross + 4 * int64_t(q);
      const double dA = (a[0] - b[0]) * (a[0] - b[0]) + (a[1] - b[1]) * (a[1] - b[1]);
      const double dB = (a[2] - b[2]) * (a[2] - b[2]) + (a[3] - b[3]) * (a[3] - b[3]);
      start = (dA > g.tol2 || dB > g.tol2) ? 1 : 0;
    }
  }
  g.stencil[t] = start;
}

// The same decision against the group's first line: a walk along each
// pair's sorted queries.  One wave per pair loads 64 positions at a time into
// LDS; its first lane then walks them in order, carrying the leader.
__global__ __launch_bounds__(64) void grid_stencil_leader_kernel(GridView v, GroupView g) {
  __shared__ double cx[64][4];
  __shared__ int32_t hs[64], out[64];
  const int32_t pr = blockIdx.x;
  const int lane = threadIdx.x;
  const int32_t* order = g.val[0];
  const int32_t begin = g.seg_begin[pr], end = g.seg_end[pr];
  bool have_lead = false, lead_hit = false;
  double L0 = 0.0, L1 = 0.0, L2 = 0.0, L3 = 0.0;
  for (int32_t base = begin; base < end; base += 64) {
    const int32_t t = base + lane;
    if (t < end) {
      const int32_t s = order[t];
      hs[lane] = g.hit[s];
#pragma unroll
      for (int c = 0; c < 4; ++c) cx[lane][c] = g.cross[4 * int64_t(s) + c];
    }
    __syncthreads();
    if (lane == 0) {
      const int32_t cnt = min(64, end - base);
      for (int32_t k = 0; k < cnt; ++k) {
        int32_t start = 1;
        if (have_lead && hs[k] && lead_hit) {
          const double dA = (cx[k][0] - L0) * (cx[k][0] - L0) + (cx[k][1] - L1) * (cx[k][1] - L1);
          const double dB = (cx[k][2] - L2) * (cx[k][2] - L2) + (cx[k][3] - L3) * (cx[k][3] - L3);
          start = (dA > g.tol2 || dB > g.tol2) ? 1 : 0;
        }
        if (start) {
          have_lead = true;
          lead_hit = hs[k] != 0;
          L0 = cx[k][0]; L1 = cx[k][1]; L2 = cx[k][2]; L3 = cx[k][3];
        }
        out[k] = start;
      }
    }
    __syncthreads();
    if (t < end) g.stencil[t] = out[lane];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void grid_gstart_kernel(GroupView g) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < g.n && g.stencil[t]) g.gstart[g.gid[t] - 1] = t;
}

__global__ __launch_bounds__(64) void grid_group_query_kernel(GridView v, GroupView g,
                                                              int32_t n_groups) {
  __shared__ int32_t cand[kGridMaxCand];
  __shared__ int32_t list[kListCap];
  __shared__ Segment seg;
  const int32_t gi = blockIdx.x;
  const int32_t t0 = g.gstart[gi], t1 = gi + 1 < n_groups ? g.gstart[gi + 1] : g.n;
  const int32_t pr = pair_of(g.seg_begin, v.n_pairs, t0);
  const GridPair* P = v.pairs + pr;
  const ImageDev A = v.images[P->a], B = v.images[P->b];
  const int64_t q_off = P->q_off;
  const int32_t* order = g.val[0];
  const int32_t* items = v.items + P->item_off;
  const int lane = threadIdx.x;
  if (lane == 0) seg = query_segment(v, P, pr, A, int32_t(order[t0] - q_off));
  __syncthreads();
  const Sampler S(seg, true, P);
  int32_t n = 0;
  auto consume = [&](int32_t count) {
    count = min(count, kGridMaxCand - n);
    for (int32_t e = lane; e < count; e += 64) cand[n + e] = items[list[e]];
    n += max(count, 0);
  };
  int32_t found = 0;
  for (int pass = 0; pass < 2; ++pass) {
    bool back;
    n = 0;
    found = walk<64>(v, P, S, list, lane, pass != 0, back, consume);
    if (!back) break;   // uniform
  }
  if (found > kGridMaxCand && lane == 0) *v.err = 1;
  __syncthreads();
  for (int32_t t = t0; t < t1; ++t) grid_decide(v, q_off, pr, A, B, int32_t(order[t] - q_off), cand, n);
}

int32_t blocks256(int32_t n) { return (n + 255) / 256; }

}  // namespace

// Radix-sort tile counts, then the scan's block sums (reused by the stencil
// scan).
static int32_t sort_tiles(int32_t n) { return (n + kSortTile - 1) / kSortTile; }

hipError_t grid_group_temp_bytes(int32_t n, int32_t n_pairs, size_t* bytes) {
  (void)n_pairs;
  const int64_t ncount = int64_t(kRadix) * sort_tiles(n);
  if (ncount > scan_limit() || int64_t(n) > scan_limit()) return hipErrorInvalidValue;
  *bytes = sizeof(int32_t) * size_t(ncount) + std::max(scan_temp_bytes(ncount), scan_temp_bytes(n));
  return hipSuccess;
}

hipError_t launch_grid_group_prepare(const GridView& v, const GroupView& g, hipStream_t st) {
  if (g.n <= 0) return hipSuccess;
  const int32_t ntiles = sort_tiles(g.n);
  const int64_t ncount = int64_t(kRadix) * ntiles;
  int32_t* counts = static_cast<int32_t*>(g.temp);
  int32_t* sums = counts + ncount;
  size_t need = 0;
  hipError_t e = grid_group_temp_bytes(g.n, v.n_pairs, &need);
  if (e != hipSuccess) return e;
  if (g.temp_bytes < need) return hipErrorInvalidValue;
  hipLaunchKernelGGL(grid_cross_kernel, dim3(blocks256(g.n)), dim3(256), 0, st, v, g);
  // Passes: every byte of components 3, 2, 1, 0, then the pair index's bytes.
  int pair_bytes = 0;
  while (pair_bytes < 4 && (int64_t(1) << (8 * pair_bytes)) < int64_t(v.n_pairs)) ++pair_bytes;
  int cur = 0;
  for (int comp = 3; comp >= -1; --comp) {
    const int key = comp >= 0 ? comp : 4;
    const int nbytes = comp >= 0 ? 8 : pair_bytes;
    for (int byte = 0; byte < nbytes; ++byte) {
      hipLaunchKernelGGL(sort_count_kernel, dim3(ntiles), dim3(kSortThreads), 0, st, v, g,
                         g.val[cur], key, byte, counts, ntiles);
      e = launch_scan(counts, counts, ncount, false, sums, nullptr, st);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(sort_scatter_kernel, dim3(ntiles), dim3(kSortThreads), 0, st, v, g,
                         g.val[cur], g.val[1 - cur], key, byte, counts, ntiles);
      cur = 1 - cur;
    }
  }
  if (cur != 0)
    hipLaunchKernelGGL(copy_i32_kernel, dim3(blocks256(g.n)), dim3(256), 0, st, g.val[1],
                       g.val[0], g.n);
  if (g.to_leader)
    hipLaunchKernelGGL(grid_stencil_leader_kernel, dim3(v.n_pairs), dim3(64), 0, st, v, g);
  else
    hipLaunchKernelGGL(grid_stencil_kernel, dim3(blocks256(g.n)), dim3(256), 0, st, v, g);
  e = launch_scan(g.stencil, g.gid, g.n, true, sums, nullptr, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(grid_gstart_kernel, dim3(blocks256(g.n)), dim3(256), 0, st, g);
  return hipGetLastError();
}

hipError_t launch_grid_groups(const GridView& v, const GroupView& g, int32_t n_groups,
                              hipStream_t st) {
  if (n_groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(grid_group_query_kernel, dim3(uint32_t(n_groups)), dim3(64), 0, st, v, g,
                     n_groups);
  return hipGetLastError();
}

hipError_t launch_grid(const GridView& v, int64_t n_blocks, hipStream_t st) {
  if (v.n_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL(grid_bin_kernel, dim3(v.n_pairs, v.strips), dim3(kBinThreads),
                     sizeof(int32_t) * size_t(v.strip_cells), st, v);
  if (n_blocks > 0)
    hipLaunchKernelGGL(grid_query_kernel, dim3(uint32_t(n_blocks)), dim3(64), 0, st, v);
  return hipGetLastError();
}

}  // namespace sfm
