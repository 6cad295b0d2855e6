// Guided matching of few pairs (a4-a6), without preparation: no geometry, no
// binning, no tiles.  Registration left b's features in spatial order, with a
// bounding box per 16 of them and one per 16 boxes.  Sixteen lanes take a query,
// four queries side by side in a wave:
//   - the lanes test 16 outer boxes at once against the band (a superset of the
//     exact test), then the 16 boxes of each outer box that it crosses, and
//     list the boxes hit in LDS;
//   - listed boxes are opened four at a time, one feature per lane: the FP32
//     test of eqs. (2)-(3) on centred coordinates, and FP64 on the caller's F
//     and the original keypoints for every slot within the margin of d (the
//     same operations as the binned form, so the same members and the same
//     borderline slots).  Each lane keeps its own members;
//   - the lanes' members are put into one list, each lane takes one of them, the
//     four lanes of a quad read their rows together, and the two smallest
//     distances are merged over the query's lanes (lowest index on ties).
// Whatever direction the lines have, also through an epipole inside the image,
// a line of an image of n features crosses about 2 sqrt(n / 16) boxes.
//
// What it is for: the binned form runs seven kernels, each of them 3.5 to 17 us
// on one pair however small, and scans all of b where the epipole is in the
// image.  Beyond some work per call the binned form wins, whose tiles share
// every candidate row among 16 to 128 queries where here each query reads its
// own (direct_pays in api.hip).
//
// Measured: a pair of 2,000 features 12.5 us (the call 27, binned 44), of 7,001
// with the epipole in the image 28 us (43 and 157), of 16,000 61 us (75 and 63:
// such a pair is binned).  Bound by the VALU and by chains of L2 reads; of the 61
// us the box tests take 22, the opened boxes 14, the distances 20.  A wave per
// query, with boxes of 64 features and scalar bookkeeping, took 62 us there and
// 130 instead of 75 on 37 pairs of 301 to 6,007 features.
#include <algorithm>
#include <cmath>

#include "line.h"
#include "sfm_internal.h"

namespace sfm {
namespace {

constexpr int kDirectWaves = 8;
constexpr int kLanes = 16;                      // lanes of a query
constexpr int kSide = 64 / kLanes;              // queries side by side
constexpr int kOpen = 4;                        // boxes opened together
constexpr int kLook = 4;                        // loads of box tests in flight together
constexpr int kBoxCap = 192;                    // boxes listed before they are opened
constexpr int kOwnCap = 24;                     // members a lane keeps before distances are computed
static_assert(kLanes == kBoxFeatures && kLanes == kOuterBoxes, "one feature, one box per lane");

// LDS of a wave (7.5 KB).
struct DirectLds {
  uint16_t own[kOwnCap][64];                    // members by lane: positions in spatial order
  uint16_t all[kSide][kLanes * kOwnCap];        // the same by query, without gaps
  uint16_t box[kSide][kBoxCap];
};

__device__ __forceinline__ double lane_double(double x, int lane) {
  const long long b = __double_as_longlong(x);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(b), lane));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(b >> 32), lane));
  return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}

__global__ __launch_bounds__(64 * kDirectWaves) __attribute__((amdgpu_waves_per_eu(4,4))) void direct_kernel(BatchView v, int32_t pb,
                                                                   int32_t per_wave) {
  __shared__ __attribute__((aligned(16))) DirectLds lds[kDirectWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int quad = lane & 3, sub = lane & (kLanes - 1), grp = lane / kLanes;
  const int32_t p = pb + int32_t(blockIdx.x);
  const PairDesc P = read_uniform(v.pairs, p);
  if (int32_t(blockIdx.y) * kDirectWaves * per_wave >= P.na) return;   // uniform
  const int32_t q0 = (int32_t(blockIdx.y) * kDirectWaves + wave) * per_wave;
  const ImageDev A = read_uniform(v.images, P.a), B = read_uniform(v.images, P.b);
  DirectLds& L = lds[wave];
  const double* F = v.F + 9 * int64_t(p);

  // F / ||F||, one entry per lane, then the line of query q0 + lane.
  double Fn[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) Fn[k] = ldg(F + k);
  const double fro = frobenius(Fn);
  const double mine = ldg(F + min(lane, 8)) / fro;
#pragma unroll
  for (int k = 0; k < 9; ++k) Fn[k] = lane_double(mine, k);
  const int32_t nq = max(0, min(per_wave, P.na - q0));
  const double ox = centre(B.bbox[0], B.bbox[2]), oy = centre(B.bbox[1], B.bbox[3]);
  float la = NAN, lb = NAN, lc = NAN;
  {
    const float2 xy = ldg_xy(A.xy, min(q0 + lane, P.na - 1));
    UnitLine l;
    if (unit_line(Fn, ox, oy, xy.x, xy.y, l)) {
      la = float(l.a);
      lb = float(l.b);
      lc = float(l.cc);
    }
  }
  const float lo = float(P.band - v.margin), hi = float(P.band + v.margin);
  const int32_t nouter = (P.nb + kOuterFeatures - 1) / kOuterFeatures;
  // Bound on the FP32 errors of the box test and of the slots' test (a few
  // roundings of terms no larger than the coordinates and the line's offset).
  const float extent = (B.bbox[2] - B.bbox[0]) + (B.bbox[3] - B.bbox[1]) + 2.0f;
  typedef float v4f __attribute__((ext_vector_type(4)));
  const v4f* outer = reinterpret_cast<const v4f*>(B.outer);
  const v4f* inner = reinterpret_cast<const v4f*>(B.box);

  uint32_t comparisons = 0, boxes = 0, borderline = 0, accepted = 0;   // of the lane's queries
  for (int32_t r = 0; r < nq; r += kSide) {
    const bool live = r + grp < nq;
    const int32_t q = min(r + grp, nq - 1), i = q0 + q;
    const float a = __shfl(la, q, 64), b = __shfl(lb, q, 64), c = __shfl(lc, q, 64);
    const RowPart qr = row_part(A.desc, i, quad);
    const int32_t qn = ldg(A.norm2 + i);
    const float reach = hi + 1e-3f + 4e-6f * (fabsf(c) + extent);
    const float fa = fabsf(a), fb = fabsf(b);
    // Kept unless it is certain that no feature of the box is in the band.  A
    // degenerate line (NaN) has none.
    auto crossed = [&](const v4f& x) {
      const float e = band_dist32(a, b, c, x.x, x.y);
      return !(e > __builtin_fmaf(fa, x.z, __builtin_fmaf(fb, x.w, reach))) && a == a && live;
    };
    // This query's lanes for which x holds, as the low 16 bits.
    auto lanes_of = [&](bool x) {
      const unsigned long long m = __ballot(x);
      const uint32_t h = grp & 2 ? uint32_t(m >> 32) : uint32_t(m);
      return grp & 1 ? h >> 16 : h & 0xFFFFu;
    };
    int32_t d1 = kDistInf, j1 = 0x7FFFFFFF, d2 = kDistInf;
    int32_t total = 0;            // members so far
    int32_t own = 0;              // members this lane keeps
    int32_t nbox = 0, opened = 0; // boxes listed, and opened of them
    unsigned long long hit = 0;   // outer boxes still to look into, of 64 ...
    int32_t from = -kLook * kLanes;   // ... from this one
    bool done = false;            // uniform: every outer box has been looked into
    for (;;) {
      // List boxes.
      while (!done && !__any(nbox > kBoxCap - kLook * kLanes)) {
        if (!__any(hit != 0)) {
          from += kLook * kLanes;
          if (from >= nouter) {
            done = true;
            break;
          }
          v4f x[kLook];
#pragma unroll
          for (int u = 0; u < kLook; ++u) x[u] = ldg(outer + min(from + kLanes * u + sub, nouter - 1));
#pragma unroll
          for (int u = 0; u < kLook; ++u)
            hit |= (unsigned long long)lanes_of(crossed(x[u]) && from + kLanes * u + sub < nouter)
                   << (kLanes * u);
          continue;
        }
        int32_t k[kLook];
        bool use[kLook];
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
          use[u] = hit != 0;
          k[u] = (from + (use[u] ? __builtin_ctzll(hit) : 0)) * kOuterBoxes + sub;
          hit &= hit - 1;   // of 0: 0
        }
        v4f x[kLook];
#pragma unroll
        for (int u = 0; u < kLook; ++u) x[u] = ldg(inner + k[u]);
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
          const uint32_t m = lanes_of(crossed(x[u]) && use[u]);
          if ((m >> sub) & 1u)
            L.box[grp][nbox + __builtin_popcount(m & ((1u << sub) - 1u))] = uint16_t(k[u]);
          nbox += __builtin_popcount(m);
        }
      }
      wave_lds_fence();
      // Open them.
      bool full = false;
      int32_t at_next[kOpen];
      float2 xy_next[kOpen];
      auto load_open = [&]() {   // the boxes from `opened` on
#pragma unroll
        for (int u = 0; u < kOpen; ++u) {
          const int32_t k = L.box[grp][max(min(opened + u, nbox - 1), 0)];
          at_next[u] = (nbox > 0 ? k : 0) * kBoxFeatures + sub;
        }
#pragma unroll
        for (int u = 0; u < kOpen; ++u)
          xy_next[u] = ldg_xy(reinterpret_cast<const float*>(B.sxy), at_next[u]);
      };
      if (nouter > 0) load_open();
      while (__any(opened < nbox)) {
        full = __any(own > kOwnCap - kOpen);
        if (full) break;
        int32_t at[kOpen];
        float2 xy[kOpen];
#pragma unroll
        for (int u = 0; u < kOpen; ++u) {
          at[u] = at_next[u];
          xy[u] = xy_next[u];
        }
        const int32_t first = opened;
        opened += kOpen;
        load_open();   // the next boxes load meanwhile
        bool near = false;
#pragma unroll
        for (int u = 0; u < kOpen; ++u) {
          const float e = band_dist32(a, b, c, xy[u].x, xy[u].y);
          const bool use = first + u < nbox, in = use && e <= lo;
          near |= use && e <= hi && !in;
          if (in) L.own[own][lane] = uint16_t(at[u]);
          own += in ? 1 : 0;
        }
        if (__any(near)) {
          // Rare: slots within the margin of d, decided in FP64.
#pragma unroll
          for (int u = 0; u < kOpen; ++u) {
            const float e = band_dist32(a, b, c, xy[u].x, xy[u].y);
            if (first + u < nbox && e <= hi && !(e <= lo)) {
              ++borderline;
              const int32_t j = ldg(B.sj + at[u]);
              const float2 xq = ldg_xy(A.xy, i), xb = ldg_xy(B.xy, j);
              if (band_dist64(F, xq.x, xq.y, xb.x, xb.y) <= P.band) L.own[own++][lane] = uint16_t(at[u]);
            }
          }
        }
      }
      if (!full) {
        boxes += sub == 0 ? uint32_t(nbox) : 0u;
        nbox = opened = 0;
        if (!done) continue;
      }
      // The members' distances: first one list per query.
      int32_t inc = own;
#pragma unroll
      for (int o = 1; o < kLanes; o <<= 1) {
        const int32_t y = __shfl_up(inc, o, kLanes);
        if (sub >= o) inc += y;
      }
      const int32_t count = __shfl(inc, kLanes - 1, kLanes);
      for (int32_t t = 0; t < own; ++t) L.all[grp][inc - own + t] = L.own[t][lane];
      wave_lds_fence();
      if (count > 0) {
        int32_t jn = ldg(B.sj + L.all[grp][min(sub, count - 1)]);
        for (int32_t e0 = 0; e0 < count; e0 += kLanes) {
          const int32_t j = jn;   // the next sixteen's indices load meanwhile
          jn = ldg(B.sj + L.all[grp][min(e0 + kLanes + sub, count - 1)]);
          const int32_t nb2 = ldg(B.norm2 + j);
          const int32_t dot = quad_dots(qr, quad_rows(B.desc, j, quad), quad);
          const int32_t D = e0 + sub < count ? qn + nb2 - 2 * dot : kDistInf;
          const bool better = D < d1 || (D == d1 && j < j1);
          d2 = min(d2, better ? d1 : D);
          j1 = better ? j : j1;
          d1 = better ? D : d1;
        }
      }
      wave_lds_fence();
      total += count;
      own = 0;
      if (done && !full) break;
    }
    // Smallest distance, its lowest index, and the smallest of all others.
#pragma unroll
    for (int o = 1; o < kLanes; o <<= 1) {
      const int32_t e1 = __shfl_xor(d1, o, 64), ej = __shfl_xor(j1, o, 64);
      const int32_t e2 = __shfl_xor(d2, o, 64);
      const bool other = e1 < d1 || (e1 == d1 && ej < j1);
      d2 = min(min(d2, e2), max(d1, e1));
      j1 = other ? ej : j1;
      d1 = min(d1, e1);
    }
    if (sub == 0 && live) {
      bool accept = false;
      if (total >= 2)
        accept = int64_t(v.ratio_den) * d1 < int64_t(v.ratio_num) * d2;
      else if (total == 1)
        accept = v.accept_single != 0;
      QueryResult res;
      res.match = total > 0 ? j1 : -1;
      res.d1 = total > 0 ? d1 : kDistInf;
      res.d2 = total > 1 ? d2 : kDistInf;
      res.flags = (accept ? 1 : 0) | (v.keep_counts ? (total << 1) : 0);
      v.res[P.q_off + i] = res;
      comparisons += uint32_t(total);
      accepted += accept ? 1u : 0u;
    }
  }
  // One addition per workgroup: the pair's counters share a cache line, and an
  // addition per wave (8,000 for a pair of 2,000 queries) took 57 us.
  __shared__ unsigned long long sums[4];
  if (threadIdx.x < 4) sums[threadIdx.x] = 0;
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) {
    comparisons += uint32_t(__shfl_xor(int32_t(comparisons), o, 64));
    boxes += uint32_t(__shfl_xor(int32_t(boxes), o, 64));
    borderline += uint32_t(__shfl_xor(int32_t(borderline), o, 64));
    accepted += uint32_t(__shfl_xor(int32_t(accepted), o, 64));
  }
  if (lane == 0 && nq > 0) {
    atomicAdd(&sums[0], (unsigned long long)comparisons);
    atomicAdd(&sums[1], (unsigned long long)boxes * kBoxFeatures);
    atomicAdd(&sums[2], (unsigned long long)borderline);
    atomicAdd(&sums[3], (unsigned long long)accepted);
  }
  __syncthreads();
  PairCounters* C = v.counters + p;
  if (threadIdx.x == 0 && sums[0]) atomicAdd(&C->comparisons, sums[0]);
  if (threadIdx.x == 1 && sums[1]) atomicAdd(&C->elements, sums[1]);
  if (threadIdx.x == 2 && sums[2]) atomicAdd(&C->borderline, sums[2]);
  if (threadIdx.x == 3 && sums[3]) atomicAdd(&C->accepted, uint32_t(sums[3]));
}

}  // namespace

// Queries of a wave, in fours: 16 waves per CU before a wave takes more.
int32_t direct_queries(int64_t total_queries) {
  const int64_t fours = (total_queries + 4 * 4096 - 1) / (4 * 4096);
  return 4 * int32_t(std::min<int64_t>(16, std::max<int64_t>(1, fours)));
}

hipError_t launch_direct(const BatchView& v, int32_t pb, int32_t pc, int32_t max_queries,
                         int32_t per_wave, hipStream_t st) {
  if (pc <= 0 || max_queries <= 0) return hipSuccess;
  const int32_t per_block = kDirectWaves * per_wave;
  // Pairs along x, which takes any number of them (y ends at 65,535).
  hipLaunchKernelGGL(direct_kernel, dim3(pc, (max_queries + per_block - 1) / per_block),
                     dim3(64 * kDirectWaves), 0, st, v, pb, per_wave);
  return hipGetLastError();
}

}  // namespace sfm
