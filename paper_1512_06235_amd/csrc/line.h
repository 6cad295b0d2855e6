// Device functions of the epipolar line and the band test, shared by the binned
// and the direct form of guided matching: both must take the same FP32 line and
// distance of a slot, so that they count the same borderline slots.
#pragma once

#include <hip/hip_runtime.h>

#include "sfm_internal.h"

namespace sfm {

// A global load through an address-space-1 pointer: the pointers used with it
// come from records, and the flat loads the compiler would otherwise emit also
// count against the LDS counter, so each would be waited for alone.
template <class T>
__device__ __forceinline__ T ldg(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}

// Two floats, 4-byte aligned (keypoints are the caller's).
__device__ __forceinline__ float2 ldg_xy(const float* xy, int64_t i) {
  typedef float v2f __attribute__((ext_vector_type(2), aligned(4)));
  const v2f p = *(const __attribute__((address_space(1))) v2f*)(xy + 2 * i);
  return make_float2(p.x, p.y);
}

// ||F||_F.
__device__ __forceinline__ double frobenius(const double* F) {
  double fro = 0.0;
  for (int k = 0; k < 9; ++k) fro += F[k] * F[k];
  return sqrt(fro);
}

// Origin of the centred FP32 coordinates of an image, one axis of its box.
__device__ __forceinline__ double centre(double lo, double hi) { return floor(0.5 * (lo + hi)); }

// The line l = F (x, y, 1)^T with a unit normal, and its offset on coordinates
// centred at (ox, oy); false when it is degenerate (no feature is in its band).
struct UnitLine {
  double a, b, c, cc;
};
__device__ __forceinline__ bool unit_line(const double* F, double ox, double oy, float xq, float yq,
                                          UnitLine& l) {
  const double x = xq, y = yq;
  double a = F[0] * x + F[1] * y + F[2];
  double b = F[3] * x + F[4] * y + F[5];
  double c = F[6] * x + F[7] * y + F[8];
  const double s = sqrt(a * a + b * b);
  if (!(s > 0.0) || !isfinite(s) || !isfinite(c)) return false;
  const double inv_s = 1.0 / s;
  a *= inv_s; b *= inv_s; c *= inv_s;
  l.a = a;
  l.b = b;
  l.c = c;
  l.cc = c + a * ox + b * oy;
  return true;
}

// Epipolar distance of eqs. (2)-(3) on centred FP32 coordinates,
// |a x + b y + c| with (a, b) unit.  The single FP32 evaluation every pass uses.
__device__ __forceinline__ float band_dist32(float a, float b, float c, float x, float y) {
  return __builtin_fabsf(__builtin_fmaf(a, x, __builtin_fmaf(b, y, c)));
}

// The epipolar distance of eqs. (2)-(3) in FP64, on the caller's F and the
// original keypoints, every operation as written (no contraction): the line
// l = F (x, y, 1)^T row by row, s = sqrt(l0^2 + l1^2), then
// |l0 x' + l1 y' + l2| / s.  NaN when s = 0 or s or l2 is not finite (such a
// line has no candidates).
__device__ __forceinline__ double band_dist64(const double* F, float xq, float yq, float xb,
                                           float yb) {
#pragma clang fp contract(off)
  const double x = xq, y = yq;
  double f[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) f[k] = ldg(F + k);
  const double a = f[0] * x + f[1] * y + f[2];
  const double b = f[3] * x + f[4] * y + f[5];
  const double c = f[6] * x + f[7] * y + f[8];
  const double s = sqrt(a * a + b * b);
  const bool line = s > 0.0 && isfinite(s) && isfinite(c);
  // Computed either way and selected, so the loads of (xb, yb) are not
  // moved into a branch behind this one's.
  const double e = fabs(a * double(xb) + b * double(yb) + c) / s;
  return line ? e : NAN;
}

// Entry i (uniform) of a table that the kernel only reads, by scalar loads.
template <class T>
__device__ __forceinline__ T read_uniform(const T* table, int32_t i) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  typedef const __attribute__((address_space(4))) int32_t c_i32;
  c_i32* src = (c_i32*)(table + __builtin_amdgcn_readfirstlane(i));
  union {
    int32_t w[sizeof(T) / 4];
    T t;
  } u;
#pragma unroll
  for (int k = 0; k < int(sizeof(T) / 4); ++k) u.w[k] = src[k];
  return u.t;
}

// Within each four lanes: lane u's value; the value of lane ^ 1; of lane ^ 2.
__device__ __forceinline__ int32_t quad_lane(int32_t x, int u) {
  switch (u) {
    case 0: return __builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, true);
    case 1: return __builtin_amdgcn_mov_dpp(x, 0x55, 0xF, 0xF, true);
    case 2: return __builtin_amdgcn_mov_dpp(x, 0xAA, 0xF, 0xF, true);
    default: return __builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, true);
  }
}
__device__ __forceinline__ int32_t quad_swap1(int32_t x) {
  return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);
}
__device__ __forceinline__ int32_t quad_swap2(int32_t x) {
  return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);
}

// A query's row as the four lanes of a quad hold it: 16-byte chunks `quad` and
// `quad + 4` in lane quad.
struct RowPart {
  uint4 a, b;
};
__device__ __forceinline__ RowPart row_part(const uint8_t* desc, int64_t i, int quad) {
  typedef unsigned int v4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(1))) v4 g_v4;
  g_v4* row = (g_v4*)(desc + kDescBytes * i) + quad;
  const v4 x = row[0], y = row[4];
  return {{x.x, x.y, x.z, x.w}, {y.x, y.y, y.z, y.w}};
}

// Dot products of the query with four candidates per quad, one of them (row j
// of desc) per lane: the four lanes read each row together, 64 bytes a load (a
// lane that reads whole rows asks the L2 for every line eight times), and sum
// their parts.  Every lane of a quad must be active.
struct QuadRows {
  RowPart r[4];
};
__device__ __forceinline__ QuadRows quad_rows(const uint8_t* desc, int32_t j, int quad) {
  QuadRows q;
#pragma unroll
  for (int u = 0; u < 4; ++u) q.r[u] = row_part(desc, quad_lane(j, u), quad);
  return q;
}
__device__ __forceinline__ int32_t quad_dots(const RowPart& q, const QuadRows& rows, int quad) {
  int32_t dot = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const RowPart& r = rows.r[u];
    uint32_t s = 0;
    s = __builtin_amdgcn_udot4(r.a.x, q.a.x, s, false);
    s = __builtin_amdgcn_udot4(r.a.y, q.a.y, s, false);
    s = __builtin_amdgcn_udot4(r.a.z, q.a.z, s, false);
    s = __builtin_amdgcn_udot4(r.a.w, q.a.w, s, false);
    s = __builtin_amdgcn_udot4(r.b.x, q.b.x, s, false);
    s = __builtin_amdgcn_udot4(r.b.y, q.b.y, s, false);
    s = __builtin_amdgcn_udot4(r.b.z, q.b.z, s, false);
    s = __builtin_amdgcn_udot4(r.b.w, q.b.w, s, false);
    s += uint32_t(quad_swap1(int32_t(s)));
    s += uint32_t(quad_swap2(int32_t(s)));
    dot = quad == u ? int32_t(s) : dot;
  }
  return dot;
}

// Keeps the compiler from moving a wave's LDS accesses across this point (a
// wave's LDS accesses are carried out in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace sfm
