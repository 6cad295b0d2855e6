// Exhaustive two-nearest matching: every feature of b is a candidate of every
// query of a (the band of eqs. (2)-(3) ignored).  The comparison point of
// Section 6 and the matcher of both stages of staged coarse matching (Section 4).
//
// Work item: (pair, block of 256 queries, slice of up to 1024 targets starting
// at a multiple of 1024).  A workgroup of four waves takes one item:
//   - Wave w owns queries 64 w .. 64 w + 63 of the block as four 16-query
//     tiles; their rows, as signed bytes 127 - 2 q, are the resident B operands
//     of v_mfma_i32_16x16x64_i8 (two per tile: bytes 0..63 and 64..127).
//   - The slice's rows stream through two LDS buffers of 128 targets by LDS
//     DMA (rows XOR-swizzled: chunk c of row r at slot c ^ (r & 7)); the next
//     buffer loads while the current one is used, one barrier per buffer.
//     Targets past n_b read a zero row, so their products are 0.
//   - Per 16-target step: eight MFMAs, whose C operand is each target's
//     constant term ||c||^2 - 127 sum(c) + 2^21 (from registration), give
//         ||c||^2 - 2 q.c + 2^21
//     for 16 targets x 64 queries: sum((127 - 2 q) c) = 127 sum(c) - 2 q.c.
//     Each lane takes the smallest of its four results per tile (v_min,
//     v_min3) and folds it into its two smallest group keys
//         (distance << 10) | (target mod 1024) / 4
//     with v_lshl_add, v_med3 and v_min: 1.25 VALU instructions a comparison.
//     A group is four consecutive targets of one lane, so groups order like
//     their targets.  (Padding targets carry the largest distance.)
// The slice's two smallest group keys of every query go to a partial-result
// array; the merge kernel folds a query's slices in ascending order and looks
// into the best group for the match and the second smallest distance.
//
// What bounds it: the matrix core and the VALU share most of an MFMA's
// cycles (beside eight MFMAs about eight VALU instructions issue for free,
// each further one costs its own cycles), and LDS operands add to that.  With
// the key of every single product (v_lshl_add, v_med3, v_min: three VALU
// instructions a comparison) the 16,000 x 16,000 pair took 46.0 us and a
// staged launch of 1,770 pairs 352 us; with group keys 34 and 250 us.  Eight
// tiles a wave halve the LDS reads but leave two waves a SIMD: 34 and 317 us.
#include <algorithm>

#include "line.h"
#include "sfm_internal.h"

namespace sfm {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int nv4u __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) nv4u g_nv4u;
typedef const __attribute__((address_space(1))) int32_t g_i32;
typedef int v2i __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) v2i g_v2i;
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) v2u g_v2u;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kExWaves = 4;
constexpr int kExTiles = 4;                                    // 16-query tiles per wave
constexpr int32_t kExQueries = kExWaves * kExTiles * kQueryTile;   // queries per work item
constexpr int32_t kExSlice = kChunk;                           // targets per work item
constexpr int kExBuf = 128;                                    // targets per LDS buffer
constexpr int kExRowsPerWave = kExBuf / kExWaves;              // rows one wave fetches per buffer
constexpr int kExSteps = kExBuf / kQueryTile;                  // 16-target steps per buffer
static_assert(kExQueries == 256 && kExSlice == 1024, "the size limits of item indices");
static_assert(int64_t(kExhaustiveMaxQueries) <= int64_t(32767) * kExQueries &&
                  int64_t(kExhaustiveMaxTargets) <= int64_t(65535) * kExSlice,
              "query blocks fit 15 bits, slices 16");
static_assert(kExSlice % kExBuf == 0 && kExBuf % kQueryTile == 0, "whole steps per buffer");
static_assert(kExRowsPerWave % 8 == 0, "one DMA instruction fetches eight rows");
constexpr uint32_t kExKeyDistInf = kKeyInf >> kPosBits;

// Two buffers of rows and keys' norm words: 33 KB, four workgroups per CU.
struct ExLds {
  uint8_t rows[2][kExBuf * kDescBytes];
  uint32_t nc[2][kExBuf];
};
static_assert(sizeof(ExLds) <= 40960, "four workgroups per CU");

// The DMA source of targets past n_b.
__device__ __attribute__((aligned(16))) const uint8_t zero_row[kDescBytes] = {};

__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

// Waits for all of this wave's vector-memory operations (LDS DMA included).
__device__ __forceinline__ void wait_all_loads() {
  compiler_fence();
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), expcnt and lgkmcnt untouched
  compiler_fence();
}

__device__ __forceinline__ void barrier() {
  compiler_fence();
  __builtin_amdgcn_s_barrier();
  compiler_fence();
}

// LDS DMA of 16 bytes per lane: lane l's bytes at src land at LDS offset
// lds_off + 16 l (lds_off wave-uniform).  Inline asm with M0 set in the same
// statement; the kernel orders these writes itself (wait_all_loads, barrier).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void* src, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(__builtin_amdgcn_readfirstlane(lds_off)), "v"(src) : "memory", "m0");
}
// The same with a uniform base address in SGPRs plus a 32-bit lane offset:
// no per-lane address arithmetic.
__device__ __forceinline__ void dma16s(const void* base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(__builtin_amdgcn_readfirstlane(lds_off)), "v"(voff), "s"(base)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// 127 - 2 q of four bytes q in 0..127, as signed bytes.
__device__ __forceinline__ int query_bytes(uint32_t w) { return int((w << 1) ^ 0x7F7F7F7Fu); }

__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));   // selects v_med3_u32
}

// Rows of targets t .. t + kExBuf - 1 into the buffer at LDS offset
// lds_rows: wave w fetches rows
// kExRowsPerWave w .. + kExRowsPerWave - 1, eight per instruction (lane l:
// row 8 u + (l >> 3), chunk (l & 7) ^ (row & 7), landing at slot l & 7).
// A buffer wholly inside b takes the base-address form: the lane's offset
// voff = (kExRowsPerWave w + (l >> 3)) * 128 + 16 ((l & 7) ^ (l >> 3)) is the
// same for every buffer and instruction (row 8 u + (l >> 3) of the wave's
// rows: the base advances by 8 rows per instruction).
__device__ __forceinline__ void issue_rows(const uint8_t* b_desc, int32_t nb, int32_t t,
                                           uint32_t lds_rows, uint32_t voff, int w, int lane) {
  const uint32_t lw = lds_rows + uint32_t(kExRowsPerWave * w * kDescBytes);
  if (t + kExBuf <= nb) {
    const uint8_t* base = b_desc + int64_t(t) * kDescBytes;
#pragma unroll
    for (int u = 0; u < kExRowsPerWave / 8; ++u)
      dma16s(base + 8 * u * kDescBytes, voff, lw + uint32_t(8 * u * kDescBytes));
    return;
  }
#pragma unroll
  for (int u = 0; u < kExRowsPerWave / 8; ++u) {
    const int r = kExRowsPerWave * w + 8 * u + (lane >> 3);
    const int c = (lane & 7) ^ (r & 7);
    const int32_t j = t + r;
    const uint8_t* src = j < nb ? b_desc + int64_t(j) * kDescBytes + 16 * c : zero_row + 16 * c;
    dma16(src, lw + uint32_t(8 * u * kDescBytes));
  }
}

// The constant term of target j of the slice (threads 0 .. kExBuf - 1 of the
// workgroup, one target each); past n_b the largest distance.
__device__ __forceinline__ uint32_t const_term(const int32_t* cword, int32_t nb, int32_t j) {
  const int32_t c = ((g_i32*)cword)[min(j, nb - 1)];
  return j < nb ? uint32_t(c) : kExKeyDistInf;
}

// One step's LDS operands: the lane's chunks of both k-halves of its target
// row and the constant terms of its four targets.
struct StepIn {
  v4i a0, a1, c;
};
__device__ __forceinline__ StepIn read_step(const uint8_t* a0p, const uint8_t* a1p,
                                            const uint32_t* cp) {
  return {*reinterpret_cast<const v4i*>(a0p), *reinterpret_cast<const v4i*>(a1p),
          *reinterpret_cast<const v4i*>(cp)};
}

// Eight MFMAs of one step: the biased key distances of 16 targets and the
// wave's four query tiles (the constant terms enter as the C operand).
__device__ __forceinline__ void mfma_step(const StepIn& in, const v4i (&bq)[kExTiles][2],
                                          v4i (&acc)[kExTiles]) {
#pragma unroll
  for (int k = 0; k < kExTiles; ++k)
    acc[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(in.a0, bq[k][0], in.c, 0, 0, 0);
#pragma unroll
  for (int k = 0; k < kExTiles; ++k)
    acc[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(in.a1, bq[k][1], acc[k], 0, 0, 0);
}

// The smallest of the lane's four distances per tile, as one group key, into
// the two smallest (gid: the group's index in the slice).
__device__ __forceinline__ void fold_step(uint32_t gid, const v4i (&acc)[kExTiles],
                                          uint32_t (&k1)[kExTiles], uint32_t (&k2)[kExTiles]) {
#pragma unroll
  for (int k = 0; k < kExTiles; ++k) {
    const uint32_t m = min(min(min(uint32_t(acc[k][0]), uint32_t(acc[k][1])), uint32_t(acc[k][2])),
                           uint32_t(acc[k][3]));
    const uint32_t key = (m << kPosBits) + gid;
    k2[k] = umed3(k1[k], key, k2[k]);
    k1[k] = min(k1[k], key);
  }
}

// Asks the scheduler for one step's MFMAs with the previous step's fold
// between them (one MFMA keeps the matrix core busy for as long as four VALU
// instructions issue), so a wave overlaps the two itself.
__device__ __forceinline__ void interleave_step() {
  __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);     // the LDS reads
#pragma unroll
  for (int k = 0; k < 2 * kExTiles; ++k) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);   // three VALU
  }
}

// Whether pair p takes part in the launch (its predecessor's counters are an
// earlier launch's).
__device__ __forceinline__ bool stage_open(const BatchView& v, const ExStage& stage, int32_t p) {
  return !stage.gated || stage.open(v.counters[p - 1].accepted);
}

__global__ __launch_bounds__(64 * kExWaves) __attribute__((amdgpu_waves_per_eu(4, 8)))
void exhaustive_kernel(BatchView v, ExStage stage, const int2* items, int32_t n_items,
                       uint2* part) {
  __shared__ __attribute__((aligned(128))) ExLds lds;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tid = threadIdx.x;
  // The per-pair counters the merge kernel adds its accepted queries to:
  // workgroup k sets 256 of the stage's pairs.
  {
    const int64_t at = stage.first + (int64_t(blockIdx.x) * (64 * kExWaves) + tid) * stage.step;
    if (at < v.n_pairs) {
      const int32_t p = int32_t(at);
      const PairDesc P = v.pairs[p];
      const int64_t nqb = (P.na + kExQueries - 1) / kExQueries;
      const int64_t tail = P.nb - int64_t(kExSlice) * ((P.nb - 1) / kExSlice);
      PairCounters c;
      c.comparisons = (unsigned long long)(int64_t(P.na) * P.nb);
      c.elements = P.nb > 0 ? (unsigned long long)(nqb * kExQueries *
                                                   (P.nb - tail + ((tail + 15) & ~int64_t(15))))
                            : 0ull;
      c.borderline = 0;
      c.accepted = 0;
      c.ties = 0;
      if (!stage_open(v, stage, p)) c.comparisons = c.elements = 0;
      v.counters[p] = c;
    }
  }
  if (int32_t(blockIdx.x) >= n_items) return;
  const v2i it = ((g_v2i*)items)[blockIdx.x];
  const int32_t p = __builtin_amdgcn_readfirstlane(it.x);
  if (!stage_open(v, stage, p)) return;   // uniform
  const int32_t qb = __builtin_amdgcn_readfirstlane(it.y) >> 16;
  const int32_t s = __builtin_amdgcn_readfirstlane(it.y) & 0xFFFF;
  const PairDesc P = v.pairs[p];
  const ImageDev A = v.images[P.a], B = v.images[P.b];
  const int32_t t0 = s * kExSlice;
  const int32_t cnt = min(kExSlice, P.nb - t0);
  const int32_t nfill = (cnt + kExBuf - 1) / kExBuf;
  const uint32_t lbase = uint32_t(reinterpret_cast<uintptr_t>((lds_void*)&lds));
  const uint32_t lrows = lbase + uint32_t(offsetof(ExLds, rows));

  // The first buffer, the wave's query rows and the first norm words.
  const uint32_t voff = uint32_t((kExRowsPerWave * w + (lane >> 3)) * kDescBytes +
                                 16 * ((lane & 7) ^ ((lane >> 3) & 7)));
  issue_rows(B.desc, P.nb, t0, lrows, voff, w, lane);
  const int col = lane & (kQueryTile - 1), g = lane >> 4;
  const int32_t qw = qb * kExQueries + kExTiles * kQueryTile * w;   // the wave's first query
  nv4u qr[kExTiles][2];
#pragma unroll
  for (int k = 0; k < kExTiles; ++k) {
    const int32_t i = min(qw + kQueryTile * k + col, P.na - 1);
    const uint8_t* row = A.desc + int64_t(i) * kDescBytes + 16 * g;
    qr[k][0] = *(g_nv4u*)row;
    qr[k][1] = *(g_nv4u*)(row + 64);
  }
  uint32_t nw = tid < kExBuf ? const_term(B.cword, P.nb, t0 + tid) : 0u;
  if (tid < kExBuf) lds.nc[0][tid] = nw;
  v4i bq[kExTiles][2];
#pragma unroll
  for (int k = 0; k < kExTiles; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      bq[k][h] = v4i{query_bytes(qr[k][h].x), query_bytes(qr[k][h].y), query_bytes(qr[k][h].z),
                     query_bytes(qr[k][h].w)};
  uint32_t k1[kExTiles], k2[kExTiles];
#pragma unroll
  for (int k = 0; k < kExTiles; ++k) k1[k] = k2[k] = kKeyInf;
  wait_all_loads();
  barrier();

  for (int32_t f = 0; f < nfill; ++f) {
    const int cur = f & 1;
    const int32_t tf = t0 + kExBuf * f;   // first target of this buffer
    const bool more = f + 1 < nfill;
    // The next buffer: its rows by DMA, its norm words into a register.
    if (more) {
      issue_rows(B.desc, P.nb, tf + kExBuf, lrows + uint32_t((cur ^ 1) * kExBuf * kDescBytes),
                 voff, w, lane);
      if (tid < kExBuf) nw = const_term(B.cword, P.nb, tf + kExBuf + tid);
    }
    // A wave whose queries all lie past n_a only fetches its share of the
    // buffers and meets the barriers.
    const int32_t nsteps =
        qw < P.na ? (min(kExBuf, t0 + cnt - tf) + kQueryTile - 1) / kQueryTile : 0;
    // Step i: A operand from buffer row 16 i + col, k-slices g and g + 4
    // (chunk slots g ^ (row & 7) and that ^ 4); constant terms of rows
    // 16 i + 4 g .. + 3.  A whole buffer runs unrolled: step i + 2's operands
    // are read and step i + 1's MFMAs issued around step i's fold.  A partial
    // buffer (the end of b) runs step by step.
    const uint8_t* r0 = lds.rows[cur] + col * kDescBytes + ((g ^ (col & 7)) << 4);
    const uint8_t* r1 = lds.rows[cur] + col * kDescBytes + (((g ^ (col & 7)) ^ 4) << 4);
    const uint32_t* cp = lds.nc[cur] + 4 * g;
    constexpr int kStepBytes = kQueryTile * kDescBytes;
    const uint32_t gid0 = uint32_t((kExBuf / 4) * f + g);   // the lane's group of step 0
    if (nsteps == kExSteps) {
      v4i acc[2][kExTiles];
      StepIn in = read_step(r0, r1, cp);
      mfma_step(in, bq, acc[0]);
      in = read_step(r0 + kStepBytes, r1 + kStepBytes, cp + kQueryTile);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kExSteps; ++i) {
        StepIn next = in;
        if (i + 2 < kExSteps)
          next = read_step(r0 + (i + 2) * kStepBytes, r1 + (i + 2) * kStepBytes,
                           cp + (i + 2) * kQueryTile);
        if (i + 1 < kExSteps) mfma_step(in, bq, acc[(i + 1) & 1]);
        fold_step(gid0 + uint32_t(4 * i), acc[i & 1], k1, k2);
        if (i + 1 < kExSteps) interleave_step();
        __builtin_amdgcn_sched_barrier(0);
        in = next;
      }
    } else {
      for (int32_t i = 0; i < nsteps; ++i) {
        v4i acc[kExTiles];
        mfma_step(read_step(r0 + i * kStepBytes, r1 + i * kStepBytes, cp + i * kQueryTile), bq,
                  acc);
        fold_step(gid0 + uint32_t(4 * i), acc, k1, k2);
      }
    }
    if (more) {
      // Every wave is done with the other buffer (last barrier); this one's
      // reads end at the barrier below, after which the next buffer is whole.
      if (tid < kExBuf) lds.nc[cur ^ 1][tid] = nw;
      wait_all_loads();
      barrier();
    }
  }

  // The four lanes of each query merge their two smallest; lanes 0..15 write.
  uint2* pp = part + P.ex_off + int64_t(s) * P.na;
#pragma unroll
  for (int k = 0; k < kExTiles; ++k) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const uint32_t p1 = __shfl_xor(k1[k], o, 64), p2 = __shfl_xor(k2[k], o, 64);
      k2[k] = min(max(k1[k], p1), min(k2[k], p2));
      k1[k] = min(k1[k], p1);
    }
    const int32_t i = qw + kQueryTile * k + col;
    if (g == 0 && i < P.na) pp[i] = make_uint2(k1[k], k2[k]);
  }
}

// One thread per query folds the pair's slices in ascending order (strictly
// smaller replaces, so the earlier slice keeps a shared smallest distance).
// What the slices give is the smallest distance, the group of four targets
// that holds it first, and the smallest distance of any other group.  The
// group's own four distances (four lanes per query) then name the lowest index
// at the smallest distance and complete the second smallest.  Queries that
// fail the ratio test against the other groups alone skip that, unless every
// query's result is asked for: the second distance could only get smaller.
// (The four read each of the four rows together: a lane that reads a row of its
// own asks for every line eight times, 45 us for a staged launch's 1.4 M
// queries, 28.5 so.  The rest is its chain of reads.)
constexpr int kMergeThreads = 256;
constexpr int kMergeBatch = 8;

__global__ __launch_bounds__(kMergeThreads) void exhaustive_merge_kernel(BatchView v,
                                                                         ExStage stage,
                                                                         const uint2* part) {
  const int32_t p = stage.first + int32_t(blockIdx.x) * stage.step;
  const PairDesc P = v.pairs[p];
  const int lane = threadIdx.x & 63;
  const int32_t i0 = int32_t(blockIdx.y) * kMergeThreads + int32_t(threadIdx.x & ~63u);
  if (i0 >= P.na) return;   // uniform over the wave
  const int32_t i = i0 + lane;
  if (!stage_open(v, stage, p)) {
    if (i < P.na) v.res[P.q_off + i] = {-1, kDistInf, kDistInf, 0};
    return;
  }
  const ImageDev A = v.images[P.a], B = v.images[P.b];
  int32_t d1 = kDistInf, d2 = kDistInf, j1 = -1;
  const int32_t nq = ((g_i32*)A.norm2)[min(i, P.na - 1)];
  if (i < P.na) {
    const int32_t nsl = (P.nb + kExSlice - 1) / kExSlice;
    const uint2* pp = part + P.ex_off + i;
    uint32_t s1 = kExKeyDistInf, s2 = kExKeyDistInf;
    // kMergeBatch slices' loads in flight together (clamped past the last).
    for (int32_t s0 = 0; s0 < nsl; s0 += kMergeBatch) {
      v2u kk[kMergeBatch];
#pragma unroll
      for (int b = 0; b < kMergeBatch; ++b)
        kk[b] = *(g_v2u*)(pp + int64_t(min(s0 + b, nsl - 1)) * P.na);
#pragma unroll
      for (int b = 0; b < kMergeBatch; ++b) {
        if (s0 + b >= nsl) break;
        const uint32_t kd1 = kk[b].x >> kPosBits, kd2 = kk[b].y >> kPosBits;
        if (kd1 < s1) {
          s2 = min(s1, kd2);
          s1 = kd1;
          j1 = (s0 + b) * kExSlice + 4 * int32_t(kk[b].x & (kChunk - 1));
        } else if (kd1 == s1) {
          s2 = s1;
        } else {
          s2 = min(s2, kd1);
        }
      }
    }
    if (s1 != kExKeyDistInf) d1 = int32_t(s1) - int32_t(kDistBias) + nq;
    if (s2 != kExKeyDistInf) d2 = int32_t(s2) - int32_t(kDistBias) + nq;
  }
  const bool open = d1 != kDistInf &&
                    (v.keep_counts || d2 == kDistInf ||
                     int64_t(v.ratio_den) * d1 < int64_t(v.ratio_num) * d2);
  // The open queries of the wave, sixteen at a time, four lanes each.
  unsigned long long todo = __ballot(open);
  while (todo) {
    unsigned long long left = todo;   // lane's query: the (lane / 4)-th one left
    for (int k = 0; k < (lane >> 2) && left; ++k) left &= left - 1;
    const int src = left ? __builtin_ctzll(left) : -1;
    const int from = max(src, 0);
    const int32_t jj = __shfl(j1, from, 64) + (lane & 3);
    const int32_t qn = __shfl(nq, from, 64);
    // (Every lane takes part: clamped rows where it has none.)
    const int32_t jc = min(max(jj, 0), P.nb - 1);
    const QuadRows rows = quad_rows(B.desc, jc, lane & 3);
    const RowPart own = row_part(A.desc, i0 + from, lane & 3);
    const int32_t norm = ((g_i32*)B.norm2)[jc];
    const int32_t dot = quad_dots(own, rows, lane & 3);
    const int32_t D = src >= 0 && jj < P.nb ? qn + norm - 2 * dot : kDistInf;
    // The two smallest of the four and the lowest index of the smallest.
    int32_t w1 = D, w2 = kDistInf, wj = jj;
#pragma unroll
    for (int o = 1; o <= 2; o <<= 1) {
      const int32_t e1 = __shfl_xor(w1, o, 64), e2 = __shfl_xor(w2, o, 64);
      const int32_t ej = __shfl_xor(wj, o, 64);
      w2 = min(max(w1, e1), min(w2, e2));
      wj = e1 < w1 || (e1 == w1 && ej < wj) ? ej : wj;
      w1 = min(w1, e1);
    }
    // Back to the query's own lane: it is number r of the queries left.
    const int r = __builtin_popcountll(todo & ((1ull << lane) - 1));
    const bool mine = ((todo >> lane) & 1) && r < 16;
    const int32_t g2 = __shfl(w2, 4 * (r & 15), 64), gj = __shfl(wj, 4 * (r & 15), 64);
    if (mine) {
      d2 = min(d2, g2);
      j1 = gj;
    }
    todo &= ~__ballot(mine);
  }
  bool accept = false;
  if (d2 != kDistInf)
    accept = int64_t(v.ratio_den) * d1 < int64_t(v.ratio_num) * d2;
  else
    accept = d1 != kDistInf && v.accept_single;
  if (i < P.na) {
    QueryResult r;
    r.match = d1 != kDistInf ? j1 : -1;
    r.d1 = d1;
    r.d2 = d2;
    r.flags = (accept ? 1 : 0) | (v.keep_counts ? (P.nb << 1) : 0);
    v.res[P.q_off + i] = r;
  }
  const unsigned long long m = __ballot(accept);
  if (lane == 0 && m)
    atomicAdd(&v.counters[p].accepted, uint32_t(__builtin_popcountll(m)));
}

}  // namespace

void exhaustive_plan(PairDesc* pd, int32_t n_pairs, const ExStage& stage, int2* items,
                     int64_t* n_items, int64_t* n_part) {
  int64_t ni = 0, np = 0;
  for (int64_t k = stage.first; k < n_pairs; k += stage.step) {
    PairDesc& P = pd[k];
    P.ex_off = np;
    const int32_t nqb = (P.na + kExQueries - 1) / kExQueries;
    const int32_t nsl = (P.nb + kExSlice - 1) / kExSlice;
    np += int64_t(P.na) * nsl;
    for (int32_t s = 0; s < nsl; ++s)
      for (int32_t qb = 0; qb < nqb; ++qb) {
        if (items) items[ni] = make_int2(int32_t(k), (qb << 16) | s);
        ++ni;
      }
  }
  *n_items = ni;
  *n_part = np;
}

hipError_t launch_exhaustive(const BatchView& v, const ExStage& stage, const int2* items,
                             int64_t n_items, uint2* part, hipStream_t st) {
  const int32_t pairs = (v.n_pairs - stage.first + stage.step - 1) / stage.step;
  if (pairs <= 0) return hipSuccess;
  const int64_t count_wgs = (int64_t(pairs) + 64 * kExWaves - 1) / (64 * kExWaves);
  const int64_t wgs = std::max(n_items, count_wgs);
  if (wgs > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(exhaustive_kernel, dim3(uint32_t(wgs)), dim3(64 * kExWaves), 0, st, v, stage,
                     items, int32_t(std::min<int64_t>(n_items, INT32_MAX)), part);
  const uint32_t chunks =
      uint32_t(std::max(1, (v.max_na + kMergeThreads - 1) / kMergeThreads));
  hipLaunchKernelGGL(exhaustive_merge_kernel, dim3(uint32_t(pairs), chunks), dim3(kMergeThreads),
                     0, st, v, stage, part);
  return hipGetLastError();
}

}  // namespace sfm
