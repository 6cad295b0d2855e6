// Candidate images from point-camera covisibility (Section 6.1).
//
// For images i and j of the coarse model, the covisible points are the
// points both observe, P_cv(i, j) = Points(i) ∩ Points(j).  Image q's
// candidates are the images sharing more than T points with it, ranked by
// |P_cv(q, i)| (ties: lower index), at most k of them; the unique unordered
// pairs over all queries are what the matcher then runs.
//
// GPU form, by one of two exact counting methods:
//   - the co-observer histogram: the visibility (points of each image) is
//     transposed into the observers of each point by a counting sort, then one
//     workgroup per image q adds one, in an LDS row, for every other observer
//     of every point q sees;
//   - the bit-matrix product: each image's points become a bitset row, and the
//     counts are the products V V^T of 0/1 rows on the matrix cores (FP4).
// Then one workgroup per image ranks its row: a binary search finds the count
// that top_k images reach, and only those are sorted (packed keys count, ~j).
// Every candidate sets the bit of its unordered pair; the bits are counted per
// row, and the unique pairs written in ascending order from those counts.
// (Counting a bit where it is first set takes its old value from the atomic:
// 30 us of waiting for 1,000 images, against 5 us for the counts' own kernel.)
#include <algorithm>

#include "sfm_internal.h"

namespace sfm {
namespace {

constexpr int kCovisThreads = 1024;   // histogram rows
constexpr int kRankThreads = 512;     // rows that are only ranked

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* p, int64_t n, int32_t value) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = value;
}

// The [begin, end) range of image i's points, clamped to [0, nnz).
__device__ __forceinline__ void image_range(const int32_t* vis_off, int32_t i, int64_t nnz,
                                            int64_t& b, int64_t& e) {
  b = min(max(int64_t(vis_off[i]), int64_t(0)), nnz);
  e = min(max(int64_t(vis_off[i + 1]), b), nnz);
}

// Clears image i's row of pair bits (bits may be NULL).
__device__ __forceinline__ void clear_pair_row(uint32_t* bits, int32_t i, int32_t words) {
  if (!bits) return;
  for (int32_t w = threadIdx.x; w < words; w += blockDim.x) bits[int64_t(i) * words + w] = 0u;
}

// Pass 1 of the transpose: observers per point.  One block per image.
__global__ __launch_bounds__(256) void covis_count_kernel(const int32_t* vis_off,
                                                          const int32_t* vis_pts, int64_t nnz,
                                                          int32_t n_points, int32_t* pt_count,
                                                          uint32_t* bits, int32_t bit_words,
                                                          int32_t* err) {
  clear_pair_row(bits, int32_t(blockIdx.x), bit_words);
  int64_t b, e;
  image_range(vis_off, blockIdx.x, nnz, b, e);
  for (int64_t s = b + threadIdx.x; s < e; s += blockDim.x) {
    const int32_t p = vis_pts[s];
    if (p < 0 || p >= n_points) {
      *err = 1;
      continue;
    }
    atomicAdd(&pt_count[p], 1);
  }
}

// Pass 2 of the transpose: image i into the observer list of each of its
// points.  Positions past nnz (inconsistent input) raise the error flag.
__global__ __launch_bounds__(256) void covis_scatter_kernel(const int32_t* vis_off,
                                                            const int32_t* vis_pts, int64_t nnz,
                                                            int32_t n_points, int32_t* cursor,
                                                            int32_t* pt_imgs, int32_t* err) {
  int64_t b, e;
  image_range(vis_off, blockIdx.x, nnz, b, e);
  for (int64_t s = b + threadIdx.x; s < e; s += blockDim.x) {
    const int32_t p = vis_pts[s];
    if (p < 0 || p >= n_points) continue;
    const int32_t pos = atomicAdd(&cursor[p], 1);
    if (pos < 0 || int64_t(pos) >= nnz) {
      *err = 1;
      continue;
    }
    pt_imgs[pos] = int32_t(blockIdx.x);
  }
}

// One block per query image q: |P_cv(q, j)| for every j, then the ranked
// candidates.  Thread t holds the counts of images t, t + NT, ... (0 for
// non-candidates).  When more than top_k images are candidates, a binary search
// over the bits of the counts finds the largest v that at least top_k of
// them reach; only those (v itself may be shared) are sorted, as keys that
// pack (count, 2^32 - 1 - j), so a descending sort ranks by count, then by
// lower index.  (1,000 images, top 100: 22 us with the sum over eight slices;
// sorting whole rows took 34 us, without a sum.)
// kGram: row q is the sum of `slices` n x n count matrices; otherwise it is
// counted here.  bits (may be NULL) receives the pairs.
template <bool kGram, int NT>
__global__ __launch_bounds__(NT) void covis_rows_kernel(
    const int32_t* vis_off, const int32_t* vis_pts, int64_t nnz, int32_t n_images,
    int32_t n_points, const int32_t* pt_off, const int32_t* pt_imgs, const int32_t* gram,
    int32_t slices, int32_t threshold, int32_t top_k, int32_t* cand, int32_t* n_shared,
    int32_t* n_cand, uint32_t* bits) {
  constexpr int kPer = kMaxCovisImages / NT;
  constexpr int kWaves = NT / 64;
  __shared__ unsigned long long keys[kMaxCovisImages];
  __shared__ int32_t wsum[2][kWaves];
  __shared__ int32_t filled;
  const int32_t q = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t == 0) filled = 0;
  uint32_t c[kPer];
  if (kGram) {
    // Eight slices' loads in flight together (clamped past the last).
    const int64_t matrix = int64_t(n_images) * n_images;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      c[k] = 0u;
      if (k * NT >= n_images) continue;   // uniform
      const int32_t* at = gram + int64_t(q) * n_images + min(t + k * NT, n_images - 1);
      for (int32_t s0 = 0; s0 < slices; s0 += 8) {
        uint32_t x[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = uint32_t(at[min(s0 + s, slices - 1) * matrix]);
#pragma unroll
        for (int s = 0; s < 8; ++s) c[k] += s0 + s < slices ? x[s] : 0u;
      }
      if (t + k * NT >= n_images) c[k] = 0u;
    }
  } else {
    uint32_t* row = reinterpret_cast<uint32_t*>(keys);
    for (int32_t j = t; j < n_images; j += NT) row[j] = 0u;
    __syncthreads();
    // A wave takes one point at a time and its lanes the point's observers:
    // the observers of a point are distinct images, so the LDS atomics of one
    // instruction never collide (lanes each walking their own point's list hit
    // the same nearby images together and serialise).
    // Four points per wave and iteration, their loads issued before any of
    // their atomics, so the chain point -> offsets -> observers overlaps.
    int64_t b, e;
    image_range(vis_off, q, nnz, b, e);
    constexpr int kPts = 4;
    constexpr int64_t kWaveStride = int64_t(kWaves) * kPts;
    for (int64_t s0 = b + int64_t(wave) * kPts; s0 < e; s0 += kWaveStride) {
      int64_t o0[kPts], o1[kPts];
#pragma unroll
      for (int u = 0; u < kPts; ++u) {
        const int32_t p = s0 + u < e ? vis_pts[s0 + u] : -1;
        o0[u] = o1[u] = 0;
        if (p >= 0 && p < n_points) {
          // Offsets past nnz only arise from inconsistent input (the scatter
          // raised the error flag); reads stay inside pt_imgs.
          o0[u] = max(int64_t(pt_off[p]), int64_t(0));
          o1[u] = min(int64_t(pt_off[p + 1]), nnz);
        }
      }
      int32_t jj[kPts];
#pragma unroll
      for (int u = 0; u < kPts; ++u) jj[u] = o0[u] + lane < o1[u] ? pt_imgs[o0[u] + lane] : -1;
#pragma unroll
      for (int u = 0; u < kPts; ++u) {
        if (jj[u] != q && jj[u] >= 0 && jj[u] < n_images) atomicAdd(&row[jj[u]], 1u);
        for (int64_t o = o0[u] + 64 + lane; o < o1[u]; o += 64) {
          const int32_t j = pt_imgs[o];
          if (j != q && j >= 0 && j < n_images) atomicAdd(&row[j], 1u);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) c[k] = t + k * NT < n_images ? row[t + k * NT] : 0u;
  }
  // Candidates among this thread's images, their number and the bits of the
  // largest count.
  uint32_t any = 0u;
  int32_t mine = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (t + k * NT == q || c[k] <= uint32_t(threshold)) c[k] = 0u;
    any |= c[k];
    mine += c[k] ? 1 : 0;
  }
  for (int o = 32; o > 0; o >>= 1) {
    any |= __shfl_xor(any, o, 64);
    mine += __shfl_xor(mine, o, 64);
  }
  __shared__ uint32_t wany[kWaves];
  if (lane == 0) {
    wsum[0][wave] = mine;
    wany[wave] = any;
  }
  __syncthreads();   // also ends the reads of `row`, whose place the keys take
  int32_t total = 0;
  any = 0u;
  for (int w = 0; w < kWaves; ++w) {
    total += wsum[0][w];
    any |= wany[w];
  }
  const int32_t taken = min(top_k, total);
  uint32_t v = 1u;   // candidates have counts of at least 1
  if (total > top_k && top_k > 0) {
    v = 0u;
    int par = 1;
    for (int bit = 31 - __builtin_clz(any); bit >= 0; --bit, par ^= 1) {
      const uint32_t at = v | (1u << bit);
      int32_t n = 0;
#pragma unroll
      for (int k = 0; k < kPer; ++k) n += __builtin_popcountll(__ballot(c[k] >= at));
      if (lane == 0) wsum[par][wave] = n;
      __syncthreads();
      n = 0;
      for (int w = 0; w < kWaves; ++w) n += wsum[par][w];
      if (n >= top_k) v = at;
    }
    v = max(v, 1u);
  }
  bool sorted = false;
  int32_t rank = taken;
  unsigned long long key = 0ull;
  if (taken > 0) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const bool in = c[k] >= v;
      const unsigned long long m = __ballot(in);
      if (!m) continue;
      int32_t base = 0;
      if (lane == 0) base = atomicAdd(&filled, __builtin_popcountll(m));
      base = __shfl(base, 0, 64);
      if (in)
        keys[base + __builtin_popcountll(m & ((1ull << lane) - 1))] =
            ((unsigned long long)c[k] << 32) | (0xFFFFFFFFull - uint32_t(t + k * NT));
    }
    __syncthreads();
    const int32_t n = filled;
    if (n <= NT) {
      // Few keys (top_k of them, more only when v is shared): each thread
      // counts the keys above its own, which are all read by broadcast.
      rank = n;
      if (t < n) {
        key = keys[t];
        rank = 0;
#pragma unroll 8
        for (int32_t i = 0; i < n; ++i) rank += keys[i] > key ? 1 : 0;
      }
    } else {
      // Bitonic sort, descending, of nsort (a power of two) keys.
      int32_t nsort = 2 * NT;
      while (nsort < n) nsort <<= 1;
      for (int32_t r = n + t; r < nsort; r += NT) keys[r] = 0ull;
      __syncthreads();
      for (int32_t size = 2; size <= nsort; size <<= 1) {
        for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
          for (int32_t i = t; i < nsort / 2; i += NT) {
            const int32_t lo = 2 * i - (i & (stride - 1));
            const int32_t hi = lo + stride;
            const bool desc = (lo & size) == 0;
            const unsigned long long x = keys[lo], y = keys[hi];
            if ((x < y) == desc) {
              keys[lo] = y;
              keys[hi] = x;
            }
          }
          __syncthreads();
        }
      }
      sorted = true;
    }
  }
  const int32_t words = (n_images + 31) / 32;
  auto put = [&](int32_t r, unsigned long long k) {
    const int32_t j = int32_t(0xFFFFFFFFull - (k & 0xFFFFFFFFull));
    const int64_t at = int64_t(q) * top_k + r;
    cand[at] = j;
    n_shared[at] = int32_t(k >> 32);
    if (bits) atomicOr(&bits[int64_t(min(q, j)) * words + (max(q, j) >> 5)], 1u << (max(q, j) & 31));
  };
  if (sorted) {
    for (int32_t r = t; r < taken; r += NT) put(r, keys[r]);
  } else if (rank < taken) {
    put(rank, key);
  }
  for (int32_t r = taken + t; r < top_k; r += NT) {
    cand[int64_t(q) * top_k + r] = -1;
    n_shared[int64_t(q) * top_k + r] = 0;
  }
  if (t == 0) n_cand[q] = taken;
}

// ---------------------------------------------------------------------------
// Bit-matrix path: V[i] = the bitset of image i's points (words of 32
// points, rows padded with zeros to whole units where the workspace has room),
// and |P_cv(i, j)| = sum over points of V[i] V[j].
// ---------------------------------------------------------------------------
constexpr int kBitsLdsWords = 8192;   // points per LDS pass of the bitset build: 262,144

// Bitset rows: one block per image, its row built in LDS a chunk of words at
// a time (LDS atomics) and written out coalesced.
__global__ __launch_bounds__(1024) void bitset_rows_kernel(const int32_t* vis_off,
                                                           const int32_t* vis_pts, int64_t nnz,
                                                           int32_t n_points, int64_t words,
                                                           uint32_t* V, uint32_t* bits,
                                                           int32_t bit_words, int32_t* err) {
  __shared__ uint32_t lds[kBitsLdsWords];
  const int32_t i = blockIdx.x;
  clear_pair_row(bits, i, bit_words);
  int64_t b, e;
  image_range(vis_off, i, nnz, b, e);
  for (int64_t w0 = 0; w0 < words; w0 += kBitsLdsWords) {
    const int64_t nw = min(int64_t(kBitsLdsWords), words - w0);
    for (int64_t w = threadIdx.x; w < nw; w += blockDim.x) lds[w] = 0u;
    __syncthreads();
    const int64_t p_lo = w0 * 32, p_hi = (w0 + nw) * 32;
    for (int64_t s = b + threadIdx.x; s < e; s += blockDim.x) {
      const int32_t p = vis_pts[s];
      if (p < 0 || p >= n_points) {
        *err = 1;
        continue;
      }
      if (p < p_lo || p >= p_hi) continue;
      atomicOr(&lds[(p >> 5) - w0], 1u << (p & 31));
    }
    __syncthreads();
    for (int64_t w = threadIdx.x; w < nw; w += blockDim.x) V[int64_t(i) * words + w0 + w] = lds[w];
    __syncthreads();
  }
}

// Counts of one 64 x 64 block of image pairs (block I <= block J) over one
// slice of the points.  Four waves take every fourth unit of 512 points of
// the slice; a wave keeps the block in sixteen 16 x 16 accumulators of
// v_mfma_f32_16x16x128_f8f6f4 with FP4 operands.  Lane (r, g) reads words
// 4 g .. 4 g + 3 of row r of a unit, 16 bytes; word w of all lanes is one
// K = 128 product.  A word's 32 bits become 32 FP4 values with a few masks:
// bit 4 i + k goes to nibble i of register k, the same on both sides, where
// bits 0, 1 and 2 of a nibble already read as 0.5, 1 and 2.  Rows of I are
// left at 0.5, 1, 2 and (shifted) 0.5, rows of J shifted to 2, 1, 0.5 and 2, so
// every product of two ones is 1 and the FP32 sums are exact (they are moved
// to integers every 64 units, far below 2^24).  The waves add up in LDS, and
// the block is written to the slice's matrix both ways round.
// Bound by the expansion: 48 VALU instructions beside 16 MFMAs of 16 cycles,
// which hide about one each.  1,000 images x 200,000 points: 60 us (3.3 FP4
// Pop/s); with AND and popcount on the VALU, from LDS, 420 us.
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kGramRows = 64;
constexpr int kGramTiles = kGramRows / 16;
constexpr int kUnitWords = 16;        // words of a unit (512 points)
constexpr int kGramFlush = 64;        // units between moves to integers

__device__ __forceinline__ v8i expand_i(uint32_t w) {
  return v8i{int(w & 0x11111111u), int(w & 0x22222222u), int(w & 0x44444444u),
             int((w >> 3) & 0x11111111u), 0, 0, 0, 0};
}
__device__ __forceinline__ v8i expand_j(uint32_t w) {
  return v8i{int((w << 2) & 0x44444444u), int(w & 0x22222222u), int((w >> 2) & 0x11111111u),
             int((w >> 1) & 0x44444444u), 0, 0, 0, 0};
}

// kWhole: rows are whole units.  Otherwise the words past a row's end read as 0.
template <bool kWhole>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void gram_kernel(const uint32_t* V, int32_t n_images, int64_t words, int32_t slices,
                 int32_t nblk, int32_t* gram) {
  __shared__ int32_t sum[kGramRows][kGramRows + 1];
  // One slice per XCD (or a few): workgroups are dealt to the XCDs round-robin,
  // so with eight slices the rows of a slice stay in one L2.
  const int32_t slice = int32_t(blockIdx.x) % slices;
  int32_t I = 0, rem = int32_t(blockIdx.x) / slices;   // block (I, J), I <= J
  while (rem >= nblk - I) {
    rem -= nblk - I;
    ++I;
  }
  const int32_t J = I + rem;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int r = lane & 15, g = lane >> 4;
  for (int x = t; x < kGramRows * (kGramRows + 1); x += 256) (&sum[0][0])[x] = 0;
  const int64_t units = (words + kUnitWords - 1) / kUnitWords;
  const int64_t u0 = units * slice / slices, u1 = units * (slice + 1) / slices;
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  typedef uint32_t v4w __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length
  typedef const __attribute__((address_space(1))) v4u g_v4u;
  typedef const __attribute__((address_space(1))) v4w g_v4w;
  typedef const __attribute__((address_space(1))) uint32_t g_u32;
  // Rows past the last image read the last one; their counts are not written.
  const uint32_t* pi[kGramTiles];
  const uint32_t* pj[kGramTiles];
#pragma unroll
  for (int k = 0; k < kGramTiles; ++k) {
    pi[k] = V + int64_t(min(I * kGramRows + 16 * k + r, n_images - 1)) * words + 4 * g;
    pj[k] = V + int64_t(min(J * kGramRows + 16 * k + r, n_images - 1)) * words + 4 * g;
  }
  // The lane's four words of unit u of a row (p: the row's word 4 g).
  auto unit = [&](const uint32_t* p, int64_t u) -> v4u {
    if (kWhole) return *(g_v4u*)(p + u * kUnitWords);
    const int64_t left = words - (u * kUnitWords + 4 * g);
    if (left >= 4) return *(g_v4w*)(p + u * kUnitWords);
    v4u x = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < left) x[k] = *(g_u32*)(p + u * kUnitWords + k);
    return x;
  };
  v4f acc[kGramTiles][kGramTiles];
#pragma unroll
  for (int a = 0; a < kGramTiles; ++a)
#pragma unroll
    for (int b = 0; b < kGramTiles; ++b) acc[a][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  auto flush = [&]() {
#pragma unroll
    for (int a = 0; a < kGramTiles; ++a)
#pragma unroll
      for (int b = 0; b < kGramTiles; ++b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int32_t n = int32_t(acc[a][b][e]);
          if (n) atomicAdd(&sum[16 * a + 4 * g + e][16 * b + r], n);
        }
        acc[a][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
      }
  };
  __syncthreads();
  int32_t held = 0;
  v4u ni[kGramTiles], nj[kGramTiles];
  int64_t u = u0 + wave;
  if (u < u1) {
#pragma unroll
    for (int k = 0; k < kGramTiles; ++k) {
      ni[k] = unit(pi[k], u);
      nj[k] = unit(pj[k], u);
    }
  }
  for (; u < u1; u += 4) {
    v4u wi[kGramTiles], wj[kGramTiles];
    const int64_t un = min(u + 4, u1 - 1);   // the next unit's words load meanwhile
#pragma unroll
    for (int k = 0; k < kGramTiles; ++k) {
      wi[k] = ni[k];
      wj[k] = nj[k];
      ni[k] = unit(pi[k], un);
      nj[k] = unit(pj[k], un);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      v8i b[kGramTiles];
#pragma unroll
      for (int k = 0; k < kGramTiles; ++k) b[k] = expand_j(wj[k][w]);
#pragma unroll
      for (int a = 0; a < kGramTiles; ++a) {
        const v8i x = expand_i(wi[a][w]);
#pragma unroll
        for (int k = 0; k < kGramTiles; ++k)
          acc[a][k] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x, b[k], acc[a][k], 4, 4,
                                                                      0, 0, 0, 0);
      }
    }
    if (++held == kGramFlush) {
      flush();
      held = 0;
    }
  }
  flush();
  __syncthreads();
  int32_t* out = gram + int64_t(slice) * n_images * n_images;
  for (int x = t; x < kGramRows * kGramRows; x += 256) {
    const int y = x / kGramRows, z = x % kGramRows;
    const int32_t i = I * kGramRows + y, j = J * kGramRows + z;
    if (i < n_images && j < n_images) out[int64_t(i) * n_images + j] = sum[y][z];
    const int32_t i2 = J * kGramRows + y, j2 = I * kGramRows + z;
    if (I != J && i2 < n_images && j2 < n_images) out[int64_t(i2) * n_images + j2] = sum[z][y];
  }
}

// Pairs per row i (set bits); one wave per row.
__global__ __launch_bounds__(256) void pair_count_kernel(const uint32_t* bits, int32_t words,
                                                         int32_t n_images, int32_t* row_count) {
  const int32_t i = int32_t(blockIdx.x) * 4 + int32_t(threadIdx.x >> 6);
  if (i >= n_images) return;
  const int lane = threadIdx.x & 63;
  int32_t c = 0;
  for (int32_t w = lane; w < words; w += 64) c += __builtin_popcount(bits[int64_t(i) * words + w]);
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if (lane == 0) row_count[i] = c;
}

// Writes row i's pairs (i, j) in ascending j after those of the rows before
// it; one block per row, one thread per word (words <= kMaxCovisImages / 32 =
// 128).
constexpr int kWriteThreads = 128;
__global__ __launch_bounds__(kWriteThreads) void pair_write_kernel(
    const uint32_t* bits, int32_t words, const int32_t* row_count, int32_t n_images,
    int32_t* pairs, int64_t* n_pairs) {
  __shared__ int32_t tot[2][kWriteThreads / 64];
  const int32_t i = blockIdx.x;
  const int w = threadIdx.x, lane = w & 63, wave = w >> 6;
  const uint32_t word = w < words ? bits[int64_t(i) * words + w] : 0u;
  int32_t before = 0;   // pairs of the rows before i
  for (int32_t k = w; k < i; k += kWriteThreads) before += row_count[k];
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  const int32_t own = __builtin_popcount(word);
  int32_t x = own;      // inclusive scan of the row's words
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) {
    tot[0][wave] = before;
    tot[1][wave] = x;
  }
  __syncthreads();
  const int64_t row0 = int64_t(tot[0][0]) + tot[0][1];
  int64_t at = row0 + (wave ? tot[1][0] : 0) + x - own;
  if (i == n_images - 1 && w == 0) *n_pairs = row0 + tot[1][0] + tot[1][1];
  uint32_t m = word;
  while (m) {
    const int bit = __builtin_ctz(m);
    m &= m - 1;
    pairs[2 * at] = i;
    pairs[2 * at + 1] = 32 * w + bit;
    ++at;
  }
}

int32_t grid_for(int64_t n, int32_t per_block) {
  return int32_t(std::max<int64_t>(1, std::min<int64_t>((n + per_block - 1) / per_block, 65535)));
}

}  // namespace

int64_t covis_bitset_words(int32_t n_points) {
  return (int64_t(n_points) + 32 * kUnitWords - 1) / (32 * kUnitWords) * kUnitWords;
}

// About four workgroups per CU, in whole XCDs' worth from eight on; a slice
// has at least a unit per wave.
int32_t covis_gram_slices(int32_t n_images, int32_t n_points) {
  const int64_t nblk = (n_images + kGramRows - 1) / kGramRows, blocks = nblk * (nblk + 1) / 2;
  const int64_t units = covis_bitset_words(n_points) / kUnitWords;
  int32_t s = 1;
  while (s < 64 && int64_t(s) * blocks < 1024 && int64_t(s) * 8 <= units) s <<= 1;
  return s;
}

hipError_t launch_candidates(const CovisArgs& a, hipStream_t st) {
  const int64_t np1 = int64_t(a.n_points) + 1;
  const bool pairs = a.pairs && a.n_images > 0 && a.top_k > 0;
  uint32_t* bits = pairs ? a.bits : nullptr;
  const int32_t bit_words = (a.n_images + 31) / 32;
  if (a.gram) {
    // Bit-matrix path: bitset rows, the count matrices, then each row's ranking.
    if (a.n_images > 0) {
      const int64_t words = a.row_words;
      hipLaunchKernelGGL(bitset_rows_kernel, dim3(a.n_images), dim3(1024), 0, st, a.vis_off,
                         a.vis_pts, a.nnz, a.n_points, words, a.bitset, bits, bit_words,
                         a.err);
      const int32_t nblk = (a.n_images + kGramRows - 1) / kGramRows;
      const dim3 blocks(nblk * (nblk + 1) / 2 * a.slices);
      if (words % kUnitWords == 0)
        hipLaunchKernelGGL(gram_kernel<true>, blocks, dim3(256), 0, st, a.bitset, a.n_images, words,
                           a.slices, nblk, a.gram);
      else
        hipLaunchKernelGGL(gram_kernel<false>, blocks, dim3(256), 0, st, a.bitset, a.n_images,
                           words, a.slices, nblk, a.gram);
      hipLaunchKernelGGL((covis_rows_kernel<true, kRankThreads>), dim3(a.n_images), dim3(kRankThreads), 0, st,
                         a.vis_off, a.vis_pts, a.nnz, a.n_images, a.n_points, a.pt_off,
                         a.pt_imgs, a.gram, a.slices, a.threshold, a.top_k, a.cand, a.n_shared,
                         a.n_cand, bits);
    }
  } else {
    // Point-histogram path: observers of every point (counts, exclusive
    // offsets, scatter), then each image's co-observers in LDS.
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(np1, 256)), dim3(256), 0, st, a.pt_count,
                       np1, 0);
    if (a.n_images > 0)
      hipLaunchKernelGGL(covis_count_kernel, dim3(a.n_images), dim3(256), 0, st, a.vis_off,
                         a.vis_pts, a.nnz, a.n_points, a.pt_count, bits, bit_words, a.err);
    if (const hipError_t e = launch_scan(a.pt_count, a.pt_off, np1, false, a.sums, a.cursor, st); e != hipSuccess)
      return e;
    if (a.n_images > 0) {
      hipLaunchKernelGGL(covis_scatter_kernel, dim3(a.n_images), dim3(256), 0, st, a.vis_off,
                         a.vis_pts, a.nnz, a.n_points, a.cursor, a.pt_imgs, a.err);
      hipLaunchKernelGGL((covis_rows_kernel<false, kCovisThreads>), dim3(a.n_images),
                         dim3(kCovisThreads), 0, st, a.vis_off, a.vis_pts, a.nnz, a.n_images,
                         a.n_points, a.pt_off, a.pt_imgs, nullptr, 1, a.threshold, a.top_k,
                         a.cand, a.n_shared, a.n_cand, bits);
    }
  }
  if (pairs) {
    hipLaunchKernelGGL(pair_count_kernel, dim3((a.n_images + 3) / 4), dim3(256), 0, st, a.bits,
                       bit_words, a.n_images, a.row_count);
    hipLaunchKernelGGL(pair_write_kernel, dim3(a.n_images), dim3(kWriteThreads), 0, st, a.bits,
                       bit_words, a.row_count, a.n_images, a.pairs, a.n_pairs);
  } else if (a.pairs && a.n_pairs) {
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, st,
                       reinterpret_cast<int32_t*>(a.n_pairs), 2, 0);
  }
  return hipGetLastError();
}

}  // namespace sfm
