// Track merging and triangulation (Section 6.3).
//
// Tracks are the connected components of the match graph: its nodes are
// observations (one feature of one image), its edges the accepted matches of
// all matched pairs.  The paper finds them with a sequential depth-first
// search; here a lock-free union-find runs over all edges at once.  First
// every node with a smaller neighbour is hooked under one (a plain store:
// whichever stays makes a forest) and the paths are compressed: in a match
// graph, where a track's observations are matched many times over, that leaves
// few trees per track.  Then an edge whose ends still have different roots hooks the
// larger root under the smaller with a compare-and-swap; finds halve paths as
// they go.  Parents only ever decrease, so paths terminate and each component's
// root is its smallest node id: a label independent of the order of work.  Few
// edges are left to the compare-and-swaps alone (kHookEdges).
// (About 1 M edges over 0.5 M observations: hook 12 us, two label passes 18, union
// 30.  Hooking roots from the start, the edges raced for them: 158 us.  The
// union is bound by its link reads, four random words per edge, and the few
// compare-and-swaps left; its 8 MB of edges alone pass in 2 us.)
//
// Each track is then triangulated by linear least squares in FP64: an
// observation (x, y) in a camera with rows p1, p2, p3 gives the equations
// (x p3 - p1) . (X, 1) = 0 and (y p3 - p2) . (X, 1) = 0.  The members of
// every track are gathered into lists (each node's rank among its track's from
// the count, a start per track, a scatter), and sixteen lanes per track sum its
// normal equations in registers and solve them in closed form.
#include <algorithm>
#include <cmath>

#include "sfm_internal.h"

namespace sfm {
namespace {

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = 0;
}

// Parent links are read through the caches: a stale link is an older one, so
// still an ancestor's, and the compare-and-swap (at device scope) decides; a
// failed one returns the link as it is and the walk goes on from there.  (Reads
// at device scope go past the L2.)
__device__ __forceinline__ int32_t load_link(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
// The same past the caches, for walks that links of a moment ago shorten.
__device__ __forceinline__ int32_t load_fresh(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_link(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void uf_init_kernel(int32_t* parent, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    parent[i] = int32_t(i);
}

// Hooks every node that has a smaller neighbour under one of them.  Nodes that
// look unhooked (however stale) are stored to by several threads at once, and
// any of their values is a smaller neighbour.
__global__ __launch_bounds__(256) void uf_hook_kernel(int32_t* parent, const int32_t* edges,
                                                      int64_t n_edges, int64_t n_nodes,
                                                      int32_t* err) {
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < n_edges;
       k += int64_t(gridDim.x) * blockDim.x) {
    const int32_t u = edges[2 * k], v = edges[2 * k + 1];
    if (u < 0 || v < 0 || int64_t(u) >= n_nodes || int64_t(v) >= n_nodes) {
      *err = 1;
      continue;
    }
    const int32_t lo = min(u, v), hi = max(u, v);
    if (lo != hi && load_link(&parent[hi]) == hi)
      __hip_atomic_store(&parent[hi], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
}

// Root of x, halving the path on the way (each write replaces a parent by
// one of its own ancestors, so concurrent finds and hooks stay consistent).
// kFresh: links are read past the caches.
template <bool kFresh>
__device__ __forceinline__ int32_t uf_find(int32_t* parent, int32_t x) {
  auto load = [](const int32_t* p) { return kFresh ? load_fresh(p) : load_link(p); };
  int32_t cur = load(&parent[x]);
  if (cur == x) return x;
  int32_t prev = x;
  int32_t next;
  while (cur > (next = load(&parent[cur]))) {
    store_link(&parent[prev], next);
    prev = cur;
    cur = next;
  }
  return cur;
}

template <bool kFresh>
__global__ __launch_bounds__(256) void uf_union_kernel(int32_t* parent, const int32_t* edges,
                                                       int64_t n_edges, int64_t n_nodes,
                                                       int32_t* err) {
  auto load = [](const int32_t* p) { return kFresh ? load_fresh(p) : load_link(p); };
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < n_edges;
       k += int64_t(gridDim.x) * blockDim.x) {
    const int32_t u = edges[2 * k], v = edges[2 * k + 1];
    if (u < 0 || v < 0 || int64_t(u) >= n_nodes || int64_t(v) >= n_nodes) {
      *err = 1;
      continue;
    }
    if (load(&parent[u]) == load(&parent[v])) continue;   // one set already
    int32_t ru = uf_find<kFresh>(parent, u), rv = uf_find<kFresh>(parent, v);
    while (ru != rv) {
      if (ru < rv) {
        const int32_t t = ru;
        ru = rv;
        rv = t;
      }
      // Hook the larger root under the smaller; a failed swap means it got a
      // parent meanwhile: find both roots again.
      const int32_t old = atomicCAS(&parent[ru], ru, rv);
      if (old == ru) break;
      ru = uf_find<kFresh>(parent, old);
      rv = uf_find<kFresh>(parent, rv);
    }
  }
}

// Root of x without writing: the labelling pass below must not use the
// halving find, whose writes (an ancestor read before another thread stored
// its node's root) could replace a finished label by a non-root ancestor.
// Walks longer than eight links read them past the caches, where labels that
// other threads have stored meanwhile cut them short (a chain of 20,000 nodes: 206
// us for the whole call with cached links throughout, 79 so; chains of tens of
// links, as tracks have, are as fast as with cached links).
__device__ __forceinline__ int32_t uf_root(const int32_t* parent, int32_t x) {
  int32_t cur = x, next;
  for (int hops = 0; hops < 8; ++hops) {
    next = load_link(&parent[cur]);
    if (!(cur > next)) return cur;
    cur = next;
  }
  while (cur > (next = load_fresh(&parent[cur]))) cur = next;
  return cur;
}

// Final labels in place: every node points straight at its root.  Each
// thread writes only its own node, and only a root, so concurrent walks see
// either the old ancestor or the root and every label ends as the root.  Also
// the compression between the hooks and the unions.
__global__ __launch_bounds__(256) void uf_label_kernel(int32_t* parent, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    store_link(&parent[i], uf_root(parent, int32_t(i)));
}

// Observations per track: every node but the root counts itself at its root
// and keeps its rank there (the root is number 0, so single observations, most
// nodes, take no atomic).  rank -1: a bad label or image, flagged.
__global__ __launch_bounds__(256) void tri_count_kernel(const int32_t* label,
                                                        const int32_t* node_image,
                                                        int32_t n_images, int64_t n_nodes,
                                                        int32_t* cnt, int32_t* rank,
                                                        int32_t* err) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n_nodes;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int32_t r = label[i], img = node_image[i];
    if (r < 0 || int64_t(r) >= n_nodes || img < 0 || img >= n_images) {
      *err = 1;
      rank[i] = -1;
      continue;
    }
    rank[i] = r == int32_t(i) ? 0 : 1 + atomicAdd(&cnt[r], 1);
  }
}

// A run of the member array and an entry {root, members} of the track list for
// every track of at least two, in any order: one addition to the common totals
// (tracks << 32 | members) per workgroup.  cnt becomes the start of the run
// (-1: none).  Also every node's n_obs, and the points of single observations.
__global__ __launch_bounds__(1024) void tri_start_kernel(const int32_t* label, const int32_t* rank,
                                                         int64_t n_nodes, int32_t* cnt,
                                                         int2* tracks, unsigned long long* totals,
                                                         double* X, int32_t* n_obs) {
  __shared__ unsigned long long wsum[16];
  __shared__ unsigned long long base;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + t;
  const bool root = i < n_nodes && label[i] == int32_t(i);
  const int32_t c = root ? cnt[i] : 0;
  // Observations, and members in the list (a root with a bad image keeps its
  // place there).
  const int32_t obs = root ? c + (rank[i] == 0 ? 1 : 0) : 0;
  const int32_t m = obs >= 2 ? c + 1 : 0;
  if (i < n_nodes) n_obs[i] = obs;
  if (root && obs < 2) X[3 * i] = X[3 * i + 1] = X[3 * i + 2] = NAN;
  const unsigned long long own = m ? (1ull << 32) | uint32_t(m) : 0ull;
  unsigned long long inc = own;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  unsigned long long before = 0, all = 0;
  for (int w = 0; w < 16; ++w) {
    before += w < wave ? wsum[w] : 0;
    all += wsum[w];
  }
  if (t == 0) base = all ? atomicAdd(totals, all) : 0;
  __syncthreads();
  const unsigned long long at = base + before + inc - own;
  if (i < n_nodes) cnt[i] = m ? int32_t(uint32_t(at)) : -1;
  if (m) tracks[at >> 32] = make_int2(int32_t(i), m);
}

__global__ __launch_bounds__(256) void tri_scatter_kernel(const int32_t* label,
                                                          const int32_t* rank, int64_t n_nodes,
                                                          const int32_t* start,
                                                          int32_t* members) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n_nodes;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int32_t k = rank[i];
    if (k < 0) continue;
    const int32_t s = start[label[i]];
    if (s >= 0) members[s + k] = int32_t(i);
  }
}

// Per track of at least two observations: its normal equations summed in
// registers over its members (each observation (x, y) in camera P gives the
// rows x p3 - p1 and y p3 - p2 of A; M = sum of the first three columns' outer
// products, b = -sum a a4), then X = M^-1 b by the adjugate; NaN when M is
// singular (all rays through one centre).  Sixteen lanes per track.  (A thread
// per track, found among all nodes, walked its list alone: 57 us for 0.5 M
// observations of 60 images.  Sixteen lanes per track, but 64 nodes per wave:
// 42 us, as the roots, each track's lowest node, sit close together.  Over the
// list of tracks: 14.)
constexpr int kTrackLanes = 16;
constexpr int kSolveBlocks = 2048;
__global__ __launch_bounds__(256) void tri_solve_kernel(
    const int32_t* node_image, const float* node_xy, const double* P, int32_t n_images,
    const int32_t* start, const int2* tracks, const unsigned long long* totals,
    const int32_t* members, double* X) {
  const int sub = threadIdx.x & (kTrackLanes - 1);
  const int32_t n = int32_t(*totals >> 32);
  // Every lane of a wave runs the same rounds: the sums cross lanes.
  const int32_t groups = int32_t(gridDim.x * blockDim.x) / kTrackLanes;
  const int32_t rounds = (n + groups - 1) / groups;
  for (int32_t r = 0; r < rounds; ++r) {
    const int32_t k0 = r * groups + int32_t(blockIdx.x * blockDim.x + threadIdx.x) / kTrackLanes;
    const bool live = k0 < n;
    const int2 track = tracks[min(k0, n - 1)];
    const int32_t s = start[track.x], m = live ? track.y : 0;
    const int32_t root_image = node_image[track.x];
    const bool bad_root = root_image < 0 || root_image >= n_images;
    double t[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int32_t k = sub + (sub == 0 && bad_root ? kTrackLanes : 0); k < m; k += kTrackLanes) {
      const int32_t j = members[s + k];
      const double* p = P + 12 * int64_t(node_image[j]);
      const double x = node_xy[2 * int64_t(j)], y = node_xy[2 * int64_t(j) + 1];
      double a[2][4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[0][c] = x * p[8 + c] - p[c];
        a[1][c] = y * p[8 + c] - p[4 + c];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        t[0] += a[q][0] * a[q][0];
        t[1] += a[q][0] * a[q][1];
        t[2] += a[q][0] * a[q][2];
        t[3] += a[q][1] * a[q][1];
        t[4] += a[q][1] * a[q][2];
        t[5] += a[q][2] * a[q][2];
        t[6] -= a[q][0] * a[q][3];
        t[7] -= a[q][1] * a[q][3];
        t[8] -= a[q][2] * a[q][3];
      }
    }
#pragma unroll
    for (int o = 1; o < kTrackLanes; o <<= 1)
#pragma unroll
      for (int q = 0; q < 9; ++q) t[q] += __shfl_xor(t[q], o, 64);
    if (!live || sub != 0) continue;
    const int64_t at = 3 * int64_t(track.x);
    const double a = t[0], b = t[1], c = t[2], d = t[3], e = t[4], f = t[5];
    const double c00 = d * f - e * e, c01 = c * e - b * f, c02 = b * e - c * d;
    const double c11 = a * f - c * c, c12 = b * c - a * e, c22 = a * d - b * b;
    const double det = a * c00 + b * c01 + c * c02;
    const double scale = fabs(a) * fabs(d) * fabs(f) + 1e-300;
    if (!(fabs(det) > 1e-12 * scale)) {
      X[at] = X[at + 1] = X[at + 2] = NAN;
      continue;
    }
    const double r0 = t[6], r1 = t[7], r2 = t[8];
    X[at] = (c00 * r0 + c01 * r1 + c02 * r2) / det;
    X[at + 1] = (c01 * r0 + c11 * r1 + c12 * r2) / det;
    X[at + 2] = (c02 * r0 + c12 * r1 + c22 * r2) / det;
  }
}

int32_t blocks_for(int64_t n) {
  return int32_t(std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 65535)));
}

}  // namespace

// Up to this many edges the hooks and their compression, two launches, cost more
// than they spare the unions, whose links are then read past the caches: a match
// graph of 497 edges takes 16 us without them and 22 with, chains of 1,000 nodes 26
// to 50 and 29.  Above it the unions alone depend on the order of the edges (a
// chain of 4,000 nodes: 43 to 323 us without, 45 to 47 with; match graphs of 4,255
// edges: 20 and 22, of 19,637: 28 and 23, of 152,870: 64 and 26).
constexpr int64_t kHookEdges = 1024;

// The label array is the union-find's parent array.
hipError_t launch_tracks(int64_t n_nodes, const int32_t* edges, int64_t n_edges, int32_t* label,
                         int32_t* err, hipStream_t st) {
  if (n_nodes <= 0) return hipSuccess;
  hipLaunchKernelGGL(uf_init_kernel, dim3(blocks_for(n_nodes)), dim3(256), 0, st, label, n_nodes);
  if (n_edges > 0 && n_edges <= kHookEdges) {
    hipLaunchKernelGGL(uf_union_kernel<true>, dim3(blocks_for(n_edges)), dim3(256), 0, st, label,
                       edges, n_edges, n_nodes, err);
  } else if (n_edges > 0) {
    const dim3 per_edge(blocks_for(n_edges)), per_node(blocks_for(n_nodes));
    hipLaunchKernelGGL(uf_hook_kernel, per_edge, dim3(256), 0, st, label, edges, n_edges, n_nodes,
                       err);
    hipLaunchKernelGGL(uf_label_kernel, per_node, dim3(256), 0, st, label, n_nodes);
    hipLaunchKernelGGL(uf_union_kernel<false>, per_edge, dim3(256), 0, st, label, edges, n_edges,
                       n_nodes, err);
  }
  hipLaunchKernelGGL(uf_label_kernel, dim3(blocks_for(n_nodes)), dim3(256), 0, st, label, n_nodes);
  return hipGetLastError();
}

hipError_t launch_triangulate(int64_t n_nodes, const int32_t* label, const int32_t* node_image,
                              const float* node_xy, const double* P, int32_t n_images,
                              int32_t* ws, double* X, int32_t* n_obs, int32_t* err,
                              hipStream_t st) {
  if (n_nodes <= 0) return hipSuccess;
  // The totals (8 bytes), then counts (later starts), ranks, member lists and
  // the track list.
  unsigned long long* totals = reinterpret_cast<unsigned long long*>(ws);
  int2* tracks = reinterpret_cast<int2*>(ws + 2);
  int32_t* cnt = ws + 2 + n_nodes + (n_nodes & 1);
  int32_t* rank = cnt + n_nodes;
  int32_t* members = rank + n_nodes;
  const dim3 grid(blocks_for(n_nodes));
  hipLaunchKernelGGL(fill_i32_kernel, grid, dim3(256), 0, st, cnt, n_nodes);
  hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(256), 0, st, ws, int64_t(2));
  hipLaunchKernelGGL(tri_count_kernel, grid, dim3(256), 0, st, label, node_image, n_images,
                     n_nodes, cnt, rank, err);
  hipLaunchKernelGGL(tri_start_kernel, dim3(uint32_t((n_nodes + 1023) / 1024)), dim3(1024), 0, st,
                     label, rank, n_nodes, cnt, tracks, totals, X, n_obs);
  hipLaunchKernelGGL(tri_scatter_kernel, grid, dim3(256), 0, st, label, rank, n_nodes, cnt,
                     members);
  const int64_t most = (n_nodes / 2 * kTrackLanes + 255) / 256;
  hipLaunchKernelGGL(tri_solve_kernel,
                     dim3(uint32_t(std::max<int64_t>(1, std::min<int64_t>(kSolveBlocks, most)))),
                     dim3(256), 0, st, node_image, node_xy, P, n_images, cnt, tracks, totals,
                     members, X);
  return hipGetLastError();
}

}  // namespace sfm
