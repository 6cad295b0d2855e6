// Staged matching of coarse features (Section 4): the pair's first stage
// matches a prefix of the query image's features against a prefix of the
// target image's, a second stage the next run of queries against the same
// targets.  Features are registered in decreasing scale, so a prefix is the
// highest-scale part of an image; a stage is the exhaustive matcher run on
// views that point into the registered arrays.  The two stages of a pair are
// neighbours in one batch: the second's kernels read on the device whether the
// first found enough, and one emission writes each pair's rows of both stages
// one after the other in query order.  (With the counts back on the host
// between the stages, a merge of both stages' rows and the rest of two calls,
// 1,770 pairs took 947 us for 508 of matching; 680 so.)
#include <algorithm>

#include "sfm_internal.h"

namespace sfm {
namespace {

__global__ __launch_bounds__(256) void make_views_kernel(const ImageDev* images,
                                                         const int32_t* spec, int32_t n_views,
                                                         ImageDev* views) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_views;
       i += gridDim.x * blockDim.x) {
    const int32_t img = spec[3 * i], first = spec[3 * i + 1], count = spec[3 * i + 2];
    ImageDev d = images[img];
    d.xy += 2 * int64_t(first);
    d.desc += 128 * int64_t(first);
    d.norm2 += first;
    d.cword += first;
    d.sxy = nullptr;   // a view has no spatial order
    d.sj = nullptr;
    d.box = nullptr;
    d.outer = nullptr;
    d.n = count;
    views[i] = d;
  }
}

__global__ __launch_bounds__(256) void stage_outputs_kernel(BatchView v, int32_t n_pairs,
                                                            const int64_t* offset2,
                                                            const int64_t* n_cmp2,
                                                            int64_t* offset, int64_t* n_cmp,
                                                            int32_t* found) {
  const int32_t k = int32_t(blockIdx.x * blockDim.x + threadIdx.x);
  if (k > n_pairs) return;
  offset[k] = offset2[2 * int64_t(k)];
  if (k == n_pairs) return;
  if (n_cmp) n_cmp[k] = n_cmp2[2 * int64_t(k)] + n_cmp2[2 * int64_t(k) + 1];
  found[k] = int32_t(v.counters[2 * int64_t(k)].accepted);
}

int32_t grid_for(int64_t n, int64_t per) {
  return int32_t(std::max<int64_t>(1, std::min<int64_t>((n + per - 1) / per, 65535)));
}

}  // namespace

hipError_t launch_make_views(const ImageDev* images, const int32_t* spec, int32_t n_views,
                             ImageDev* views, hipStream_t st) {
  if (n_views <= 0) return hipSuccess;
  hipLaunchKernelGGL(make_views_kernel, dim3(grid_for(n_views, 256)), dim3(256), 0, st, images,
                     spec, n_views, views);
  return hipGetLastError();
}

hipError_t launch_stage_outputs(const BatchView& v, int32_t n_pairs, const int64_t* offset2,
                                const int64_t* n_cmp2, int64_t* offset, int64_t* n_cmp,
                                int32_t* found, hipStream_t st) {
  if (n_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL(stage_outputs_kernel, dim3(n_pairs / 256 + 1), dim3(256), 0, st, v, n_pairs,
                     offset2, n_cmp2, offset, n_cmp, found);
  return hipGetLastError();
}

}  // namespace sfm
