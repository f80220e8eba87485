// Stage kernel variant KV_SPLIT, one workgroup per tile: the light tiles plus split conv tiles.  One translation unit per
// (variant, launch kind) so that the kernels build in parallel (see
// stage_kernel.h and stage_launch.cpp).
#include "stage_kernel.h"

namespace ios {

void *stage_kernel_fn_split() { return (void *)ios_split_kernel<KV_SPLIT, false>; }

hipError_t stage_launch_split(const int4 *t, int words, const StageArgs &a, int grid, int lds, hipStream_t s) {
  hipLaunchKernelGGL((ios_split_kernel<KV_SPLIT, false>), dim3(grid), dim3(kThreads), lds, s, t, words, a);
  return hipGetLastError();
}

}  // namespace ios
