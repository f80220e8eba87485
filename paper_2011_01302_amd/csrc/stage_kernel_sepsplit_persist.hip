// Stage kernel variant KV_SEPSPLIT, persistent launch: the light tiles plus split SEPCONV tiles.  One translation unit per
// (variant, launch kind) so that the kernels build in parallel (see
// stage_kernel.h and stage_launch.cpp).
#include "stage_kernel.h"

namespace ios {

void *stage_kernel_fn_sepsplit_persist() { return (void *)ios_split_kernel<KV_SEPSPLIT, true>; }

hipError_t stage_launch_sepsplit_persist(const int4 *t, int words, const StageArgs &a, int grid, int lds, hipStream_t s) {
  hipLaunchKernelGGL((ios_split_kernel<KV_SEPSPLIT, true>), dim3(grid), dim3(kThreads), lds, s, t, words, a);
  return hipGetLastError();
}

}  // namespace ios
