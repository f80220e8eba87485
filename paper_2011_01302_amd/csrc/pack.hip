// Weights of the split conv tiles, packed on the device: a network's weights
// or a merge stage's are uploaded once as they are and split here (the host
// took 6 to 20 ns a weight for it, which a schedule's first pass would pay).
#include "ios_internal.h"

namespace ios {

namespace {

typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// Thread (b, chunk, tap, lane): output channel 32 b + lane % 32, input
// channels 16 chunk + 8 (lane / 32) .. + 7; per part 8 bf16 in 16 bytes.
__global__ __launch_bounds__(256) void pack_split_kernel(const float *w, int cout, int cin, int taps, int nch,
                                                          int groups, uintx4 *out) {
  const int gid = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (gid >= groups) return;
  const int tap = gid % taps, bc = gid / taps, chunk = bc % nch, b = bc / nch;
  const int n = b * 32 + (lane & 31), c0 = chunk * kSplitCK + (lane >> 5) * 8;
  uintx4 p[3];
  for (int i = 0; i < 3; ++i) p[i] = uintx4{0, 0, 0, 0};
  for (int j = 0; j < 8; ++j) {
    if (n >= cout || c0 + j >= cin) continue;
    float v = w[((size_t)n * cin + c0 + j) * taps + tap];
    for (int i = 0; i < 3; ++i) {
      // the nearest bf16 to what is left (ties to even; the weights are finite and below 2^40)
      const uint32_t u = __builtin_bit_cast(uint32_t, v), r = (u + 0x7FFFu + ((u >> 16) & 1)) & 0xFFFF0000u;
      p[i][j >> 1] |= (r >> 16) << ((j & 1) * 16);
      v -= __builtin_bit_cast(float, r);
    }
  }
  for (int i = 0; i < 3; ++i) out[((size_t)gid * 3 + i) * 64 + lane] = p[i];
}

}  // namespace

size_t split_words(int cout, int cin, int kh, int kw) {
  return (size_t)((cout + 31) / 32) * ((cin + kSplitCK - 1) / kSplitCK) * kh * kw * kSplitWords;
}

void pack_conv_split(const float *w, int cout, int cin, int kh, int kw, float *d_out, hipStream_t stream) {
  const int taps = kh * kw, nch = (cin + kSplitCK - 1) / kSplitCK, groups = (cout + 31) / 32 * nch * taps;
  const size_t bytes = (size_t)cout * cin * taps * sizeof(float);
  float *raw = nullptr;
  hip_check(hipMalloc(&raw, bytes), "hipMalloc(weights)");
  hipError_t e = hipMemcpy(raw, w, bytes, hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(pack_split_kernel, dim3((groups + 3) / 4), dim3(256), 0, stream, raw, cout, cin, taps, nch, groups,
                       (uintx4 *)d_out);
    e = hipGetLastError();
    const hipError_t s = hipStreamSynchronize(stream);
    if (e == hipSuccess) e = s;
  }
  (void)hipFree(raw);
  hip_check(e, "pack_conv_split");
}

}  // namespace ios
