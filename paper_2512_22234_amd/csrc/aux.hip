// float32 -> bf16 conversion of the inputs of callers that hand the library
// float32 tensors (the kernels widen their own results).
#include "device.hpp"
#include "kernels.hpp"

namespace bd {
namespace {

constexpr int CAST_PER = 8;                // elements per thread
constexpr int CAST_BLOCK = 256 * CAST_PER;  // ... and per workgroup

struct CastParams {
  CastList c;
  unsigned first[CAST_MAX];  // first workgroup of each tensor
};

// Every tensor of a call in one launch (a launch per tensor was most of a small
// call: 5 + 3 of them, one element per thread, around the two backward
// kernels), 32 bytes in and 16 bytes out per thread: bound by HBM.
__global__ __launch_bounds__(256) void cast_f32_bf16_kernel(CastParams p) {
  int k = 0;
#pragma unroll
  for (int t = 1; t < CAST_MAX; ++t)
    if (t < p.c.count && blockIdx.x >= p.first[t]) k = t;
  const size_t i = ((size_t)(blockIdx.x - p.first[k]) * 256 + threadIdx.x) * CAST_PER;
  if (i >= p.c.n[k]) return;
  const float* x = static_cast<const float*>(p.c.src[k]) + i;
  const f32x4 a = *reinterpret_cast<const f32x4*>(x), b = *reinterpret_cast<const f32x4*>(x + 4);
  bf16x8 y;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    y[e] = (bf16)a[e];
    y[e + 4] = (bf16)b[e];
  }
  *reinterpret_cast<bf16x8*>(static_cast<bf16*>(p.c.dst[k]) + i) = y;
}

}  // namespace

hipError_t launch_cast_f32_to_bf16(const CastList& c, hipStream_t st, LaunchEvents ev) {
  CastParams p;
  p.c = c;
  unsigned blocks = 0;
  for (int t = 0; t < c.count; ++t) {
    p.first[t] = blocks;
    blocks += (unsigned)((c.n[t] + CAST_BLOCK - 1) / CAST_BLOCK);
  }
  hipExtLaunchKernelGGL(cast_f32_bf16_kernel, dim3(blocks), dim3(256), 0, st, ev.start, ev.stop, 0, p);
  return hipGetLastError();
}

}  // namespace bd
