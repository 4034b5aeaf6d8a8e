// The last step of the retaining head for a single token (Section 3.3): the product of its hidden activations with one
// column of W2, formed by a workgroup of 256 threads.
#pragma once
#include <hip/hip_runtime.h>

namespace locret {

// sum_r act[r] W2f[r][m] in every thread; red: 4 floats of LDS that nothing else uses
__device__ __forceinline__ float token_score(const float* __restrict__ act, int d_R, const float* __restrict__ W2f, int h_kv, int m,
                                             float* red) {
  const int tid = threadIdx.x;
  float s = 0.f;
  for (int r = tid; r < d_R; r += 256) s = fmaf(act[r], W2f[(int64_t)r * h_kv + m], s);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

}  // namespace locret
