// The retaining head of a single token (Section 3.3) in two steps: its hidden activations, a wavefront per hidden unit, and
// their product with one column of W2, a workgroup per KV head.
#pragma once
#include "device_util.h"

namespace locret {

// act[r] = SiLU(W1t[r][:] . [q; k; v]) by one wavefront, 16 bytes per lane at a time (hd, kvd and K are multiples of 64: 8
// elements lie in one of q, k, v)
__device__ __forceinline__ void token_hidden(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                             int hd, int kvd, const bf16_t* __restrict__ W1t, int K, int r, float* __restrict__ act) {
  const int lane = threadIdx.x & 63;
  const bf16_t* w = W1t + (int64_t)r * K;
  float acc = 0.f;
#pragma unroll 4
  for (int c = lane * 8; c < K; c += 512) {
    const bf16_t* x = c < hd ? q + c : c < hd + kvd ? k + (c - hd) : v + (c - hd - kvd);
    Vec16<bf16_t> a, b;
    a.raw = *(const uint4*)(w + c);
    b.raw = *(const uint4*)x;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(a.get(e), b.get(e), acc);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) act[r] = acc * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc * -1.4426950408889634f));
}

// sum_r act[r] W2f[r][m] by the first 256 threads of a workgroup, in every thread; red: 4 floats of LDS that nothing else
// uses.  The loads of four hidden units are requested together.
__device__ __forceinline__ float token_score(const float* __restrict__ act, int d_R, const float* __restrict__ W2f, int h_kv, int m,
                                             float* red) {
  const int tid = threadIdx.x;
  if (tid < 256) {
    float s = 0.f;
    for (int r0 = tid; r0 < d_R; r0 += 4 * 256) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = min(r0 + 256 * i, d_R - 1);
        a[i] = act[r];
        w[i] = W2f[(int64_t)r * h_kv + m];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (r0 + 256 * i < d_R) s = fmaf(a[i], w[i], s);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((tid & 63) == 0) red[tid >> 6] = s;
  }
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

}  // namespace locret
