// The 4-bit quantizer of one K or V row (quant_rows.hip states the format), for the lanes that share the row.
#pragma once
#include "device_util.h"

namespace locret {

__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) { return (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16); }

typedef unsigned int q4_u32x4 __attribute__((ext_vector_type(4)));

// A row of D bf16 values is shared by NP = D/16 lanes (a power-of-two block of NPP lanes is reserved for it); lane p
// owns two pieces of 8 dims, [8p, 8p+8) and [D/2 + 8p, D/2 + 8p + 8): eight rotary pairs (i, i + D/2).  Piece ids
// run 0 .. 2 NP - 1 in dim order (piece q = dims [8q, 8q+8)); a quantization group is four consecutive pieces.
template <int D>
struct Q4Lanes {
  static constexpr int NP = D / 16;
  static constexpr int NPP = NP <= 4 ? 4 : 8;
};

// min and max of the group that piece `piece` belongs to, gathered from the lanes of the row (lane block starts at
// lane `base`): every lane offers the (min, max) of its two pieces.
template <int D>
__device__ __forceinline__ void group_min_max(int piece, int base, float mn0, float mx0, float mn1, float mx1, float& lo, float& hi) {
  constexpr int NP = Q4Lanes<D>::NP;
  const int g = piece >> 2;
  lo = INFINITY;
  hi = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int q = 4 * g + j;                      // a member piece: slot q / NP of lane q % NP
    const int src = base + q % NP;
    const float a0 = __shfl(mn0, src, 64), a1 = __shfl(mn1, src, 64);
    const float b0 = __shfl(mx0, src, 64), b1 = __shfl(mx1, src, 64);
    lo = fminf(lo, q / NP ? a1 : a0);
    hi = fmaxf(hi, q / NP ? b1 : b0);
  }
}

// codes of 8 values against (lo, s); returns the packed dword (dim e in nibble e) and leaves the dequantized values
__device__ __forceinline__ uint32_t quant8(float (&x)[8], float lo, float s) {
  uint32_t w = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float c = fminf(fmaxf(rintf(__fdiv_rn(x[e] - lo, s)), 0.f), 15.f);
    w |= (uint32_t)c << (4 * e);
    x[e] = fmaf(c, s, lo);
  }
  return w;
}

__device__ __forceinline__ void unpack8_bf16(q4_u32x4 v, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = bf2f((bf16_t)(v[i] & 0xffffu));
    x[2 * i + 1] = bf2f((bf16_t)(v[i] >> 16));
  }
}
__device__ __forceinline__ q4_u32x4 pack8_bf16(const float (&x)[8]) {
  q4_u32x4 r = {pack2_bf16(x[0], x[1]), pack2_bf16(x[2], x[3]), pack2_bf16(x[4], x[5]), pack2_bf16(x[6], x[7])};
  return r;
}

// Lane p's two pieces of a row: the code dwords, each piece's (scale, minimum), and the dequantized values.
struct Q4Pieces {
  float a[8], b[8];
  uint32_t w0, w1;
  float s0, lo0, s1, lo1;
  __device__ __forceinline__ void rotate(const float2 (&cs)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float lo = a[e] * cs[e].x - b[e] * cs[e].y, hi = b[e] * cs[e].x + a[e] * cs[e].y;
      a[e] = lo;
      b[e] = hi;
    }
  }
};

// every lane of the row's block, which starts at lane `base`, calls it together (spare lanes with a clamped p)
template <int D>
__device__ __forceinline__ Q4Pieces quantize_pieces(const bf16_t* __restrict__ src, int p, int base) {
  constexpr int NP = Q4Lanes<D>::NP;
  Q4Pieces r;
  unpack8_bf16(*(const q4_u32x4*)(src + 8 * p), r.a);
  unpack8_bf16(*(const q4_u32x4*)(src + D / 2 + 8 * p), r.b);
  float mn0 = r.a[0], mx0 = r.a[0], mn1 = r.b[0], mx1 = r.b[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) {
    mn0 = fminf(mn0, r.a[e]); mx0 = fmaxf(mx0, r.a[e]);
    mn1 = fminf(mn1, r.b[e]); mx1 = fmaxf(mx1, r.b[e]);
  }
  float hi0, hi1;
  group_min_max<D>(p, base, mn0, mx0, mn1, mx1, r.lo0, hi0);
  group_min_max<D>(NP + p, base, mn0, mx0, mn1, mx1, r.lo1, hi1);
  r.s0 = bf2f(f2bf(__fdiv_rn(hi0 - r.lo0, 15.0f)));
  r.s1 = bf2f(f2bf(__fdiv_rn(hi1 - r.lo1, 15.0f)));
  r.s0 = r.s0 > 0.f ? r.s0 : 1.0f;
  r.s1 = r.s1 > 0.f ? r.s1 : 1.0f;
  r.w0 = quant8(r.a, r.lo0, r.s0);
  r.w1 = quant8(r.b, r.lo1, r.s1);
  return r;
}

// codes, and from the first lane of every group its (scale, minimum)
template <int D>
__device__ __forceinline__ void store_pieces(const Q4Pieces& r, uint8_t* __restrict__ qrow, int p) {
  constexpr int NP = Q4Lanes<D>::NP;
  *(uint32_t*)(qrow + 4 * p) = r.w0;
  *(uint32_t*)(qrow + D / 4 + 4 * p) = r.w1;
  if ((p & 3) == 0) *(uint32_t*)(qrow + D / 2 + 4 * (p >> 2)) = (uint32_t)f2bf(r.s0) | ((uint32_t)f2bf(r.lo0) << 16);
  if (((NP + p) & 3) == 0) *(uint32_t*)(qrow + D / 2 + 4 * ((NP + p) >> 2)) = (uint32_t)f2bf(r.s1) | ((uint32_t)f2bf(r.lo1) << 16);
}

}  // namespace locret
