// float32 chunk attention (Eq. 1) and retaining head (Section 3.3) on the float32 matrix instructions of gfx950
// (v_mfma_f32_16x16x4_f32: float32 products and sums, 256 flop per clock and CU).
//
// The instruction takes one float per lane of each operand, A[i = lane % 16][k = lane / 16] and
// B[k = lane / 16][j = lane % 16], and leaves C[4 (lane / 16) + r][lane % 16] in register r.  A contraction may run over
// its terms in any order as long as both operands agree, so every operand is fetched 16 bytes at a time: a lane's four
// consecutive elements feed four instructions.  Operands come straight from memory, only the keys by way of LDS.  The wavefronts of
// a workgroup divide the contraction (attention: the keys) among themselves, so no element of W1 and of the inputs
// (attention: of keys and values; every wavefront reads the queries) is read twice by a workgroup, and meet in LDS at the
// end.  That also fills the chip at the small sizes float32 layers have: 512 tokens x 8 heads are 256 workgroups of 8
// wavefronts.
#include "append_body.h"
#include "device_util.h"
#include "kernels.h"
#include "launch_rules.h"
#include "select_body.h"

namespace locret {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int F32_NW = 8;                      // wavefronts per workgroup

// Launches number their workgroups through, in rows of at most F32_ROW: one grid dimension of 512-thread workgroups ends at 2^23,
// which 2^27 tokens of the retaining head (a few milliseconds' work) are beyond.  The last row may be short of workgroups to do.
constexpr int64_t F32_ROW = 1 << 16;
static dim3 f32_rows(int64_t n, unsigned z = 1) {
  return dim3((unsigned)(n < F32_ROW ? n : F32_ROW), (unsigned)((n + F32_ROW - 1) / F32_ROW), z);
}
__device__ __forceinline__ int f32_workgroup() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }

// N consecutive floats (N = 1, 2, 4; 4 N bytes aligned)
template <int N> __device__ __forceinline__ void load_floats(const float* p, float* x) {
  if constexpr (N == 4) { const float4 v = *(const float4*)p; x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
  else if constexpr (N == 2) { const float2 v = *(const float2*)p; x[0] = v.x; x[1] = v.y; }
  else x[0] = *p;
}

// ---- attention -----------------------------------------------------------------------------------------------------
// Workgroup = QB blocks of 16 queries of one head; wavefront w takes key tiles w, w + 8, ... of 16 keys.
//   S^T[key][query] = K Q^T       A: lane (key, kg) holds dims 16 c + 4 kg .. + 3 of its key row, B: the query's same dims
//   O^T[dim][query] += V^T P^T    B: P^T from the S accumulator as it lies (key 4 kg + r), A: lane (i, kg) holds dims
//                                 4 i .. + 3 (+ 64 ...) of value row 4 kg + r, so accumulator row i of block b is dim 4 i + b
// The running max moves only when some logit exceeds it by 8 binary orders.  Bound by the matrix instructions and, for
// one query block, by the L2 (a key row is read once per 16 queries): 512 tokens on 1024 + 512 units,
// 8 heads x 64: 21 us against 199 of a vector-ALU kernel with K, V and P tiles in LDS; the error against 64 bits halved.
// QB = 2 where that still gives every CU a workgroup.
// The keys pass through LDS, two tiles of the wavefront's own: straight into the operand's layout 16 neighbouring lanes read 16 rows, a cache
// line each (4096 tokens in chunks of 512 on 64 dims 236 -> 227 us, 2900 tokens in chunks of 921 with rotary 205 -> 195, 128 dims
// 719 -> 680).  What is left is not memory: without any load in the loop a step on 1536 keys takes 19.2 us instead of 21.0, without either
// product 16.5.  (Two tiles ahead in registers 245 us, 16 wavefronts 255, the next tile's S beside the softmax 230.)
// The first n_sel workgroups of the launch do not attend: each carries out the selection of one KV head, which depends on
// the scores only, and sums their partials.  As a launch of its own it took 8.4 us behind 20 us of attention (2 heads, 1472
// candidates): 4096 tokens in chunks of 512 333 us, 279 us in this form.
typedef __attribute__((address_space(3))) void* f32_lds_ptr;
// Rows of D floats in LDS: what the pieces of row r are exchanged by, so that 16 lanes that read the same piece of 16 rows meet 16
// different groups of four banks (row r starts at group (r D / 4) mod 16)
template <int D> __device__ __forceinline__ int f32_swizzle(int r) {
  return D == 16 ? (r >> 2) & 3 : D == 32 || D == 96 ? (r >> 1) & 7 : r & 15;
}
constexpr int F32_SEL_MAXR = 24;               // keys per thread of a selection workgroup: up to 12288 candidates per head
template <int D, int QB>
__global__ __launch_bounds__(F32_NW * 64) void attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ Kx,
                                                               const float* __restrict__ V, float* __restrict__ out, int Tn,
                                                               int h, int g, int cap, int n_c_common, float c_log2, HeadLens n_c_h, int n_ttiles,
                                                               SelectArgs sel, int n_sel) {
  constexpr int NC = D / 16;                   // 16-dim pieces of a row = dim blocks of O^T
  constexpr int V4 = D / 64 * 64;              // dims fetched four (then two, one) per lane
  constexpr int V2 = (D - V4) / 32 * 32;
  constexpr int ROW = D + 2;
  constexpr int TILE = 16 * D;                 // floats of a key tile
  constexpr int RED = F32_NW * 16 * QB * ROW, SEL = select_body_smem_words(F32_NW * 64, 1), KEYS = F32_NW * 2 * TILE;
  __shared__ __attribute__((aligned(1024))) float smem[RED > SEL ? (RED > KEYS ? RED : KEYS) : (SEL > KEYS ? SEL : KEYS)];
  const int wg = f32_workgroup();
  if (wg < n_sel) {
    select_reg_body<F32_SEL_MAXR, F32_NW * 64, 1>(sel, wg, (uint32_t*)smem);
    return;
  }
  float (*red)[16 * QB][ROW] = (float (*)[16 * QB][ROW])smem;             // O, max, sum of every wavefront
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, kg = lane >> 4;
  const int item = wg - n_sel, j = item / n_ttiles, m = j / g;
  if (j >= h) return;
  const int n_c = head_len(n_c_h, m, n_c_common);
  const int t0 = (n_ttiles - 1 - item % n_ttiles) * (16 * QB);            // longest key ranges first
  const int n_keys = n_c + min(Tn, t0 + 16 * QB);
  const float* Kb = Kx + (int64_t)m * cap * D;
  const float* Vb = V + (int64_t)m * cap * D;

  float qf[QB][NC][4];
  int limit[QB];                               // last visible slot of this lane's query
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int t = min(t0 + b * 16 + i16, Tn - 1);
    limit[b] = n_c + t;
    const float* qp = q + ((int64_t)t * h + j) * D + kg * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      load_floats<4>(qp + c * 16, qf[b][c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[b][c][e] *= c_log2;      // logits in log2 units
    }
  }
  f32x4 o[QB][NC];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    m_run[b] = -INFINITY;
    l_run[b] = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[b][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float kf[NC][4], vf[4][NC];
  // This wavefront's two key tiles in LDS.  Position p of row r holds the row's 16-byte piece p ^ f32_swizzle(r).
  float* const keys = smem + wave * (2 * TILE);
  constexpr int PIECES = D / 4;                // of a row
  int piece[NC];                               // where in the tile the pieces that this lane requests lie (bytes)
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int x = i * 64 + lane, r = x / PIECES;
    piece[i] = (r * PIECES + ((x % PIECES) ^ f32_swizzle<D>(r))) * 16;
  }
  auto request_k = [&](int k0, int buf) __attribute__((always_inline)) {      // rows past the end arrive as zeros (masked below)
    __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Kb + (int64_t)k0 * D), 0, min(16, n_keys - k0) * (D * 4), 0x00020000);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int at = piece[i];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (f32_lds_ptr)(keys + buf * TILE + i * 256), 16, at, 0, 0, 0);
    }
  };
  auto read_k = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) load_floats<4>(keys + buf * TILE + i16 * D + (((4 * c + kg) ^ f32_swizzle<D>(i16)) * 4), kf[c]);
  };
  auto load_v = [&](int k0) {                  // rows past the end repeat the last one
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* vp = Vb + (int64_t)min(k0 + 4 * kg + r, n_keys - 1) * D;
#pragma unroll
      for (int x = 0; x < V4 / 64; ++x) load_floats<4>(vp + x * 64 + i16 * 4, &vf[r][x * 4]);
      if constexpr (V2 > 0) load_floats<2>(vp + V4 + i16 * 2, &vf[r][V4 / 16]);
      if constexpr (D - V4 - V2 > 0) load_floats<1>(vp + V4 + V2 + i16, &vf[r][(V4 + V2) / 16]);
    }
  };
  int k0 = wave * 16, buf = 0;
  if (k0 < n_keys) request_k(k0, 0);
  for (; k0 < n_keys; k0 += F32_NW * 16, buf ^= 1) {
    // all that is in flight here is this tile's keys, requested a tile ago (the tiles are the wavefront's own: no barrier)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    read_k(buf);
    load_v(k0);
    if (k0 + F32_NW * 16 < n_keys) request_k(k0 + F32_NW * 16, buf ^ 1);
    f32x4 s[QB][2];
#pragma unroll
    for (int b = 0; b < QB; ++b) s[b][0] = s[b][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < QB; ++b) s[b][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[b][c][e], s[b][e & 1], 0, 0, 0);
    float p[QB][4];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[b][r] = s[b][0][r] + s[b][1][r];
        if (k0 + 4 * kg + r > limit[b]) p[b][r] = -INFINITY;
        mx = fmaxf(mx, p[b][r]);
      }
      if (__any(mx > m_run[b] + 8.f)) {        // the four lanes of a query move together: its accumulators are shared
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run[b], mx);
        const float alpha = m_run[b] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[b] - m_new);
        l_run[b] *= alpha;
#pragma unroll
        for (int c = 0; c < NC; ++c) o[b][c] *= alpha;
        m_run[b] = m_new;
      }
      const float m_use = m_run[b] == -INFINITY ? 0.f : m_run[b];         // no key of this query seen yet: every p is 0
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[b][r] = __builtin_amdgcn_exp2f(p[b][r] - m_use);
        l_run[b] += p[b][r];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int b = 0; b < QB; ++b) o[b][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][c], p[b][r], o[b][c], 0, 0, 0);
  }
  __syncthreads();                             // the results go where the key tiles were
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    l_run[b] += __shfl_xor(l_run[b], 16, 64);
    l_run[b] += __shfl_xor(l_run[b], 32, 64);
    float* row = red[wave][b * 16 + i16];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * kg + r;              // accumulator row; its dim by the piece of the row that block c came from
        const int dim = c < V4 / 16 ? (c / 4) * 64 + i * 4 + c % 4
                                    : c < (V4 + V2) / 16 ? V4 + i * 2 + (c - V4 / 16) : V4 + V2 + i;
        row[dim] = o[b][c][r];
      }
    if (kg == 0) {
      row[D] = m_run[b];
      row[D + 1] = l_run[b];
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * QB * D; idx += F32_NW * 64) {
    const int qi = idx / D, e = idx % D, t = t0 + qi;
    if (t >= Tn) break;
    float M = red[0][qi][D];                   // key 0 is tile 0 of wavefront 0: finite
#pragma unroll
    for (int w = 1; w < F32_NW; ++w) M = fmaxf(M, red[w][qi][D]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < F32_NW; ++w) {
      const float wt = __builtin_amdgcn_exp2f(red[w][qi][D] - M);         // a wavefront without keys: 2^-inf = 0
      num = fmaf(wt, red[w][qi][e], num);
      den = fmaf(wt, red[w][qi][D + 1], den);
    }
    out[((int64_t)t * h + j) * D + e] = num / den;
  }
}

template <int D>
static void attn_f32_launch(const Dims& Dm, const float* q, const float* Kx, const float* V, float* out, int T, int n_c,
                            float scale, hipStream_t st, const HeadLens& hl, const SelectArgs* sel) {
  const float c_log2 = scale * 1.4426950408889634f;
  const SelectArgs sa = sel ? *sel : SelectArgs{};
  const int n_sel = sel ? Dm.h_kv : 0;
  const bool two = (int64_t)((T + 31) / 32) * Dm.h >= 256;
  const int n_ttiles = two ? (T + 31) / 32 : (T + 15) / 16;
  const dim3 grid = f32_rows(n_sel + (int64_t)n_ttiles * Dm.h);
  if (two)
    launch_kernel((attn_f32_kernel<D, 2>), grid, dim3(F32_NW * 64), 0, st, q, Kx, V, out, T, Dm.h, Dm.g, Dm.cap, n_c, c_log2, hl,
                  n_ttiles, sa, n_sel);
  else
    launch_kernel((attn_f32_kernel<D, 1>), grid, dim3(F32_NW * 64), 0, st, q, Kx, V, out, T, Dm.h, Dm.g, Dm.cap, n_c, c_log2, hl,
                  n_ttiles, sa, n_sel);
}

bool attention_f32_fuses_select(const Dims& Dm, int n_cand) {
  const int wseg = ((n_cand + F32_NW - 1) / F32_NW + 63) & ~63;
  return !Dm.bf16 && Dm.tune.fuse_select && wseg <= F32_SEL_MAXR * 64;
}

// As long as the sum hides behind the attention, which takes about the longer the more dims there are (a thread walks n_parts
// partials for each of its tokens).  A step with 2 KV heads, summed there or reduced before it: 16 dims, T = 1024: 16 partials 43.8,
// 48.8 us, 64 partials 94.3, 89.1, 256 partials 293.1, 239.7; 64 dims, T = 2048: 32 partials 281.1, 291.8, 128 partials 629.2, 658.7,
// 1024 partials 4529, 3995; 128 dims, T = 2048: 64 partials 746, 767.
bool attention_f32_sums_partials(const Dims& Dm, int n_parts, int T) {
  return (T + F32_NW * 64 - 1) / (F32_NW * 64) * n_parts <= 4 * Dm.d;
}

void launch_attention_f32(const Dims& Dm, const void* q, const void* Kx, const void* V, void* out, int T, int n_c, float scale,
                          hipStream_t st, const HeadLens& hl, const SelectArgs* sel) {
#define LOCRET_CASE(DD)                                                                                          \
  case DD:                                                                                                       \
    attn_f32_launch<DD>(Dm, (const float*)q, (const float*)Kx, (const float*)V, (float*)out, T, n_c, scale, st, hl, sel); \
    break;
  switch (Dm.d) {
    LOCRET_CASE(16)
    LOCRET_CASE(32)
    LOCRET_CASE(64)
    LOCRET_CASE(96)
    LOCRET_CASE(128)
  }
#undef LOCRET_CASE
}

// ---- retaining head ------------------------------------------------------------------------------------------------
// Workgroup = HB hidden units x 16 tokens; wavefront w takes contraction steps w, w + 8, ... of 16 elements (each inside one
// of q, k, v: the [q;k;v] row is read in place).  The wavefronts' sums are added in a fixed order, then SiLU and
// the product with W2; each workgroup writes its hidden block's partial part[nb][m][t].  HB = 32 or 64 by f32_hidden_units(): 768
// inputs x 256 hidden, 512 tokens 9.4 us with 32, 4096 tokens 34.5 with 64, 49.8 with 32; vector-ALU tiles of 64 x 64 took 95.7 at
// 512 tokens.  (Two steps' loads under way ahead of the present one: 64 units, 512 tokens 12.7 -> 14.4 us, 4096 34.5 -> 43.)
// APPEND 1 (2: with head-wise lengths): workgroups behind the n_nb hidden blocks, two of the append's each, append the chunk, which
// depends on nothing this launch does: a launch of 3.4 us less (4096 tokens in chunks of 512, 2 x 64 dims: 280 -> 272 us, with HB = 32 238).
constexpr int F32_TB = 16;
template <int HB, int APPEND>
__global__ __launch_bounds__(F32_NW * 64) void score_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                                const float* __restrict__ v, int Tn, int hd, int kvd,
                                                                const float* __restrict__ W1t, const float* __restrict__ W2f,
                                                                int K, int d_R, int h_kv, float* __restrict__ part, int part_T,
                                                                int n_nb, AppendArgs<float> ap) {
  if (APPEND && (int)blockIdx.z >= n_nb) {
    const int64_t wg = ((int64_t)((int)blockIdx.z - n_nb) * (gridDim.x * gridDim.y) + f32_workgroup()) * (F32_NW / 4) + (threadIdx.x >> 8);
    if (wg < (int64_t)ap.gx * ap.gy) append_any<float, APPEND == 2, false>(ap, (int)(wg % ap.gx), (int)(wg / ap.gx), threadIdx.x & 255);
    return;
  }
  constexpr int NA = HB / 16, UNITS = HB / 8;      // blocks of hidden units; units of a lane in the product with W2
  __shared__ float hs[F32_NW][F32_TB][HB + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, kg = lane >> 4;
  const int t0 = f32_workgroup() * F32_TB, nb = blockIdx.z, n0 = nb * HB;
  if (t0 >= Tn) return;
  const int t = min(t0 + i16, Tn - 1);
  const float* wp[NA];                          // hidden units past the last repeat it (no weight of W2 is applied to them)
#pragma unroll
  for (int a = 0; a < NA; ++a) wp[a] = W1t + (int64_t)min(n0 + a * 16 + i16, d_R - 1) * K + kg * 4;
  auto x_ptr = [&](int c) -> const float* {
    if (c < hd) return q + (int64_t)t * hd + c + kg * 4;
    if (c < hd + kvd) return k + (int64_t)t * kvd + (c - hd) + kg * 4;
    return v + (int64_t)t * kvd + (c - hd - kvd) + kg * 4;
  };
  f32x4 acc[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c = wave * 16; c < K; c += F32_NW * 16) {
    float x[4], w[NA][4];
    load_floats<4>(x_ptr(c), x);
#pragma unroll
    for (int a = 0; a < NA; ++a) load_floats<4>(wp[a] + c, w[a]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[a][e], x[e], acc[a], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) hs[wave][i16][a * 16 + 4 * kg + r] = acc[a][r];
  __syncthreads();
  for (int i = tid; i < F32_TB * HB; i += F32_NW * 64) {
    const int tl = i / HB, n = i % HB;
    float z = hs[0][tl][n];
#pragma unroll
    for (int w = 1; w < F32_NW; ++w) z += hs[w][tl][n];
    hs[0][tl][n] = z / (1.f + expf(-z));
  }
  __syncthreads();
  // eight lanes per score, UNITS hidden units each
  const int n_out = F32_TB * h_kv, hh_end = min(HB, d_R - n0);
  for (int i = tid; i < n_out * 8; i += F32_NW * 64) {
    const int o8 = i >> 3, tl = o8 % F32_TB, m = o8 / F32_TB, n1 = (i & 7) * UNITS;
    float sum = 0.f;
#pragma unroll
    for (int n = 0; n < UNITS; ++n)
      if (n1 + n < hh_end) sum = fmaf(hs[0][tl][n1 + n], W2f[(int64_t)(n0 + n1 + n) * h_kv + m], sum);
    sum += __shfl_xor(sum, 1, 64);
    sum += __shfl_xor(sum, 2, 64);
    sum += __shfl_xor(sum, 4, 64);
    if ((i & 7) == 0 && t0 + tl < Tn) part[((int64_t)nb * h_kv + m) * part_T + t0 + tl] = sum;
  }
}

int score_parts_f32(const Dims& D) { return (D.d_R + 63) / 64; }

int launch_score_f32(const Dims& D, const void* q, const void* k, const void* v, int T, const void* W1t, const float* W2f,
                     float* part, hipStream_t st, const ChunkAppend* app) {
  // the partials have to fit into the workspace, which is not larger for them, and into the static scratch
  const size_t room = D.part_floats < SCORE_FINE_FLOATS ? D.part_floats : SCORE_FINE_FLOATS;
  const int hb = f32_hidden_units(T, D.h_kv, D.d_R, (int64_t)room), nb = (D.d_R + hb - 1) / hb;
  dim3 grid = f32_rows((T + F32_TB - 1) / F32_TB, nb);
  AppendArgs<float> ap = {};
  if (app) {
    ap = append_args<float>(D, app->q, k, v, T, app->n_c, app->seen, app->c, app->qr, app->tab, nullptr, app->n_c_h, nullptr, 0);
    const int64_t layer = (int64_t)grid.x * grid.y * (F32_NW / 4);
    grid.z += (unsigned)(((int64_t)ap.gx * ap.gy + layer - 1) / layer);
  }
#define LOCRET_SCORE(HB, AP)                                                                                                     \
  launch_kernel((score_f32_kernel<HB, AP>), grid, dim3(F32_NW * 64), 0, st, (const float*)q, (const float*)k, (const float*)v, T, \
                D.h * D.d, D.h_kv * D.d, (const float*)W1t, W2f, D.K, D.d_R, D.h_kv, part, T, nb, ap)
#define LOCRET_SCORE_AP(HB)                          \
  if (!app) LOCRET_SCORE(HB, 0);                     \
  else if (ap.n_c_h.ragged) LOCRET_SCORE(HB, 2);     \
  else LOCRET_SCORE(HB, 1)
  if (hb == 32) { LOCRET_SCORE_AP(32); } else { LOCRET_SCORE_AP(64); }
#undef LOCRET_SCORE_AP
#undef LOCRET_SCORE
  return nb;
}

}  // namespace locret
