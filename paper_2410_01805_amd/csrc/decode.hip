// Decode step: attention of ONE new token over the retained cache (Eq. 1 with B = 1; the generate
// step that closes Algorithm 1).  The work is a single pass over K and V of every KV head, so the
// kernel is built for HBM bandwidth: rows go from memory to registers, not through LDS.
//
// Split-K over the key axis: a workgroup (split, m) owns a range of keys of KV head m and serves the query heads of its
// group, G = 4, 2 or 1 at a time.
//
// bf16 storage, head dims that are multiples of 32: both products run on the matrix cores (v_mfma_f32_16x16x32_bf16), a
// wavefront takes 32 keys at a time, straight from memory to registers in the layout of the operands (DecTile).  S^T = K Q^T has
// the heads as columns; O = P V the heads as rows and a dim as a column, 16 dims an instruction, so V's rows are needed
// dim by dim: two keys' words make two operand words with two byte permutations, half an instruction for each value where
// the vector form takes a multiply-add per value and head.  The 16 columns of S^T hold every head 16 / G times.  The copies
// carry the probability in pieces: its upper 8 significant bits, the next 8, the last 8, each exact in bf16, so the
// products are those of the 32-bit probability (error against 64 bits as with vector multiply-adds).  Nothing passes
// through LDS before the wavefronts' results are merged.  The running max of a column moves only when a logit exceeds it by
// 8 binary orders.  The first keys and values are requested before the query is rotated, the next ones as soon as the
// registers of the present ones are free.  Bound by HBM on long caches, by the chain of launch, first loads and merge
// on short ones.  Split kernel alone, against the vector form (which held 8 dims x 4 heads of a row in a lane): 8 heads x
// 16.4K x 128 dims 16.6 -> 14.1 us (67 MB), 8 x 6.1K 10.4 -> 7.6, 8 x 2K 8.2 -> 6.4, 8 x 16.4K x 64 12.1 -> 8.7, 32 x 8.2K x 96
// 17.2 -> 16.8, 32 x 2K x 96 6.3 -> 6.7 (a token there, with the merge, 9.4 -> 8.8; one query head fills a sixteenth of the matrix
// form's columns, and the vector form is still the slower one: 11.0).
//
// Other types: a key row is spread over LPR lanes (16 bytes per lane, padded to a power of two), so one load instruction of a
// wavefront fetches 64 / LPRP whole rows, contiguous in memory.  Each lane keeps the query values of its own dims for G heads
// and a logit is G short dot products plus a butterfly over the lanes of the row, which then share the probability and
// accumulate p * v for their dims.  Online softmax with a lazily raised max as in the prefill kernels, one decision per UN rows.
//
// The (max, sum, vector) triples of a workgroup are merged through LDS, those of the splits by decode_merge_kernel.
//
// The step is two launches.  The split kernel goes over the units already in the cache and rotates the
// (un-rotated) query itself; one more workgroup per KV head takes the new token: one more partial (logit from
// the rotated query and key, value row, sum 1) and the append to the cache (K, V, the rotated-key shadow, the
// original position, and a NaN score when the caller does not score generated tokens).  The merge kernel
// combines the partials.  For a scored token further workgroups of the first launch form its hidden activations and
// further ones of the second its scores: with the activations in a launch of their own in front (5 us) and their
// product in the token's workgroup, a 611-token prompt and 8 scored tokens took 181 us, 152 us in this form.
// The token's own row and the query are requested before anything is computed, and the token's workgroup skips the
// merge of its empty row slots: 152 -> 145 us there.
// A separate append launch cost 15 % of the step.
#include <stdlib.h>

#include <type_traits>

#include "attn_common.h"
#include "kernels.h"
#include "launch_rules.h"
#include "quant_row.h"
#include "token_score.h"

namespace locret {

constexpr int DEC_THREADS = 256;
constexpr int DEC_UN = 4;               // rows per lane group between max decisions
constexpr float DEC_RESCALE_LOG2 = 8.f;

template <int X> struct Pow2Ceil { static constexpr int value = X <= 1 ? 1 : 2 * Pow2Ceil<(X + 1) / 2>::value; };
template <> struct Pow2Ceil<1> { static constexpr int value = 1; };

// The new token of a decode step and where it goes (all device pointers; q, k, v un-rotated).
struct DecodeToken {
  const void* q;          // [h][d]
  const void* k;          // [h_kv][d]
  const void* v;          // [h_kv][d]
  const float2* tab;      // rotary table, or NULL
  void* K;                // cache arrays of the live copy
  void* V;
  void* Kr;
  float* S;
  int32_t* P;
  int g, cap, n_c, seen, mark_unscored;
  uint8_t* Kq;            // 4-bit rows: the packed arrays (K, Kr and V are then the staging copy), else NULL
  uint8_t* Vq;
  int qstride;
  float c_log2;
  int n_part;             // partials per query head
  TokenScore score;       // act NULL: no score to form
  HeadLens n_c_h;         // units per head before the token (ragged), else n_c
};

typedef float dec_f32x4 __attribute__((ext_vector_type(4)));

// the upper halves of a and b as one word, a's low
__device__ __forceinline__ uint32_t upper_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ uint32_t lower_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }

// max and sum over the four lanes lane % 16, + 16, + 32, + 48, in all of them: after a swap one register holds one half's value
// in both halves and the other the other's
__device__ __forceinline__ float max_across_quarters(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return max_across_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_across_quarters(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  const auto t = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// N consecutive words, 4-byte aligned
typedef uint32_t dec_u32x3 __attribute__((ext_vector_type(3), aligned(4)));
template <int N> __device__ __forceinline__ void load_words(const void* p, uint32_t* w) {
  if constexpr (N == 4) { const uint4 v = *(const uint4*)p; w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
  else if constexpr (N == 3) { const dec_u32x3 v = *(const dec_u32x3*)p; w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; }
  else if constexpr (N == 2) { const uint2 v = *(const uint2*)p; w[0] = v.x; w[1] = v.y; }
  else w[0] = *(const uint32_t*)p;
}

// 32 keys of one wavefront in the matrix-core form (see the file header).  Lane (n = lane % 16, kg = lane / 16):
//   ka[b][ks]  16 bytes of key 8 (n / 4) + 4 b + n % 4 from dim 32 ks + 8 kg: rows of the A operand of block b of
//              S^T = K Q^T, ordered so that the lane's accumulators, rows 4 kg + r of the two blocks, are its keys 8 kg + 4 b + r
//   vw[r]      dims n NV .. n NV + NV - 1 of key 8 kg + r
template <int D> struct DecTile {
  static constexpr int NKS = D / 32, NV = D / 16, PARTS = 3;
  bf16x8 ka[2][NKS];
  uint32_t vw[8][NV / 2];
  // (keys from k1 on repeat the last one; kb is the same in the whole wavefront, so only the offsets inside the block are per lane)
  __device__ __forceinline__ void load_k(const bf16_t* Kb, int kb, int k1) {
    const int n = threadIdx.x & 15, kg = (threadIdx.x & 63) >> 4, last = k1 - 1 - kb;
    const bf16_t* base = Kb + (int64_t)kb * D;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int off = min(8 * (n >> 2) + (n & 3) + 4 * b, last) * D + kg * 8;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) ka[b][ks] = *(const bf16x8*)(base + off + ks * 32);
    }
  }
  __device__ __forceinline__ void load_v(const bf16_t* Vb, int kb, int k1) {
    const int n = threadIdx.x & 15, kg = (threadIdx.x & 63) >> 4, last = k1 - 1 - kb;
    const bf16_t* base = Vb + (int64_t)kb * D;
#pragma unroll
    for (int r = 0; r < 8; ++r) load_words<NV / 2>(base + (min(8 * kg + r, last) * D + n * NV), vw[r]);
  }
  // the rows that repeat the last one: zeros, an infinite value times a probability of 0 would reach the output
  __device__ __forceinline__ void clear_v(int kb, int k1) {
    const int over = 8 * (int)((threadIdx.x & 63) >> 4) - (k1 - 1 - kb);
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int w = 0; w < NV / 2; ++w) vw[r][w] = over + r > 0 ? 0u : vw[r][w];
  }
  __device__ __forceinline__ void logits(const bf16x8 (&qb)[NKS], dec_f32x4 (&s)[2]) const {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      s[b] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) s[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[b][ks], qb[ks], s[b], 0, 0, 0);
    }
  }
  // o[i] += P V for dims n NV + i, n = 0..15: the B operand of dim i is the eight keys' values of that dim, taken two keys at
  // a time from the rows' words
  __device__ __forceinline__ void accumulate(bf16x8 p, dec_f32x4 (&o)[NV]) const {
#pragma unroll
    for (int w = 0; w < NV / 2; ++w) {
      const uint4 lo = make_uint4(lower_halves(vw[0][w], vw[1][w]), lower_halves(vw[2][w], vw[3][w]),
                                  lower_halves(vw[4][w], vw[5][w]), lower_halves(vw[6][w], vw[7][w]));
      const uint4 hi = make_uint4(upper_halves(vw[0][w], vw[1][w]), upper_halves(vw[2][w], vw[3][w]),
                                  upper_halves(vw[4][w], vw[5][w]), upper_halves(vw[6][w], vw[7][w]));
      o[2 * w] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p, __builtin_bit_cast(bf16x8, lo), o[2 * w], 0, 0, 0);
      o[2 * w + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p, __builtin_bit_cast(bf16x8, hi), o[2 * w + 1], 0, 0, 0);
    }
  }
};

// Three workgroups a CU at 128 dims: left to itself the compiler takes 200 registers, which leaves room for two, and the 520th
// of 520 workgroups waits for the first.
template <typename T, int D, int G, bool SCORED>
__global__ __launch_bounds__(DEC_THREADS, D == 128 ? 3 : 1) void decode_attn_kernel(const T* __restrict__ Kx, int g0, int keys_per_wg,
                                                                  float* __restrict__ part, DecodeToken tk) {
  // n_splits partials per query head: n_splits - 1 splits over the cached units, then the new token's, which the
  // last of these workgroups forms (it has no units of its own, so it is done long before the others).
  // SCORED: the workgroups behind them form the token's hidden activations.
  const T* __restrict__ q = (const T*)tk.q;
  const T* __restrict__ V = (const T*)tk.V;
  const float2* __restrict__ tab = tk.tab;
  const int g = tk.g, cap = tk.cap, n_splits = tk.n_part;
  const float c_log2 = tk.c_log2;
  constexpr int VEC = Vec16<T>::N;
  constexpr int LPR = D / VEC;                       // lanes that hold data of one row
  constexpr int LPRP = Pow2Ceil<LPR>::value;         // lanes reserved per row
  constexpr int KPW = 64 / LPRP;                     // rows per wavefront per load
  constexpr int NW = DEC_THREADS / 64;
  constexpr int PW = D + 2;                          // floats per partial: vector, max, sum
  typedef Vec16<T> V16;
  typedef decltype(V16().raw) raw_t;
  constexpr bool MM = std::is_same<T, bf16_t>::value && D % 32 == 0;      // on the matrix cores (see the file header)
  constexpr int NSETS = MM ? NW * DecTile<MM ? D : 32>::PARTS : NW * KPW; // accumulator sets the workgroup merges
  __shared__ __attribute__((aligned(16))) float sets[NSETS * G * (MM ? D : PW)];
  __shared__ float wml[MM ? NW * G * 2 : 1];         // max and sum of every wavefront

  const int split = blockIdx.x, m = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  static_assert(!SCORED || std::is_same<T, bf16_t>::value, "only bf16 layers' scores are formed here");
  if constexpr (SCORED) {
    if (split >= n_splits) {
      const TokenScore& sc = tk.score;
      const int r = ((split - n_splits) * (int)gridDim.y + m) * (DEC_THREADS / 64) + wave;
      if (r < sc.d_R)
        token_hidden(q, (const bf16_t*)tk.k, (const bf16_t*)tk.v, sc.hd, sc.kvd, (const bf16_t*)sc.W1t, sc.K, r, sc.act);
      return;
    }
  }
  const int sub = lane % LPRP, grp = lane / LPRP;
  const bool act = sub < LPR;
  // head-wise budgets: a head shorter than the longest leaves its last splits empty (k1 <= k0: no row is
  // read, the partial carries max -inf and sum 0, which the merge weighs with 0)
  const int n_keys = head_len(tk.n_c_h, m, tk.n_c);   // units of this head in the cache = the new token's slot and position
  const int k0 = split * keys_per_wg;
  const int k1 = min(n_keys, k0 + keys_per_wg);
  const T* Kb = Kx + (int64_t)m * cap * D;
  const T* Vb = V + (int64_t)m * cap * D;
  const int off = (act ? sub : 0) * VEC;

  constexpr int BLK = MM ? NW * 32 : NW * DEC_UN * KPW;    // keys per workgroup iteration
  const bool token_wg = split == n_splits - 1;

  // A wavefront's first keys and values are requested before anything else.  (Behind the query's pieces:
  // 14.6 us instead of 14.1 on 8 heads x 16.4K units.)
  DecTile<MM ? D : 32> tile;
  const int kb_w = k0 + wave * 32;                   // (matrix-core form) this wavefront's first block of 32 keys
  if (MM && kb_w < k1) {
    tile.load_k((const bf16_t*)Kb, kb_w, k1);
    tile.load_v((const bf16_t*)Vb, kb_w, k1);
  }
  // `tab` non-null: q is un-rotated and takes position n_keys (the slot the token is appended at).  One thread
  // per 16-byte chunk of the G query rows rotates its dims with the partner dims (+- D/2), rounds to the storage
  // type as the rotated query of a chunk is, and leaves the row in LDS for the whole workgroup: every workgroup
  // of the launch reads the same few lines of q and of the table, and those requests queue on one L2 channel
  // (with every lane rotating for itself the kernel took 26 us instead of 20).
  float qv[MM ? 1 : G][VEC];
  __shared__ float qs[G * D];
  constexpr int CPR = D / VEC;                         // chunks per row
  const int qu = tid / CPR, qoff = (tid % CPR) * VEC;  // the chunk this thread rotates
  const bool q_thread = tab != nullptr && tid < G * CPR, qlow = qoff < D / 2;
  V16 qx, qy;
  float2 qcs[VEC];
  if (q_thread) {
    const T* qr = q + (int64_t)(m * g + min(g0 + qu, g - 1)) * D;
    qx.raw = *(const raw_t*)(qr + qoff);
    qy.raw = *(const raw_t*)(qr + (qlow ? qoff + D / 2 : qoff - D / 2));
    const float2* tr = tab + (int64_t)n_keys * (D / 2) + (qlow ? qoff : qoff - D / 2);
#pragma unroll
    for (int e = 0; e < VEC; ++e) qcs[e] = tr[e];
  }
  // the new token's own row, in its workgroup (last of the head); 4-bit rows are read by the quantizer instead
  const bool token_row = token_wg && tid < D && tk.Kq == nullptr;
  const bool klow = tid < D / 2;
  T k_own, k_pair, v_own;
  float2 k_cs;
  if (token_row) {
    const T* kp = (const T*)tk.k + (int64_t)m * D;
    k_own = kp[tid];
    k_pair = kp[klow ? tid + D / 2 : tid - D / 2];
    v_own = ((const T*)tk.v)[(int64_t)m * D + tid];
    if (tab != nullptr) k_cs = tab[(int64_t)n_keys * (D / 2) + (klow ? tid : tid - D / 2)];
  }
  if (tab != nullptr) {
    if (q_thread) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        V16 r;
        r.set(0, qlow ? qx.get(e) * qcs[e].x - qy.get(e) * qcs[e].y : qx.get(e) * qcs[e].x + qy.get(e) * qcs[e].y);
        qs[qu * D + qoff + e] = r.get(0) * c_log2;     // logits in log2 units
      }
    }
    __syncthreads();
    if (!MM) {
#pragma unroll
      for (int u = 0; u < G; ++u)
#pragma unroll
        for (int e = 0; e < VEC; ++e) qv[MM ? 0 : u][e] = act ? qs[u * D + off + e] : 0.f;
    }
  } else if (MM) {                                     // the matrix-core path takes the query from LDS
    if (tid < G * CPR) {
      V16 x;
      x.raw = *(const raw_t*)(q + (int64_t)(m * g + min(g0 + qu, g - 1)) * D + qoff);
#pragma unroll
      for (int e = 0; e < VEC; ++e) qs[qu * D + qoff + e] = x.get(e) * c_log2;
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int j = m * g + min(g0 + u, g - 1);        // spare heads repeat the last one (not written)
      V16 x;
      x.raw = *(const raw_t*)(q + (int64_t)j * D + off);
#pragma unroll
      for (int e = 0; e < VEC; ++e) qv[MM ? 0 : u][e] = act ? x.get(e) * c_log2 : 0.f;   // logits in log2 units
    }
  }
  // ---- the new token (last workgroup of the head): its partial for the G heads, and the append ------------------
  if (token_wg) {
    __shared__ float ks[D];                              // its key, rotated to position n_keys and rounded as stored
    __shared__ float dots[G][DEC_THREADS / 64];
    __shared__ float vs[D];                              // its value as stored
    if constexpr (std::is_same<T, bf16_t>::value && (D == 64 || D == 96 || D == 128)) {
      // 4-bit rows: attention sees the token as the cache holds it, so it is quantized first (wavefront 0 the key,
      // wavefront 1 the value).  As a launch of its own in front of this kernel that took 6 us a token.
      if (tk.Kq != nullptr && wave < 2) {
        constexpr int NP = Q4Lanes<D>::NP;
        const int p = min(lane, NP - 1);
        Q4Pieces r = quantize_pieces<D>((const bf16_t*)(wave == 0 ? tk.k : tk.v) + (int64_t)m * D, p, 0);
        if (wave == 0 && tab != nullptr) {
          float2 cs[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) cs[e] = tab[(int64_t)n_keys * (D / 2) + 8 * p + e];
          r.rotate(cs);
        }
        if (lane < NP) {
          const q4_u32x4 ra = pack8_bf16(r.a), rb = pack8_bf16(r.b);
          if (g0 == 0) {                                 // one launch per step appends
            const int64_t slot = (int64_t)m * cap + n_keys;
            store_pieces<D>(r, (wave == 0 ? tk.Kq : tk.Vq) + slot * tk.qstride, p);
            bf16_t* st = (bf16_t*)(wave == 0 ? tk.Kr : tk.V) + slot * D;
            *(q4_u32x4*)(st + 8 * p) = ra;
            *(q4_u32x4*)(st + D / 2 + 8 * p) = rb;
          }
          float a[8], b[8];
          unpack8_bf16(ra, a);
          unpack8_bf16(rb, b);
          float* dst = wave == 0 ? ks : vs;
#pragma unroll
          for (int e = 0; e < 8; ++e) { dst[8 * p + e] = a[e]; dst[D / 2 + 8 * p + e] = b[e]; }
        }
      }
    }
    if (g0 == 0 && tid == 0) {
      tk.P[(int64_t)m * cap + n_keys] = tk.seen;
      if (tk.mark_unscored) tk.S[(int64_t)m * cap + n_keys] = __uint_as_float(0x7fc00000u);   // NaN: ranks last
    }
    if (token_row) {
      float ke = Elem<T>::ld(&k_own);
      if (tab != nullptr) {
        const float kpar = Elem<T>::ld(&k_pair);
        T rounded;
        Elem<T>::st(&rounded, klow ? ke * k_cs.x - kpar * k_cs.y : ke * k_cs.x + kpar * k_cs.y);
        ke = Elem<T>::ld(&rounded);
      }
      ks[tid] = ke;
      vs[tid] = Elem<T>::ld(&v_own);
      if (g0 == 0) {
        const int64_t row = ((int64_t)m * cap + n_keys) * D + tid;
        ((T*)tk.K)[row] = k_own;
        ((T*)tk.V)[row] = v_own;
        if (tab != nullptr) Elem<T>::st((T*)tk.Kr + row, ke);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < G; ++u) {
      float pr = 0.f;
      if (tid < D) {
        const int j = m * g + min(g0 + u, g - 1);
        const float qe = tab != nullptr ? qs[u * D + tid] : Elem<T>::ld(q + (int64_t)j * D + tid) * c_log2;
        pr = qe * ks[tid];
      }
#pragma unroll
      for (int x = 32; x >= 1; x >>= 1) pr += __shfl_xor(pr, x, 64);
      if (lane == 0) dots[u][wave] = pr;
    }
    __syncthreads();
    for (int idx = tid; idx < G * PW; idx += DEC_THREADS) {
      const int u = idx / PW, e = idx % PW;
      if (g0 + u >= g) continue;
      float val;
      if (e < D) {
        val = vs[e];
      } else if (e == D) {
        val = 0.f;
        for (int w2 = 0; w2 < (D + 63) / 64; ++w2) val += dots[u][w2];     // the wavefronts that hold dims, in order
      } else {
        val = 1.f;
      }
      const int j = m * g + g0 + u;
      part[((int64_t)j * n_splits + n_splits - 1) * PW + e] = val;
    }
    return;
  }

  if constexpr (MM) {
    typedef DecTile<D> Tile;
    constexpr int NV = Tile::NV, PARTS = Tile::PARTS;
    const int n = lane & 15, kg = lane >> 4;
    // B operand of S^T = K Q^T: column n is head n % G (every column of a head is the same), lane (n, kg) holds
    // q[32 ks + 8 kg .. + 8], scaled, rounded to bf16 (as the chunk kernels round their pre-scaled queries)
    bf16x8 qb[Tile::NKS];
#pragma unroll
    for (int ks = 0; ks < Tile::NKS; ++ks) {
      const float* x = qs + (n % G) * D + ks * 32 + kg * 8;
      const uint4 pk = make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7]));
      qb[ks] = __builtin_bit_cast(bf16x8, pk);
    }
    // this lane's column takes piece n / G of the probability: what the masks leave after each step
    const uint32_t cut1 = n / G >= 1 ? 0xffff0000u : 0u, cut2 = n / G >= 2 ? 0xffff0000u : 0u;
    dec_f32x4 o[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) o[i] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f;                // of head n % G; the sum over this lane's keys only
    for (int kb = kb_w; kb < k1; kb += BLK) {
      dec_f32x4 s[2];
      tile.logits(qb, s);
      if (kb + BLK < k1) tile.load_k((const bf16_t*)Kb, kb + BLK, k1);
      float p[8];
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p[j] = kb + 8 * kg + j < k1 ? s[j >> 2][j & 3] : -INFINITY;
        mx = fmaxf(mx, p[j]);
      }
      if (__any((mx - mrun) > DEC_RESCALE_LOG2)) {     // also true from -inf to a number
        // the four lanes of a column move together: its accumulators are shared
        mx = max_across_quarters(mx);
        const bool up = (mx - mrun) > DEC_RESCALE_LOG2;
        const float alpha = up ? __builtin_amdgcn_exp2f(mrun - mx) : 1.f;
        if (up) mrun = mx;
        if (kb != kb_w) {                              // (nothing to scale before the first block)
          lrun *= alpha;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float ar = __shfl(alpha, (4 * kg + r) % G, 64);    // accumulator row 4 kg + r is of that head
#pragma unroll
            for (int i = 0; i < NV; ++i) o[i][r] *= ar;
          }
        }
      }
      uint32_t x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float y = kb + 8 * kg + j < k1 ? __builtin_amdgcn_exp2f(p[j] - mrun) : 0.f;
        lrun += y;
        y -= __uint_as_float(__float_as_uint(y) & cut1);
        y -= __uint_as_float(__float_as_uint(y) & cut2);
        x[j] = __float_as_uint(y);
      }
      const uint4 pk = make_uint4(upper_halves(x[0], x[1]), upper_halves(x[2], x[3]), upper_halves(x[4], x[5]), upper_halves(x[6], x[7]));
      if (kb + 32 > k1) tile.clear_v(kb, k1);
      tile.accumulate(__builtin_bit_cast(bf16x8, pk), o);
      if (kb + BLK < k1) tile.load_v((const bf16_t*)Vb, kb + BLK, k1);
    }
    lrun = sum_across_quarters(lrun);
    // ---- merge the wavefronts (and the pieces of the probabilities) ----------------------------
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * kg + r, piece = row / G, u = row % G;
      if (piece < PARTS)
#pragma unroll
        for (int i = 0; i < NV; ++i) sets[((wave * PARTS + piece) * G + u) * D + n * NV + i] = o[i][r];
    }
    if (lane < G) {
      wml[(wave * G + lane) * 2] = mrun;
      wml[(wave * G + lane) * 2 + 1] = lrun;
    }
    __syncthreads();
    for (int idx = tid; idx < G * PW; idx += DEC_THREADS) {
      const int u = idx / PW, e = idx % PW;
      if (g0 + u >= g) continue;
      float M = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) M = fmaxf(M, wml[(w * G + u) * 2]);
      float val = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float ms = wml[(w * G + u) * 2];
        const float wt = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ms - M);      // a wavefront without keys carries nothing
        float part_w;
        if (e < D) {
          const float* src = sets + (w * PARTS * G + u) * D + e;
          const float hi = src[0], rest = src[G * D] + src[2 * G * D];
          part_w = isfinite(hi) ? hi + rest : hi;      // an infinite value times a piece that is 0 is not a number
        } else {
          part_w = wml[(w * G + u) * 2 + 1];
        }
        val = fmaf(wt, part_w, val);
      }
      if (e == D) val = M;
      const int j = m * g + g0 + u;
      part[((int64_t)j * n_splits + split) * PW + e] = val;
    }
  } else {
    float o[G][VEC], mrun[G], lrun[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      mrun[u] = -INFINITY;
      lrun[u] = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[u][e] = 0.f;
    }
    for (int kb = k0; kb < k1; kb += BLK) {
      // (spare rows re-read the first row)
      V16 kf[DEC_UN], vf[DEC_UN];
      bool valid[DEC_UN];
#pragma unroll
      for (int i = 0; i < DEC_UN; ++i) {
        const int key = kb + (wave * DEC_UN + i) * KPW + grp;
        valid[i] = key < k1;
        const int64_t row = (int64_t)(valid[i] ? key : k0) * D + off;
        kf[i].raw = *(const raw_t*)(Kb + row);
        vf[i].raw = *(const raw_t*)(Vb + row);
      }
      float s[DEC_UN][G];
#pragma unroll
      for (int i = 0; i < DEC_UN; ++i)
#pragma unroll
        for (int u = 0; u < G; ++u) {
          float a = 0.f;
#pragma unroll
          for (int e = 0; e < VEC; ++e) a = fmaf(kf[i].get(e), qv[MM ? 0 : u][e], a);
#pragma unroll
          for (int x = 1; x < LPRP; x <<= 1) a += __shfl_xor(a, x, 64);
          s[i][u] = valid[i] ? a : -INFINITY;
        }
      // one max decision per head for the UN rows of this lane group
      float muse[G];
      bool up_any = false;
#pragma unroll
      for (int u = 0; u < G; ++u) {
        float mx = s[0][u];
#pragma unroll
        for (int i = 1; i < DEC_UN; ++i) mx = fmaxf(mx, s[i][u]);
        const float m_new = fmaxf(mrun[u], mx);
        const bool up = (m_new - mrun[u]) > DEC_RESCALE_LOG2;   // also true from -inf to a number
        muse[u] = up ? m_new : mrun[u];
        up_any = up_any || up;
      }
      if (__any(up_any)) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const float alpha = (muse[u] == mrun[u]) ? 1.f : __builtin_amdgcn_exp2f(mrun[u] - muse[u]);
          lrun[u] *= alpha;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[u][e] *= alpha;
        }
      }
#pragma unroll
      for (int u = 0; u < G; ++u) mrun[u] = muse[u];
#pragma unroll
      for (int i = 0; i < DEC_UN; ++i)
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const float p = valid[i] ? __builtin_amdgcn_exp2f(s[i][u] - muse[u]) : 0.f;
          lrun[u] += p;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[u][e] = fmaf(p, vf[i].get(e), o[u][e]);
        }
    }

    // ---- merge the row slots of the workgroup --------------------------------------------------
    const int set = wave * KPW + grp;
    if (act) {
#pragma unroll
      for (int u = 0; u < G; ++u) {
        float* dst = sets + (set * G + u) * PW;
#pragma unroll
        for (int e = 0; e < VEC; ++e) dst[off + e] = o[u][e];
        if (sub == 0) {
          dst[D] = mrun[u];
          dst[D + 1] = lrun[u];
        }
      }
    }
    __syncthreads();
    for (int idx = tid; idx < G * PW; idx += DEC_THREADS) {
      const int u = idx / PW, e = idx % PW;
      if (g0 + u >= g) continue;
      float M = -INFINITY;
      for (int s2 = 0; s2 < NSETS; ++s2) M = fmaxf(M, sets[(s2 * G + u) * PW + D]);
      float val;
      if (e == D) {
        val = M;
      } else {
        float acc = 0.f;
        for (int s2 = 0; s2 < NSETS; ++s2) {
          const float ms = sets[(s2 * G + u) * PW + D];
          const float w = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ms - M);   // empty slots carry nothing
          acc = fmaf(w, sets[(s2 * G + u) * PW + e], acc);     // e == D + 1 merges the sums
        }
        val = acc;
      }
      const int j = m * g + g0 + u;
      part[((int64_t)j * n_splits + split) * PW + e] = val;
    }
  }
}

// out[j][:] = sum_s w_s o_s / sum_s w_s l_s with w_s = 2^(m_s - max_s m_s).  One workgroup per head.
// A separate launch on purpose: letting the last workgroup of a head merge behind a device-scope
// fence was measured 3x slower than both kernels together (every workgroup then pays for making its
// partials visible across the eight L2s), while a kernel boundary does that once.
// The kernel is a chain of memory latencies, not of bytes (45 KB per head): every load that does not depend on another is
// requested up front, and the wavefronts meet once.  A wavefront owns 64 dims of splits sg, sg + SG, ..., and forms the
// weights of all splits itself, one or two a lane (their maxima and sums cost it two loads), from where a split's weight comes
// as a scalar.  Against a thread per (dim, eighth of the splits) of 1024 and three meetings in LDS a token (both launches, tokens back to back)
// takes 0.8 us less: 8 heads x 128 dims, 2K units 9.1 -> 8.3 us, 16.4K 17.5 -> 16.7, 32 x 8.2K x 96 20.7 -> 19.9; by the kernel trace, which
// sees the launch from its first wavefront on, this kernel takes 3.9 -> 2.6 to 3.2 us on 1K and 6K units, 3.8 as before on 16.4K.
constexpr int DEC_MERGE_THREADS = 512;
constexpr int DEC_MERGE_PRE = 96;       // splits requested before anything else

// max and sum over the wavefront, in every lane: rotations inside the rows of 16 lanes, then across the rows
template <typename F> __device__ __forceinline__ float over_row(float x, F f) {
#define LOCRET_ROR(N) __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + N, 0xf, 0xf, true))
  x = f(x, LOCRET_ROR(8));
  x = f(x, LOCRET_ROR(4));
  x = f(x, LOCRET_ROR(2));
  return f(x, LOCRET_ROR(1));
#undef LOCRET_ROR
}
__device__ __forceinline__ float wave_max(float x) {
  return max_across_quarters(over_row(x, [](float a, float b) { return fmaxf(a, b); }));
}
__device__ __forceinline__ float wave_sum(float x) {
  return sum_across_quarters(over_row(x, [](float a, float b) { return a + b; }));
}
__device__ __forceinline__ float lane_value(float x, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane)); }

// ND: wavefronts side by side over the dims (head dims up to 64 ND).  SCORED: one more workgroup per KV head multiplies the
// token's hidden activations with W2.
template <typename T, int ND, bool SCORED>
__global__ __launch_bounds__(DEC_MERGE_THREADS) void decode_merge_kernel(const float* __restrict__ part, int n_splits,
                                                                         int d, T* __restrict__ out, int h, TokenScore score,
                                                                         float* __restrict__ S, int cap, int n_c, HeadLens n_c_h) {
  static_assert(ND == 1 || ND == 2, "head dims up to 128");
  constexpr int NW = DEC_MERGE_THREADS / 64, SG = NW / ND, PRE = DEC_MERGE_PRE / SG;
  __shared__ float acc_s[NW][64];
  const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (SCORED && j >= h) {
    const int m = j - h;
    const float s = token_score(score.act, score.d_R, score.W2f, score.h_kv, m, acc_s[0]);
    if (tid == 0) {
      S[(int64_t)m * cap + head_len(n_c_h, m, n_c)] = s;
      if (score.out) score.out[m] = s;
    }
    return;
  }
  const int pw = d + 2;
  const float* p = part + (int64_t)j * n_splits * pw;
  const int sg = wave / ND, e = min((wave % ND) * 64 + lane, d - 1);      // (lanes past the last dim repeat it)
  // (addresses are clamped instead of the loads being predicated: a conditional load is a branch, and the wait
  // counters cannot be tracked across it, so every such load would be waited for before the next is issued)
  float2 ml[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) ml[i] = *(const float2*)(p + min(lane + 64 * i, n_splits - 1) * pw + d);     // pw and d are even: 8-byte aligned
  float pv[PRE];
#pragma unroll
  for (int i = 0; i < PRE; ++i) pv[i] = p[min(sg + i * SG, n_splits - 1) * pw + e];
  const float m0 = lane < n_splits ? ml[0].x : -INFINITY, m1 = lane + 64 < n_splits ? ml[1].x : -INFINITY;
  float M = fmaxf(m0, m1);
  for (int s = lane + 128; s < n_splits; s += 64) M = fmaxf(M, p[s * pw + d]);
  M = wave_max(M);
  // weights w_s = 2^(m_s - M) (a split without keys carries max -inf and weighs 0)
  const float w0 = __builtin_amdgcn_exp2f(m0 - M), w1 = __builtin_amdgcn_exp2f(m1 - M);
  float l = fmaf(w1, lane + 64 < n_splits ? ml[1].y : 0.f, w0 * (lane < n_splits ? ml[0].y : 0.f));
  for (int s = lane + 128; s < n_splits; s += 64) l = fmaf(__builtin_amdgcn_exp2f(p[s * pw + d] - M), p[s * pw + d + 1], l);
  const float inv = 1.f / wave_sum(l);
  // eight chains of sums over the splits for every head dim: SG wavefronts with ND each
  float a[ND];
#pragma unroll
  for (int c = 0; c < ND; ++c) a[c] = 0.f;
#pragma unroll
  for (int i = 0; i < PRE; ++i) {
    const int s = sg + i * SG;                           // below 64 for i < 64 / SG, below 128 for all
    const float w = i < 64 / SG ? lane_value(w0, s) : lane_value(w1, s - 64);      // 0 past the last split
    if (s < n_splits) a[i % ND] = fmaf(w, pv[i], a[i % ND]);
  }
  static_assert(PRE % ND == 0, "the chains go on in turn");
  for (int s0 = sg + PRE * SG; s0 < n_splits; s0 += ND * SG)
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      const int s = s0 + c * SG;
      if (s < n_splits) a[c] = fmaf(s < 128 ? lane_value(w1, s - 64) : __builtin_amdgcn_exp2f(p[s * pw + d] - M), p[s * pw + e], a[c]);
    }
  acc_s[wave][lane] = ND == 1 ? a[0] : a[0] + a[ND - 1];
  __syncthreads();
  if (tid < d) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < SG; ++i) t += acc_s[i * ND + wave][lane];
    Elem<T>::st(out + (int64_t)j * d + tid, t * inv);
  }
}

// Keys per split.  Tuning::dec_keys (a multiple of 64 in 64 .. 65536) fixes it; otherwise it is chosen per launch.
int decode_keys_per_split(const Dims& D, int n_keys) {
  return D.tune.dec_keys > 0 ? D.tune.dec_keys : decode_split_keys(D.bf16 != 0, D.h_kv, n_keys);
}

// partials per query head at most: the splits over a full cache at the smallest split size, and the new token's
int decode_max_splits(const Dims& D) {
  const int kmin = D.tune.dec_keys > 0 ? D.tune.dec_keys : DEC_KEYS_MIN;
  return (D.cap + kmin - 1) / kmin + 1;
}

template <typename T, int DD>
static void decode_launch(const Dims& D, DecodeToken& tk, T* out, float* part, hipStream_t st) {
  const int kpw = decode_keys_per_split(D, tk.n_c);
  const int n_attn = (tk.n_c + kpw - 1) / kpw;   // splits over the units already in the cache (the longest head's)
  const T* Kx = (const T*)(D.rope ? tk.Kr : tk.K);
  const int n_part = n_attn + 1;                          // + the workgroup of the new token
  tk.n_part = n_part;
  const bool scored = tk.score.act != nullptr;
  const int per_x = D.h_kv * (DEC_THREADS / 64);          // hidden units of one further column of workgroups
  for (int g0 = 0; g0 < D.g; g0 += 4) {
    const int left = D.g - g0;
    const dim3 grid(n_part + (scored && g0 == 0 ? (D.d_R + per_x - 1) / per_x : 0), D.h_kv);
#define LOCRET_DEC_ATTN(GG, SC)                                                                                         \
  hipLaunchKernelGGL((decode_attn_kernel<T, DD, GG, SC>), grid, dim3(DEC_THREADS), 0, st, Kx, g0, kpw, part, tk)
    if constexpr (std::is_same<T, bf16_t>::value) {       // float32 layers hand over no score to form
      if (scored && g0 == 0) {
        if (left >= 3) LOCRET_DEC_ATTN(4, true);
        else if (left == 2) LOCRET_DEC_ATTN(2, true);
        else LOCRET_DEC_ATTN(1, true);
        continue;
      }
    }
    if (left >= 3) LOCRET_DEC_ATTN(4, false);
    else if (left == 2) LOCRET_DEC_ATTN(2, false);
    else LOCRET_DEC_ATTN(1, false);
#undef LOCRET_DEC_ATTN
  }
#define LOCRET_DEC_MERGE(SC)                                                                                              \
  hipLaunchKernelGGL((decode_merge_kernel<T, (DD + 63) / 64, SC>), dim3(D.h + (SC ? D.h_kv : 0)), dim3(DEC_MERGE_THREADS), 0, st,          \
                     (const float*)part, n_part, D.d, out, D.h, tk.score, tk.S, D.cap, tk.n_c, tk.n_c_h)
  if constexpr (std::is_same<T, bf16_t>::value) {
    if (scored) {
      LOCRET_DEC_MERGE(true);
      return;
    }
  }
  LOCRET_DEC_MERGE(false);
#undef LOCRET_DEC_MERGE
}

void launch_decode_step(const Dims& D, const void* q, const void* k, const void* v, const CacheBuf& c,
                        const float2* tab, void* out, int n_c, int64_t seen, float scale, float* part, hipStream_t st,
                        bool mark_unscored, const HeadLens* n_c_h, const TokenScore* score) {
  DecodeToken tk;
  tk.Kq = (uint8_t*)c.Kq; tk.Vq = (uint8_t*)c.Vq; tk.qstride = c.qstride;
  tk.q = q; tk.k = k; tk.v = v;
  tk.tab = D.rope ? tab : nullptr;
  tk.K = c.K; tk.V = c.V; tk.Kr = c.Kr; tk.S = c.S; tk.P = c.P;
  tk.g = D.g; tk.cap = D.cap; tk.n_c = n_c; tk.seen = (int)seen; tk.mark_unscored = mark_unscored ? 1 : 0;
  tk.c_log2 = scale * 1.4426950408889634f;
  tk.score = score ? *score : TokenScore{};
  tk.n_c_h = head_lens_or_common(n_c_h);
#define LOCRET_DEC(DD)                                                                  \
  case DD:                                                                              \
    if (D.bf16) decode_launch<bf16_t, DD>(D, tk, (bf16_t*)out, part, st);               \
    else decode_launch<float, DD>(D, tk, (float*)out, part, st);                        \
    break;
  switch (D.d) {
    LOCRET_DEC(16)
    LOCRET_DEC(32)
    LOCRET_DEC(64)
    LOCRET_DEC(96)
    LOCRET_DEC(128)
  }
#undef LOCRET_DEC
}

}  // namespace locret
