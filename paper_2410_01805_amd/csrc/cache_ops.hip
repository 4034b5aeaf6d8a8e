// Bandwidth-bound cache maintenance kernels for gfx950: rotary table, weight preparation,
// chunk append (Algorithm 1 "Concat") and order-preserving compaction (Algorithm 1 gather).
// Every thread moves 16-byte vectors; a row of d elements is shared by (d/2)/VEC threads, each of
// which owns VEC rotary pairs (i, i + d/2), so the rotated shadow of K is produced from registers.
#include "device_util.h"
#include "kernels.h"

namespace locret {

// ------------------------------------------------------------------------------------------------
__global__ void rope_table_kernel(float2* tab, int cap, int half, int d, double theta) {
  int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)cap * half) return;
  int pos = (int)(gid / half), i = (int)(gid % half);
  double inv = pow(theta, -2.0 * (double)i / (double)d);
  double a = (double)pos * inv;
  tab[gid] = make_float2((float)cos(a), (float)sin(a));
}

void launch_rope_table(float2* tab, int cap, int d, float theta, hipStream_t st) {
  int64_t n = (int64_t)cap * (d / 2);
  int blocks = (int)((n + 255) / 256);
  hipLaunchKernelGGL(rope_table_kernel, dim3(blocks), dim3(256), 0, st, tab, cap, d / 2, d, (double)theta);
}

// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void prep_w1_kernel(const T* __restrict__ W1, T* __restrict__ W1t, int h, int h_kv, int g, int d,
                               int d_R, int K, int expand) {
  int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)K * d_R) return;
  int n = (int)(gid % d_R);
  int c = (int)(gid / d_R);
  int hd = h * d;
  float acc;
  if (!expand || c < hd) {
    acc = Elem<T>::ld(W1 + (int64_t)c * d_R + n);
  } else {
    int cc = c - hd;
    int blk = cc / (h_kv * d);          // 0: K block, 1: V block
    int r = cc % (h_kv * d);
    int m = r / d, i = r % d;
    int64_t base = (int64_t)hd * (1 + blk);
    acc = 0.f;
    for (int rep = 0; rep < g; ++rep)
      acc += Elem<T>::ld(W1 + (base + (int64_t)(m * g + rep) * d + i) * d_R + n);
  }
  Elem<T>::st(W1t + (int64_t)n * K + c, acc);
}

template <typename T>
__global__ void prep_w2_kernel(const T* __restrict__ W2, float* __restrict__ W2f, int n) {
  int gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid < n) W2f[gid] = Elem<T>::ld(W2 + gid);
}

void launch_prep_weights(const Dims& D, int expand, const void* W1, const void* W2, void* W1t, float* W2f,
                         hipStream_t st) {
  int64_t n1 = (int64_t)D.K * D.d_R;
  int n2 = D.d_R * D.h_kv;
  dim3 b1((unsigned)((n1 + 255) / 256)), b2((unsigned)((n2 + 255) / 256));
  if (D.bf16) {
    hipLaunchKernelGGL(prep_w1_kernel<bf16_t>, b1, dim3(256), 0, st, (const bf16_t*)W1, (bf16_t*)W1t, D.h,
                       D.h_kv, D.g, D.d, D.d_R, D.K, expand);
    hipLaunchKernelGGL(prep_w2_kernel<bf16_t>, b2, dim3(256), 0, st, (const bf16_t*)W2, W2f, n2);
  } else {
    hipLaunchKernelGGL(prep_w1_kernel<float>, b1, dim3(256), 0, st, (const float*)W1, (float*)W1t, D.h,
                       D.h_kv, D.g, D.d, D.d_R, D.K, expand);
    hipLaunchKernelGGL(prep_w2_kernel<float>, b2, dim3(256), 0, st, (const float*)W2, W2f, n2);
  }
}

// ------------------------------------------------------------------------------------------------
// 16-byte loads and stores that bypass the caches' retention: compaction touches every byte once
typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4)));
template <typename R>
__device__ __forceinline__ R nt_load16(const void* p) {
  static_assert(sizeof(R) == 16, "16-byte lanes");
  nt_u32x4 v = __builtin_nontemporal_load((const nt_u32x4*)p);
  return __builtin_bit_cast(R, v);
}
template <typename R>
__device__ __forceinline__ void nt_store16(void* p, R r) {
  static_assert(sizeof(R) == 16, "16-byte lanes");
  __builtin_nontemporal_store(__builtin_bit_cast(nt_u32x4, r), (nt_u32x4*)p);
}

// Append: a thread owns token t and VEC rotary pairs of its rows, for `hpb` consecutive KV heads (blockIdx.y), so
// the rotary-table row of the token's slot is read once for all of them and the loads of two heads are in flight
// together.  Bound by HBM: 12 us for 4096 tokens x 8 heads x 128 dims = 42 MB.  Scores that the caller has already
// (S_src) travel with the rows.  With one thread per row piece, each with its own table reads, that cost as much as
// the launch of their own it saves: 48000 tokens in 12 eviction-only steps 538 us with the separate launch, 537 us
// with one thread per piece, 500 us in this form.  With q != NULL further blocks of blockIdx.y rotate the queries
// into qr (storage types whose attention kernel does not do it itself).
// An eviction-only step that evicts nothing has the caller's list 0, 1, 2, ... written here as well (keep), every thread a
// share of it: a launch of its own for that took 4.2 us
// (48000 tokens into 8 x 32768 units in 12 steps, 8 of which evict nothing: 499 -> 486 us).
// K un-rotated is next read by a compaction, long after it has left the caches: its stores do not stay in them.
__device__ __forceinline__ void keep_all(int32_t* __restrict__ out, int n, int first, int step) {
  for (int i = first; i < n; i += step) out[i] = i;
}

template <typename T, bool RAGGED>
__global__ __launch_bounds__(256) void append_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                     const T* __restrict__ v, int Tn, int n_c_common, int seen, int h,
                                                     int h_kv, int d, int cap, T* __restrict__ Kc,
                                                     T* __restrict__ Vc, T* __restrict__ Krc,
                                                     int32_t* __restrict__ Pc, T* __restrict__ qr,
                                                     const float2* __restrict__ tab, int rope, int hpb, int kv_blocks,
                                                     float* __restrict__ S, const float* __restrict__ S_src, HeadLens n_c_h,
                                                     int32_t* __restrict__ keep, int keep_stride) {
  constexpr int VEC = Vec16<T>::N;
  typedef Vec16<T> V16;
  typedef decltype(V16().raw) raw_t;
  const int half = d / 2;
  const int tpr = half / VEC;
  const int rows = 256 / tpr;                    // tokens per workgroup
  const int lr = (int)threadIdx.x / tpr, part = (int)threadIdx.x % tpr;
  const int t = (int)blockIdx.x * rows + lr;
  if (lr >= rows || t >= Tn) return;
  const int off = part * VEC;
  float2 cs[VEC];
  auto table_row = [&](int n_c) {
    const float2* tr = tab + (int64_t)(n_c + t) * half + off;
#pragma unroll
    for (int i = 0; i < VEC; ++i) cs[i] = tr[i];
  };
  auto rotate = [&](const V16& lo, const V16& hi, V16& olo, V16& ohi) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      const float a = lo.get(i), b = hi.get(i);
      olo.set(i, a * cs[i].x - b * cs[i].y);
      ohi.set(i, b * cs[i].x + a * cs[i].y);
    }
  };
  if (rope && !RAGGED) table_row(n_c_common);
  if ((int)blockIdx.y >= kv_blocks) {
    const int j0 = ((int)blockIdx.y - kv_blocks) * hpb;
    for (int j = j0; j < min(h, j0 + hpb); ++j) {
      if (RAGGED) table_row(n_c_h.v[j / (h / h_kv)]);      // a query sits behind its own KV head's cache
      const int64_t row = ((int64_t)t * h + j) * d;
      V16 lo, hi, olo, ohi;
      lo.raw = *(const raw_t*)(q + row + off);
      hi.raw = *(const raw_t*)(q + row + half + off);
      rotate(lo, hi, olo, ohi);
      *(raw_t*)(qr + row + off) = olo.raw;
      *(raw_t*)(qr + row + half + off) = ohi.raw;
    }
    return;
  }
  const int m_lo = (int)blockIdx.y * hpb, m_hi = min(h_kv, m_lo + hpb);
  for (int m0 = m_lo; m0 < m_hi; m0 += 2) {
    V16 klo[2], khi[2], vlo[2], vhi[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t row = ((int64_t)t * h_kv + min(m0 + u, m_hi - 1)) * d;    // a spare head repeats the last one (not stored)
      klo[u].raw = *(const raw_t*)(k + row + off);
      khi[u].raw = *(const raw_t*)(k + row + half + off);
      vlo[u].raw = *(const raw_t*)(v + row + off);
      vhi[u].raw = *(const raw_t*)(v + row + half + off);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = m0 + u;
      if (m >= m_hi) break;
      const int n_c = RAGGED ? n_c_h.v[m] : n_c_common;
      const int64_t slot = (int64_t)m * cap + n_c + t, drow = slot * d;
      *(raw_t*)(Vc + drow + off) = vlo[u].raw;
      *(raw_t*)(Vc + drow + half + off) = vhi[u].raw;
      if (rope) {
        if (RAGGED) table_row(n_c);
        V16 olo, ohi;
        rotate(klo[u], khi[u], olo, ohi);
        *(raw_t*)(Krc + drow + off) = olo.raw;
        *(raw_t*)(Krc + drow + half + off) = ohi.raw;
        nt_store16(Kc + drow + off, klo[u].raw);
        nt_store16(Kc + drow + half + off, khi[u].raw);
      } else {
        *(raw_t*)(Kc + drow + off) = klo[u].raw;
        *(raw_t*)(Kc + drow + half + off) = khi[u].raw;
      }
      if (part == 0) {
        Pc[slot] = seen + t;
        if (S_src) S[slot] = S_src[(int64_t)m * Tn + t];
      }
      if (keep) keep_all(keep + (int64_t)m * keep_stride, n_c + Tn, t * tpr + part, Tn * tpr);
    }
  }
}

// Rows of 96 bf16, whose halves are not whole 128-byte lines: a thread owns one 16-byte piece of the row
// instead of a rotary pair of pieces, and fetches the partner piece of K as well (a line its neighbours have just
// fetched).  A wavefront then stores 1 KB in a row; in pairs of pieces it stores runs of half a row, which end inside
// lines.  (32 heads x 96: append of 4096 tokens 36 -> 30 us, compaction of 8192 units 70 -> 58 us.  Rows of 64 dims,
// whose halves are half a line, gain nothing from it: append of 2048 tokens on 8 heads 5.3 against 5.8 us.)
__device__ __forceinline__ uint4 rotate_piece(uint4 own, uint4 partner, const float2 (&cs)[8], bool low) {
  Vec16<bf16_t> x, y, r;
  x.raw = own;
  y.raw = partner;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    r.set(i, low ? x.get(i) * cs[i].x - y.get(i) * cs[i].y : x.get(i) * cs[i].x + y.get(i) * cs[i].y);
  return r.raw;
}

template <bool RAGGED>
__global__ __launch_bounds__(256) void append_rows_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int Tn,
                                                          int n_c_common, int seen, int h_kv, int d, int cap,
                                                          bf16_t* __restrict__ Kc, bf16_t* __restrict__ Vc,
                                                          bf16_t* __restrict__ Krc, int32_t* __restrict__ Pc,
                                                          const float2* __restrict__ tab, int rope, int hpb,
                                                          float* __restrict__ S, const float* __restrict__ S_src, HeadLens n_c_h,
                                                          int32_t* __restrict__ keep, int keep_stride) {
  constexpr int HB = 2;
  const int half = d / 2, ppr = d / 8, rows = 256 / ppr;       // pieces of a row, tokens per workgroup
  const int lr = (int)threadIdx.x / ppr, piece = (int)threadIdx.x % ppr;
  const int t = (int)blockIdx.x * rows + lr;
  if (lr >= rows || t >= Tn) return;
  const int off = piece * 8;
  const bool low = off < half;
  const int poff = low ? off + half : off - half, coff = low ? off : off - half;
  float2 cs[8];
  auto table_row = [&](int n_c) {
    const float2* tr = tab + (int64_t)(n_c + t) * half + coff;
#pragma unroll
    for (int i = 0; i < 8; ++i) cs[i] = tr[i];
  };
  if (rope && !RAGGED) table_row(n_c_common);
  const int m_lo = (int)blockIdx.y * hpb, m_hi = min(h_kv, m_lo + hpb);
  for (int m0 = m_lo; m0 < m_hi; m0 += HB) {
    uint4 kx[HB], ky[HB], vx[HB];
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int64_t row = ((int64_t)t * h_kv + min(m0 + u, m_hi - 1)) * d;    // a spare head repeats the last one (not stored)
      kx[u] = *(const uint4*)(k + row + off);
      ky[u] = *(const uint4*)(k + row + poff);
      vx[u] = *(const uint4*)(v + row + off);
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = m0 + u;
      if (m >= m_hi) break;
      const int n_c = RAGGED ? n_c_h.v[m] : n_c_common;
      const int64_t slot = (int64_t)m * cap + n_c + t, drow = slot * d;
      *(uint4*)(Vc + drow + off) = vx[u];
      if (rope) {
        if (RAGGED) table_row(n_c);
        *(uint4*)(Krc + drow + off) = rotate_piece(kx[u], ky[u], cs, low);
        nt_store16(Kc + drow + off, kx[u]);
      } else {
        *(uint4*)(Kc + drow + off) = kx[u];
      }
      if (piece == 0) {
        Pc[slot] = seen + t;
        if (S_src) S[slot] = S_src[(int64_t)m * Tn + t];
      }
      if (keep) keep_all(keep + (int64_t)m * keep_stride, n_c + Tn, t * ppr + piece, Tn * ppr);
    }
  }
}

// storage and head dim of the kernels above and below
static bool row_pieces(const Dims& D) { return D.bf16 && D.d == 96; }

void launch_append(const Dims& D, const void* q, const void* k, const void* v, int T, int n_c, int64_t seen,
                   const CacheBuf& c, void* qr, const float2* tab, hipStream_t st, const float* scores,
                   const HeadLens* n_c_h, int32_t* keep, int keep_stride) {
  const HeadLens hl = head_lens_or_common(n_c_h);
  if (row_pieces(D) && q == nullptr) {
    const int rows = 256 / (D.d / 8), gx = (T + rows - 1) / rows;
    int hpb = D.h_kv;
    while (hpb > 2 && (int64_t)gx * ((D.h_kv + hpb - 1) / hpb) < 768) hpb = (hpb + 1) / 2;
    const dim3 grid((unsigned)gx, (unsigned)((D.h_kv + hpb - 1) / hpb));
#define LOCRET_APPEND_ROWS(RG)                                                                                           \
  launch_kernel((append_rows_kernel<RG>), grid, dim3(256), 0, st, (const bf16_t*)k, (const bf16_t*)v, T, n_c, (int)seen,   \
                D.h_kv, D.d, D.cap, (bf16_t*)c.K, (bf16_t*)c.V, (bf16_t*)c.Kr, c.P, tab, D.rope, hpb, c.S, scores, hl,      \
                keep, keep_stride)
    if (hl.ragged) LOCRET_APPEND_ROWS(true); else LOCRET_APPEND_ROWS(false);
#undef LOCRET_APPEND_ROWS
    return;
  }
  const int vec = D.bf16 ? 8 : 4;
  const int tpr = (D.d / 2) / vec;
  const int rows = 256 / tpr;
  const int q_rows = (D.rope && q != nullptr) ? D.h : 0;
  const int gx = (T + rows - 1) / rows;
  // as few heads per thread as give the chip about three workgroups per CU
  int hpb = D.h_kv;
  while (hpb > 1 && (int64_t)gx * ((D.h_kv + hpb - 1) / hpb) < 768) hpb = (hpb + 1) / 2;
  const int kv_blocks = (D.h_kv + hpb - 1) / hpb;
  dim3 grid((unsigned)gx, (unsigned)(kv_blocks + (q_rows + hpb - 1) / hpb));
#define LOCRET_APPEND(TT, RG)                                                                                          \
  launch_kernel((append_kernel<TT, RG>), grid, dim3(256), 0, st, (const TT*)q, (const TT*)k, (const TT*)v, T, n_c,     \
                (int)seen, D.h, D.h_kv, D.d, D.cap, (TT*)c.K, (TT*)c.V, (TT*)c.Kr, c.P, (TT*)qr, tab, D.rope, hpb,     \
                kv_blocks, c.S, scores, hl, keep, keep_stride)
  if (D.bf16) { if (hl.ragged) LOCRET_APPEND(bf16_t, true); else LOCRET_APPEND(bf16_t, false); }
  else { if (hl.ragged) LOCRET_APPEND(float, true); else LOCRET_APPEND(float, false); }
#undef LOCRET_APPEND
}

// ------------------------------------------------------------------------------------------------
// Compaction: dst[m][r] = src[m][kept[m][r]].  A thread owns slot r (and VEC rotary pairs of it)
// for ALL KV heads: the rotary table row of slot r is read once and reused for every head, and
// the loads of HB heads are issued together before anything is stored (memory-level parallelism).
// RAGGED: head m has keep_h.v[m] rows (head-wise budgets); rows beyond that are neither read nor written.
template <typename T, int HB, bool RAGGED>
__global__ __launch_bounds__(256) void compact_kernel(const T* __restrict__ Ks, const T* __restrict__ Vs,
                                                      const float* __restrict__ Ss, const int32_t* __restrict__ Ps,
                                                      T* __restrict__ Kd, T* __restrict__ Vd, T* __restrict__ Krd,
                                                      float* __restrict__ Sd, int32_t* __restrict__ Pd,
                                                      const int32_t* __restrict__ kept, int kept_stride,
                                                      int n_keep, int h_kv, int d, int cap,
                                                      const float2* __restrict__ tab, int rope, int hpb,
                                                      HeadLens keep_h) {
  constexpr int VEC = Vec16<T>::N;
  typedef Vec16<T> V16;
  typedef decltype(V16().raw) raw_t;
  const int half = d / 2;
  const int tpr = half / VEC;
  int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r = (int)(gid / tpr);
  const int part = (int)(gid % tpr);
  if (r >= n_keep) return;
  const int off = part * VEC;
  float2 cs[VEC];
  if (rope) {
    const float2* tr = tab + (int64_t)r * half + off;
#pragma unroll
    for (int i = 0; i < VEC; ++i) cs[i] = tr[i];
  }
  const int m_lo = blockIdx.y * hpb, m_hi = min(h_kv, m_lo + hpb);   // this block's KV heads
  for (int m0 = m_lo; m0 < m_hi; m0 += HB) {
    int src[HB];
    V16 klo[HB], khi[HB], vlo[HB], vhi[HB];
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = min(m0 + u, m_hi - 1);          // spare iterations repeat the last head (stores are skipped)
      if (RAGGED) src[u] = r < keep_h.v[m] ? kept[(int64_t)m * kept_stride + r] : 0;   // row 0: a valid address
      else src[u] = kept[(int64_t)m * kept_stride + r];
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = min(m0 + u, m_hi - 1);
      const int64_t srow = ((int64_t)m * cap + src[u]) * d;
      klo[u].raw = nt_load16<raw_t>(Ks + srow + off);
      khi[u].raw = nt_load16<raw_t>(Ks + srow + half + off);
      vlo[u].raw = nt_load16<raw_t>(Vs + srow + off);
      vhi[u].raw = nt_load16<raw_t>(Vs + srow + half + off);
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = m0 + u;
      if (m >= m_hi) break;
      if (RAGGED && r >= keep_h.v[m]) continue;
      const int64_t drow = ((int64_t)m * cap + r) * d;
      nt_store16(Kd + drow + off, klo[u].raw);
      nt_store16(Kd + drow + half + off, khi[u].raw);
      nt_store16(Vd + drow + off, vlo[u].raw);
      nt_store16(Vd + drow + half + off, vhi[u].raw);
      if (rope) {
        V16 olo, ohi;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          float a = klo[u].get(i), b = khi[u].get(i);
          olo.set(i, a * cs[i].x - b * cs[i].y);
          ohi.set(i, b * cs[i].x + a * cs[i].y);
        }
        nt_store16(Krd + drow + off, olo.raw);
        nt_store16(Krd + drow + half + off, ohi.raw);
      }
      if (part == 0) {
        Sd[(int64_t)m * cap + r] = Ss[(int64_t)m * cap + src[u]];
        Pd[(int64_t)m * cap + r] = Ps[(int64_t)m * cap + src[u]];
      }
    }
  }
}

template <int HB, bool RAGGED>
__global__ __launch_bounds__(256) void compact_rows_kernel(const bf16_t* __restrict__ Ks, const bf16_t* __restrict__ Vs,
                                                           const float* __restrict__ Ss, const int32_t* __restrict__ Ps,
                                                           bf16_t* __restrict__ Kd, bf16_t* __restrict__ Vd,
                                                           bf16_t* __restrict__ Krd, float* __restrict__ Sd,
                                                           int32_t* __restrict__ Pd, const int32_t* __restrict__ kept,
                                                           int kept_stride, int n_keep, int h_kv, int d, int cap,
                                                           const float2* __restrict__ tab, int rope, int hpb,
                                                           HeadLens keep_h) {
  const int half = d / 2, ppr = d / 8, rows = 256 / ppr;
  const int lr = (int)threadIdx.x / ppr, piece = (int)threadIdx.x % ppr;
  const int r = (int)blockIdx.x * rows + lr;
  if (lr >= rows || r >= n_keep) return;
  const int off = piece * 8;
  const bool low = off < half;
  const int poff = low ? off + half : off - half;
  float2 cs[8];
  if (rope) {
    const float2* tr = tab + (int64_t)r * half + (low ? off : off - half);
#pragma unroll
    for (int i = 0; i < 8; ++i) cs[i] = tr[i];
  }
  const int m_lo = blockIdx.y * hpb, m_hi = min(h_kv, m_lo + hpb);
  for (int m0 = m_lo; m0 < m_hi; m0 += HB) {
    int src[HB];
    uint4 kx[HB], ky[HB], vx[HB];
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = min(m0 + u, m_hi - 1);          // spare iterations repeat the last head (stores are skipped)
      if (RAGGED) src[u] = r < keep_h.v[m] ? kept[(int64_t)m * kept_stride + r] : 0;   // row 0: a valid address
      else src[u] = kept[(int64_t)m * kept_stride + r];
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int64_t srow = ((int64_t)min(m0 + u, m_hi - 1) * cap + src[u]) * d;
      kx[u] = *(const uint4*)(Ks + srow + off);
      if (rope) ky[u] = *(const uint4*)(Ks + srow + poff);
      vx[u] = nt_load16<uint4>(Vs + srow + off);
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int m = m0 + u;
      if (m >= m_hi) break;
      if (RAGGED && r >= keep_h.v[m]) continue;
      const int64_t drow = ((int64_t)m * cap + r) * d;
      nt_store16(Kd + drow + off, kx[u]);
      nt_store16(Vd + drow + off, vx[u]);
      if (rope) nt_store16(Krd + drow + off, rotate_piece(kx[u], ky[u], cs, low));
      if (piece == 0) {
        Sd[(int64_t)m * cap + r] = Ss[(int64_t)m * cap + src[u]];
        Pd[(int64_t)m * cap + r] = Ps[(int64_t)m * cap + src[u]];
      }
    }
  }
}

void launch_compact(const Dims& D, const CacheBuf& s, const CacheBuf& t, const int32_t* kept, int kept_stride,
                    int n_keep, const float2* tab, hipStream_t st, const HeadLens* keep_h) {
  const HeadLens hl = head_lens_or_common(keep_h);
  if (n_keep == 0) return;
  if (row_pieces(D)) {
    const int rows = 256 / (D.d / 8), gx = (n_keep + rows - 1) / rows;
    int hpb = D.h_kv;
    while (hpb > 2 && (int64_t)gx * ((D.h_kv + hpb - 1) / hpb) < 768) hpb = (hpb + 1) / 2;
    const dim3 grid((unsigned)gx, (unsigned)((D.h_kv + hpb - 1) / hpb));
#define LOCRET_COMPACT_ROWS(RG)                                                                                          \
  launch_kernel((compact_rows_kernel<2, RG>), grid, dim3(256), 0, st, (const bf16_t*)s.K, (const bf16_t*)s.V, s.S, s.P,   \
                (bf16_t*)t.K, (bf16_t*)t.V, (bf16_t*)t.Kr, t.S, t.P, kept, kept_stride, n_keep, D.h_kv, D.d, D.cap, tab,   \
                D.rope, hpb, hl)
    if (hl.ragged) LOCRET_COMPACT_ROWS(true); else LOCRET_COMPACT_ROWS(false);
#undef LOCRET_COMPACT_ROWS
    return;
  }
  const int vec = D.bf16 ? 8 : 4;
  const int tpr = (D.d / 2) / vec;
  int64_t threads = (int64_t)n_keep * tpr;
  // A thread serves `hpb` KV heads (the rotary-table row is read once for all of them); with many heads
  // and a short cache that leaves too few workgroups, so the heads are then split over blockIdx.y.
  // (config 4, 32 heads x 8192 units: 192 workgroups took 85 us, 768 take 57 us)
  const unsigned gx = (unsigned)((threads + 255) / 256);
  int hpb = D.h_kv;
  while (hpb > 2 && (int64_t)gx * ((D.h_kv + hpb - 1) / hpb) < 768) hpb = (hpb + 1) / 2;
  dim3 grid(gx, (unsigned)((D.h_kv + hpb - 1) / hpb));
  // two heads per batch: enough loads in flight per thread while registers still allow many wavefronts
#define LOCRET_COMPACT(TT, RG)                                                                                   \
  launch_kernel((compact_kernel<TT, 2, RG>), grid, dim3(256), 0, st, (const TT*)s.K, (const TT*)s.V, s.S, s.P, \
                     (TT*)t.K, (TT*)t.V, (TT*)t.Kr, t.S, t.P, kept, kept_stride, n_keep, D.h_kv, D.d, D.cap, tab,   \
                     D.rope, hpb, hl)
  if (D.bf16) { if (hl.ragged) LOCRET_COMPACT(bf16_t, true); else LOCRET_COMPACT(bf16_t, false); }
  else { if (hl.ragged) LOCRET_COMPACT(float, true); else LOCRET_COMPACT(float, false); }
#undef LOCRET_COMPACT
}

}  // namespace locret
