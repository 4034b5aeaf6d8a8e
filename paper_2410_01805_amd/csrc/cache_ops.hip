// Bandwidth-bound cache maintenance kernels for gfx950: rotary table, weight preparation,
// chunk append (Algorithm 1 "Concat") and order-preserving compaction (Algorithm 1 gather).
// Every thread moves 16-byte vectors; a row of d elements is shared by (d/2)/VEC threads, each of
// which owns VEC rotary pairs (i, i + d/2), so the rotated shadow of K is produced from registers.
#include "append_body.h"
#include "device_util.h"
#include "kernels.h"
#include "select_body.h"

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
template <typename T, bool RAGGED, bool ROWS>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs<T> a) {
  append_any<T, RAGGED, ROWS>(a, blockIdx.x, blockIdx.y, threadIdx.x);
}

// Append and selection of an eviction-only step in one launch: the first n_sel workgroups select, one KV head each, on the scores
// that the caller has (they also store the chunk's), the others append, four of the append's workgroups each.  Neither
// needs the other, and alone the selection keeps h_kv of the 256 CUs busy.  The launch takes what the selection takes beside
// the append's traffic, 28 us for 8 x 34.8K candidates against 12 + 22 us of two launches: 48000 tokens into 8 x 32768 units 486 -> 463
// us, 9000 into 8 x 4096 129 -> 116, 33900 into 8 x 32768 in chunks of 300 1085 -> 1024, 32 x 8192 x 96 dims 373 -> 346.
// Two replicas of the first histogram, as in the selection's own launch; 4 or 8 are no faster (463, 469 us).
template <typename T, bool RAGGED, bool ROWS, int MAXR, bool TAIL>
__global__ __launch_bounds__(1024) void append_select_kernel(AppendArgs<T> a, SelectArgs sel, int n_sel) {
  __shared__ __attribute__((aligned(16))) uint32_t smem[select_body_smem_words(1024, 2)];
  if ((int)blockIdx.x < n_sel) {
    select_reg_body<MAXR, 1024, 2, TAIL, true>(sel, blockIdx.x, smem);
    return;
  }
  const int wg = ((int)blockIdx.x - n_sel) * 4 + (int)(threadIdx.x >> 8);
  if (wg < a.gx * a.gy) append_any<T, RAGGED, ROWS>(a, wg % a.gx, wg / a.gx, threadIdx.x & 255);
}

void launch_append(const Dims& D, const void* q, const void* k, const void* v, int T, int n_c, int64_t seen,
                   const CacheBuf& c, void* qr, const float2* tab, hipStream_t st, const float* scores,
                   const HeadLens* n_c_h, int32_t* keep, int keep_stride) {
#define LOCRET_APPEND(TT, RG, ROWS)                                                                            \
  do {                                                                                                         \
    const AppendArgs<TT> a = append_args<TT>(D, q, k, v, T, n_c, seen, c, qr, tab, scores, n_c_h, keep, keep_stride); \
    launch_kernel((append_kernel<TT, RG, ROWS>), dim3(a.gx, a.gy), dim3(256), 0, st, a);                       \
  } while (0)
  const bool ragged = n_c_h && n_c_h->ragged;
  if (row_pieces(D) && q == nullptr) { if (ragged) LOCRET_APPEND(bf16_t, true, true); else LOCRET_APPEND(bf16_t, false, true); }
  else if (D.bf16) { if (ragged) LOCRET_APPEND(bf16_t, true, false); else LOCRET_APPEND(bf16_t, false, false); }
  else { if (ragged) LOCRET_APPEND(float, true, false); else LOCRET_APPEND(float, false, false); }
#undef LOCRET_APPEND
}

template <typename T, bool RAGGED, bool ROWS>
static void append_select_launch(const AppendArgs<T>& a, const SelectArgs& sel, hipStream_t st) {
  const dim3 grid((unsigned)(a.h_kv + (a.gx * a.gy + 3) / 4));
  const int rounds = select_rounds(sel, 16);
#define LOCRET_AS(R, TAIL)                                                                                              \
  do {                                                                                                                  \
    launch_kernel((append_select_kernel<T, RAGGED, ROWS, R, TAIL>), grid, dim3(1024), 0, st, a, sel, a.h_kv);             \
    return;                                                                                                             \
  } while (0)
  if (rounds <= 12) LOCRET_AS(12, false);
  if (rounds <= 24) LOCRET_AS(24, false);
  if (rounds <= 36) LOCRET_AS(36, false);
  LOCRET_AS(36, true);
#undef LOCRET_AS
}

void launch_append_select(const Dims& D, const void* k, const void* v, int T, int n_c, int64_t seen, const CacheBuf& c, const float2* tab,
                          hipStream_t st, const HeadLens* n_c_h, const SelectArgs& sel) {
#define LOCRET_AS(TT, RG, ROWS) \
  append_select_launch<TT, RG, ROWS>(append_args<TT>(D, nullptr, k, v, T, n_c, seen, c, nullptr, tab, nullptr, n_c_h, nullptr, 0), sel, st)
  const bool ragged = n_c_h && n_c_h->ragged;
  if (row_pieces(D)) { if (ragged) LOCRET_AS(bf16_t, true, true); else LOCRET_AS(bf16_t, false, true); }
  else if (D.bf16) { if (ragged) LOCRET_AS(bf16_t, true, false); else LOCRET_AS(bf16_t, false, false); }
  else { if (ragged) LOCRET_AS(float, true, false); else LOCRET_AS(float, false, false); }
#undef LOCRET_AS
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
          olo.set(i, fmaf(a, cs[i].x, -(b * cs[i].y)));
          ohi.set(i, fmaf(b, cs[i].x, a * cs[i].y));
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
