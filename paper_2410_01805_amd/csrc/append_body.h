// The append of a chunk's rows (Algorithm 1 "Concat"), as workgroups of its own launch (cache_ops.hip), beside the
// selection of an eviction-only step (there too) or beside the retaining head of a float32 layer (f32_kernels.hip).
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace locret {

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

// One append: its operands, and the numbers of 256-thread workgroups along the tokens (gx) and the heads (gy).
template <typename T> struct AppendArgs {
  const T *q, *k, *v;
  int Tn, n_c_common, seen, h, h_kv, d, cap;
  T *Kc, *Vc, *Krc;
  int32_t* Pc;
  T* qr;
  const float2* tab;
  int rope, hpb, kv_blocks;
  float* S;
  const float* S_src;
  HeadLens n_c_h;
  int32_t* keep;
  int keep_stride;
  int gx, gy;
};

// workgroup (bx, by) of the append, thread tid of its 256
template <typename T, bool RAGGED>
__device__ __forceinline__ void append_body(int bx, int by, int tid, const T* __restrict__ q, const T* __restrict__ k,
                                            const T* __restrict__ v, int Tn, int n_c_common, int seen, int h,
                                            int h_kv, int d, int cap, T* __restrict__ Kc,
                                            T* __restrict__ Vc, T* __restrict__ Krc,
                                            int32_t* __restrict__ Pc, T* __restrict__ qr,
                                            const float2* __restrict__ tab, int rope, int hpb, int kv_blocks,
                                            float* __restrict__ S, const float* __restrict__ S_src, const HeadLens& n_c_h,
                                            int32_t* __restrict__ keep, int keep_stride) {
  constexpr int VEC = Vec16<T>::N;
  typedef Vec16<T> V16;
  typedef decltype(V16().raw) raw_t;
  const int half = d / 2;
  const int tpr = half / VEC;
  const int rows = 256 / tpr;                    // tokens per workgroup
  const int lr = tid / tpr, part = tid % tpr;
  const int t = bx * rows + lr;
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
      olo.set(i, fmaf(a, cs[i].x, -(b * cs[i].y)));
      ohi.set(i, fmaf(b, cs[i].x, a * cs[i].y));
    }
  };
  if (rope && !RAGGED) table_row(n_c_common);
  if (by >= kv_blocks) {
    const int j0 = (by - kv_blocks) * hpb;
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
  const int m_lo = by * hpb, m_hi = min(h_kv, m_lo + hpb);
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
    r.set(i, fmaf(x.get(i), cs[i].x, low ? -(y.get(i) * cs[i].y) : y.get(i) * cs[i].y));
  return r.raw;
}

template <bool RAGGED>
__device__ __forceinline__ void append_rows_body(int bx, int by, int tid, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int Tn,
                                                 int n_c_common, int seen, int h_kv, int d, int cap,
                                                 bf16_t* __restrict__ Kc, bf16_t* __restrict__ Vc,
                                                 bf16_t* __restrict__ Krc, int32_t* __restrict__ Pc,
                                                 const float2* __restrict__ tab, int rope, int hpb,
                                                 float* __restrict__ S, const float* __restrict__ S_src, const HeadLens& n_c_h,
                                                 int32_t* __restrict__ keep, int keep_stride) {
  constexpr int HB = 2;
  const int half = d / 2, ppr = d / 8, rows = 256 / ppr;       // pieces of a row, tokens per workgroup
  const int lr = tid / ppr, piece = tid % ppr;
  const int t = bx * rows + lr;
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
  const int m_lo = by * hpb, m_hi = min(h_kv, m_lo + hpb);
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

// ROWS: the form of 96-dim rows
template <typename T, bool RAGGED, bool ROWS>
__device__ __forceinline__ void append_any(const AppendArgs<T>& a, int bx, int by, int tid) {
  if constexpr (ROWS)
    append_rows_body<RAGGED>(bx, by, tid, a.k, a.v, a.Tn, a.n_c_common, a.seen, a.h_kv, a.d, a.cap, a.Kc, a.Vc, a.Krc, a.Pc, a.tab, a.rope,
                             a.hpb, a.S, a.S_src, a.n_c_h, a.keep, a.keep_stride);
  else
    append_body<T, RAGGED>(bx, by, tid, a.q, a.k, a.v, a.Tn, a.n_c_common, a.seen, a.h, a.h_kv, a.d, a.cap, a.Kc, a.Vc, a.Krc, a.Pc, a.qr,
                           a.tab, a.rope, a.hpb, a.kv_blocks, a.S, a.S_src, a.n_c_h, a.keep, a.keep_stride);
}
// storage and head dim of the form for 96-dim rows
inline bool row_pieces(const Dims& D) { return D.bf16 && D.d == 96; }

template <typename T>
inline AppendArgs<T> append_args(const Dims& D, const void* q, const void* k, const void* v, int T_, int n_c, int64_t seen, const CacheBuf& c,
                                 void* qr, const float2* tab, const float* scores, const HeadLens* n_c_h, int32_t* keep, int keep_stride) {
  const bool pieces = row_pieces(D) && q == nullptr;
  const int tpr = pieces ? D.d / 8 : (D.d / 2) / Vec16<T>::N;         // threads of a row
  const int rows = 256 / tpr, least = pieces ? 2 : 1;
  const int q_rows = (D.rope && q != nullptr) ? D.h : 0;
  const int gx = (T_ + rows - 1) / rows;
  // as few heads per thread as give the chip about three workgroups per CU
  int hpb = D.h_kv;
  while (hpb > least && (int64_t)gx * ((D.h_kv + hpb - 1) / hpb) < 768) hpb = (hpb + 1) / 2;
  const int kv_blocks = (D.h_kv + hpb - 1) / hpb;
  return {(const T*)q, (const T*)k, (const T*)v, T_, n_c, (int)seen, D.h, D.h_kv, D.d, D.cap, (T*)c.K, (T*)c.V, (T*)c.Kr, c.P, (T*)qr, tab,
          D.rope, hpb, kv_blocks, c.S, scores, head_lens_or_common(n_c_h), keep, keep_stride, gx, kv_blocks + (q_rows + hpb - 1) / hpb};
}

}  // namespace locret
