// Chunk attention (Eq. 1) on the bf16 matrix cores of gfx950, head_dim 128, 96 and 64: K and V tiles go
// global -> LDS directly (buffer_load ... lds), and the two wavefronts of every SIMD are held in anti-phase.
//
// Products are formed transposed with v_mfma_f32_32x32x16_bf16: S^T = K Q^T (A = 32 key rows from LDS, B = the
// wavefront's 32 queries, held in registers for the whole kernel, pre-scaled by scale * log2 e and rotated),
// O^T += V^T P^T (A = V^T from LDS through the transposing read ds_read_b64_tr_b16, B = P^T straight from the S
// accumulator registers: a lane holds 16 keys of ONE query there, so row sums are per-lane scalars and P needs
// no shuffle).  A tile is 64 keys x 128 dims of K and of V, rows of 256 bytes.  A direct load writes lane L's
// 16 bytes at base + 16 L, so rows cannot be padded; bank conflicts are avoided by choosing WHICH 16-byte
// chunk a lane fetches: position c' of K row r holds chunk c' ^ (r & 15), of V row r chunk c' ^ ((r & 3) << 2).
// Tiles past the end are fetched through a zero-length buffer descriptor (they arrive as zeros).
// Softmax: every S chain starts from an accumulator holding -(running max), so the MFMA result is the exponent;
// the running max is set by the first tile and raised only when a lane's probability sum over its 32 keys
// reaches 2^30 (which also catches any overflow).
//
// A wavefront's tile is a chain S (16 MFMAs) -> softmax (32 exp2 on the transcendental unit, ~640
// cycles) -> PV (16 MFMAs).  Left alone, the two wavefronts of a SIMD drift into the same phase:
// the older one wins every arbitration, runs its chain at full speed, and the younger one finishes
// a pair of tiles ~30 % later, mostly alone on the SIMD with the matrix pipe idle during its softmax.
// Here wavefronts 0..3 (group A, one per SIMD) and 4..7 (group B, their SIMD mates) are
// offset by one S block with two workgroup barriers per tile:
//
//      barrier X(t) | A: S(t)                    | barrier Y(t) | A: softmax, PV, prefetch K frags of t+1
//                   | B: loads of t+3, K frags t |              | B: S(t), softmax, PV
//
// so the matrix pipe sees S_A, S_B, PV_A, PV_B back to back while each softmax runs beside the
// other group's MFMAs.  Group B issues all direct loads (8 per wavefront per tile) in the slot in
// which it waits for A's S block; group A uses its slot at the end of the tile to fetch the first K
// fragments of the next one.  A passes Y some MFMAs before the end of its S block (four with 128 dims; all its fragment reads
// are out by then), so B's first MFMAs queue behind A's last ones instead of meeting an idle pipe.
//
// The first workgroups of the launch can carry the step's selection (and the sum of the retaining head's
// partial scores before it): see the kernel body and select_body.h.
//
// Ring of 4 stages, one tile per step.  Invariant at X(t): tiles t and t+1 have landed in LDS (B waits
// for its own loads of tile t+2 before it arrives at X(t+1): s_waitcnt vmcnt(8) leaves only the 8 loads
// of tile t+3 in flight) and every wavefront has finished tile t-1, whose stage the loads of tile t+3
// overwrite.
//
// The V^T fragments are read with ds_read_b64_tr_b16 from inline assembly, with hand-counted
// s_waitcnt lgkmcnt: the compiler puts an s_waitcnt vmcnt(0) in front of the intrinsic form (it
// cannot tell that those reads never touch a stage with a load in flight), which would stall every
// PV block on the loads just issued.  LDS operations return in order, so a count of the asm reads
// issued after the wanted one is always sufficient, whatever else the compiler has in flight.
#include <hip/hip_ext.h>

#include "attn_common.h"
#include "kernels.h"
#include "select_body.h"

namespace locret {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(3))) unsigned char* lds_u8_ptr;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int PP_ROWB = 256;                   // bytes of a row in LDS: 128 bf16; head_dim 96 leaves the last quarter unused
constexpr int PP_ROWS = 64;                    // rows of a tile: its keys, or with head_dim 64 two keys each
constexpr int PP_TILE_B = PP_ROWS * PP_ROWB;   // 16 KB per operand tile
__host__ __device__ constexpr int pp_tile_keys(int d) { return d == 64 ? 2 * PP_ROWS : PP_ROWS; }
constexpr int PP_STAGE_B = 2 * PP_TILE_B;      // K then V
constexpr int PP_NW = 8;
constexpr int PP_KPRE = 4;                     // K fragments fetched ahead of the S block
// MFMAs of group A's S block issued behind barrier Y.  Fewer than four where the softmax takes the longer part of a tile.  Steps of 300 to
// 4096 tokens on 4096 and 8192 units, five runs in turn (the runs of one side differ by 1 to 3 %, by 0.6 % with head-wise budgets), means over
// the ten shapes against four: 96 dims with two 0.992 on 32 heads, 0.986 on 8, with one 0.993, 0.991 (20480 tokens on 32 heads of 8192
// units, in turn: one 2509, two 2494 us); 96 dims with head-wise budgets, one 0.984, in every shape; 64 dims, one 0.993 on 8 heads, 0.998
// on 32, 1.000 with budgets.  128 dims, 15900 tokens on 8 heads of 6144, with two, four, six: 1825, 1820, 1848 us.
constexpr int pp_ytail(int d, bool general) { return d == 128 ? 4 : d == 96 && !general ? 2 : 1; }
constexpr int PP_SEL_MAXR = 48;                // keys per thread of a selection workgroup (512 threads)
constexpr int PP_MAX_PARTS = 16;               // key ranges per (head group, token tile) item at most
constexpr int PP_MAX_SLOTS = 256;              // partial results (256 query rows each) the buffer holds at most
constexpr int PP_CUT_SLACK = 4;                // key tiles by which the last part may exceed the part length
constexpr int PP_CUS = 256, PP_XCD_CUS = 32;   // compute units of the device and of one XCD

// Where a launch cuts items (head group, token tile) into parts along the keys.  Only the first n_donors items of the
// dispatch order, the longest, are cut: into k equal parts, or (k == 0) into parts of tau key tiles, the last one
// taking what is left.  Part 0 of every item comes first in the launch, then part 1 of the donors, and so on.
struct PPCut {
  int n_items;
  int n_donors;
  int k, tau;
  int n_slots;        // n_donors * (parts at most): part p of donor i leaves its partial result in slot p * n_donors + i
  __host__ __device__ int parts(int i, int tiles) const {
    if (i >= n_donors) return 1;
    if (k > 0) return k;
    return tiles <= tau + PP_CUT_SLACK ? 1 : (tiles - PP_CUT_SLACK + tau - 1) / tau;
  }
};

// Dispatch order: item i of the launch -> head group and token tile.
struct PPOrder {
  int n_hgroups, n_ttiles, gph, n_sel, spread;      // gph: head groups per KV head
  HeadOrder heads;
};
__device__ __forceinline__ void pp_item(const PPOrder& o, bool spread, int i, int& hgroup, int& tt) {
  if (spread) {
    // Head-wise budgets: with one KV head per XCD the XCD of the longest head would set the launch's time.
    // Instead the token tiles go round the XCDs head after head, the heads from the longest cache to
    // the shortest, so that all XCDs hold the same work and each hands out its long items first.
    // (Measured on 8 heads of 28672 ... 4096 units, mean 16384: 1.61 ms per step with one head
    // per XCD, 1.39 ms with the heads interleaved item by item, 1.14 ms in this order; equal heads 1.07 ms.)
    // Heads follow one another without padding: with every head starting on the first XCD a chunk of one token tile
    // puts all of its items there.  (32 heads of 96 dims with up to 16278 units, 20439 tokens in chunks of 4047 and 45 more,
    // which is two such chunks: 3381 us a prompt in this order, 3839 us padded; 3486 us before items were cut at the
    // mean load, when every item of such a chunk was cut into eight equal parts, one for each XCD.)
    const int r = i / o.n_ttiles;                          // rank of the head group, longest first
    hgroup = o.heads.v[r / o.gph] * o.gph + r % o.gph;
    tt = i % o.n_ttiles;
  } else if ((o.n_hgroups & 7) == 0) {                     // one KV head per XCD (workgroup ids go round the XCDs)
    const int g8 = o.n_hgroups >> 3;
    hgroup = ((i + o.n_sel) & 7) * g8 + (i >> 3) % g8;
    tt = i / o.n_hgroups;
  } else {
    hgroup = i % o.n_hgroups;
    tt = i / o.n_hgroups;
  }
  tt = o.n_ttiles - 1 - tt;                                // longest key ranges first
}

#define LOCRET_TR_READ(dst, addr, off) \
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "i"(off) : "memory")
#define LOCRET_LGKM_WAIT(a, b, n) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "i"(n))

// GENERAL = false is the common case: every KV head holds n_c_common units, one KV head per XCD, the whole key
// range per workgroup (n_c_h, order.spread, cut and part are ignored, so nothing of head-wise lengths, the spread
// launch order or the cut items remains in its code).
// D = 128, 96 or 64.  The tile layout in LDS is that of 128 dims for both (rows of 256 bytes): with 96 dims the lanes
// of a direct load that would fetch the last four 16-byte chunks of a row point outside the buffer instead and
// bring zeros, which nothing reads; every fragment address stays as it is, S takes 6 contraction steps and O^T
// has 3 blocks of 32 dims.  With 64 dims a tile is 128 keys: row r holds key r in its first and key r + 64 in its second
// half, so the addresses stay as they are again: the K fragment of contraction step ks >= 4 is step ks - 4 of
// keys 64 .. 127, the V^T fragment of dim block db >= 2 is block db - 2 of those keys.  A tile then takes as many MFMAs
// as with 128 dims and twice the softmax, which bounds it.  (32q/8kv x 64, chunks of 2048 on 0 .. 4096 units: 99 us a launch
// on the register-staged kernel with the selection and a reduction in launches of their own, 12 us; 87 us here with both
// inside.)
template <int D, bool GENERAL>
__global__ __launch_bounds__(PP_NW * 64, 2) void attn_pp_kernel(const bf16_t* __restrict__ q, const float2* __restrict__ tab, const bf16_t* __restrict__ Kx,
                                                             const bf16_t* __restrict__ V, bf16_t* __restrict__ out,
                                                             int Tn, int h, int g, int cap, int n_c_common, float c_log2,
                                                             int hpw, PPOrder order, SelectArgs sel, int n_sel,
                                                             HeadLens n_c_h, PPCut cut, float* __restrict__ part) {
  constexpr int NW = PP_NW;
  static_assert(D == 128 || D == 96 || D == 64, "head dims of this kernel");
  constexpr int NKS = D / 16;                  // contraction steps of S
  constexpr int NDB = D / 32;                  // 32-dim blocks of O^T
  constexpr int KT = pp_tile_keys(D);
  constexpr int KH = KT / PP_ROWS;             // keys per LDS row
  constexpr int NKB = KT / 32;                 // 32-key blocks of a tile
  constexpr int PP_VPRE = KH == 2 ? 2 : 4;     // V^T fragments in flight ahead of their MFMA (64 dims: no registers for more)
  constexpr int NKF = KH * NKS, NVF = KH * NDB;     // K fragments per row block, V^T fragments per 16-row chunk
  __shared__ __attribute__((aligned(1024))) unsigned char ring[4 * PP_STAGE_B];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31;
  const int hi = lane >> 5;

  // The first n_sel workgroups of the launch do not attend: each runs the top-k selection of one KV head
  // (it depends on the scores only, which are complete before the launch) and retires after a few tens
  // of microseconds, long before the attention workgroups that follow it on the same CU would have started
  // their second round; the selection's latency disappears from the step.
  if ((int)blockIdx.x < n_sel) {
    select_reg_body<PP_SEL_MAXR, PP_NW * 64, 4>(sel, blockIdx.x, (uint32_t*)ring);
    static_assert(select_body_smem_words(PP_NW * 64, 4) * 4 <= (int)sizeof(ring), "the selection's scratch fits the ring");
    return;
  }
  int item = blockIdx.x - n_sel, layer = 0;
  if (GENERAL && item >= cut.n_items) {
    const int x = item - cut.n_items;
    layer = 1 + x / cut.n_donors;
    item = x % cut.n_donors;
  }
  int hgroup, tt;
  pp_item(order, GENERAL && order.spread, item, hgroup, tt);
  const int wph = NW / hpw;
  const int TW = wph * 32;
  const int t0 = tt * TW;
  const int j = hgroup * hpw + wave / wph;
  const int m = (hgroup * hpw) / g;
  const int n_c = GENERAL ? __builtin_amdgcn_readfirstlane(head_len(n_c_h, m, n_c_common)) : n_c_common;   // this KV head's cache length
  const int tw0 = t0 + (wave % wph) * 32;
  const int t_last_wg = min(Tn, t0 + TW) - 1;
  const int n_keys = n_c + t_last_wg + 1;
  const int n_tiles_all = (n_keys + KT - 1) / KT;
  // A cut item: this workgroup takes the key tiles [t_lo, t_lo + n_tiles) of its queries' range and leaves
  // un-normalised partial results for the merge kernel.
  int t_lo = 0, n_tiles = n_tiles_all, n_parts = 1;
  if (GENERAL) {
    n_parts = cut.parts(item, n_tiles_all);
    if (layer >= n_parts) return;
    if (n_parts > 1) {
      const int len = cut.k > 0 ? (n_tiles_all + n_parts - 1) / n_parts : cut.tau;
      t_lo = layer * len;
      n_tiles = max(0, (layer == n_parts - 1 ? n_tiles_all : min(n_tiles_all, t_lo + len)) - t_lo);
    }
  }
  const int n_keys_s = min(n_keys, (t_lo + n_tiles) * KT);
  const int wave_last_slot = n_c + min(Tn - 1, tw0 + 31);
  const int my_t = min(tw0 + n32, Tn - 1);
  const int limit = n_c + my_t;

  auto scalar_ptr = [](const bf16_t* p) -> const bf16_t* {
    uint64_t a = (uint64_t)p;
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    uint32_t hi32 = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (const bf16_t*)(((uint64_t)hi32 << 32) | lo);
  };
  const bf16_t* Kb = scalar_ptr(Kx + (int64_t)m * cap * D);
  const bf16_t* Vb = scalar_ptr(V + (int64_t)m * cap * D);

  bf16x8 qf[NKS];
  {
    const bf16_t* qp = q + ((int64_t)my_t * h + j) * D + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8*)(qp + ks * 16);
    const float qscale = c_log2;                 // logits come out of the MFMA in log2 units
    if (tab != nullptr) {
      // un-rotated queries: rotate to position n_c + t here (pairs (i, i + D/2) sit in fragments ks
      // and ks + NKS/2 of the same lane), round to bf16 as the append kernel would have
      const float2* tp = tab + (int64_t)(n_c + my_t) * (D / 2) + hi * 8;
#pragma unroll
      for (int ks = 0; ks < NKS / 2; ++ks) {
        float lo[8], up[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float2 cs = tp[ks * 16 + e];
          const float a = (float)qf[ks][e], b = (float)qf[ks + NKS / 2][e];
          lo[e] = (a * cs.x - b * cs.y) * qscale;
          up[e] = (b * cs.x + a * cs.y) * qscale;
        }
        uint4 pl = make_uint4(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(lo[4], lo[5]), pack_bf16(lo[6], lo[7]));
        uint4 pu = make_uint4(pack_bf16(up[0], up[1]), pack_bf16(up[2], up[3]), pack_bf16(up[4], up[5]), pack_bf16(up[6], up[7]));
        qf[ks] = __builtin_bit_cast(bf16x8, pl);
        qf[ks + NKS / 2] = __builtin_bit_cast(bf16x8, pu);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (float)qf[ks][e] * qscale;
        uint4 px = make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7]));
        qf[ks] = __builtin_bit_cast(bf16x8, px);
      }
    }
  }
  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m_run = 0.f, l_run = 0.f;
  // m_run is in log2 units and negm holds -m_run in all 16 registers: the first MFMA of every S
  // chain takes it as its addend, so the accumulator ends as (logit - running max) and exp2 applies
  // to it directly.  `fresh` (wave-uniform) is true until the first tile has set the max.
  f32x16 negm;
#pragma unroll
  for (int r = 0; r < 16; ++r) negm[r] = 0.f;
  bool fresh = true;

  const bool isB = wave >= NW / 2;             // wave-uniform; wavefronts w and w + 4 share a SIMD

  // ---- direct loads (group B): instruction i of a tile covers rows 4i .. 4i+3; wavefront w issues
  // ---- instructions w%4 + 4u, so (i & 3) is the same for all of them ----------------------------------
  const int w4 = wave & 3;
  const int l_row = lane >> 4, l_pos = lane & 15;
  // the lane's LDS slot is row 4 i + l_row, position l_pos; the row's swizzle decides which chunk of the row in
  // memory belongs there.  Memory rows are D * 2 bytes; instruction i = w4 + 4 u starts at row 16 u + 4 w4.
  constexpr int NCH = D / 8;                     // 16-byte chunks of a row in memory
  constexpr int OUTSIDE = 0x7ffff000;            // an offset no buffer reaches: the load brings zeros
  const int k_ch = l_pos ^ l_row ^ (w4 << 2), v_ch = l_pos ^ (l_row << 2);
  auto offset = [&](int ch) {                    // + u * 16 rows (scalar offset)
    return ch < KH * NCH ? ((ch / NCH) * PP_ROWS + w4 * 4 + l_row) * (D * 2) + (ch % NCH) * 16 : OUTSIDE;
  };
  const int k_vo = offset(k_ch), v_vo = offset(v_ch);
  auto issue = [&](int tile, int stage) __attribute__((always_inline)) {
    const int tile_u = __builtin_amdgcn_readfirstlane(tile);
    const int left = __builtin_amdgcn_readfirstlane(max(n_keys_s - tile_u * KT, 0) * (D * 2));   // 0 past the end
    __amdgpu_buffer_rsrc_t kr =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Kb + (int64_t)tile_u * (KT * D)), 0, left, 0x00020000);
    __amdgpu_buffer_rsrc_t vr =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Vb + (int64_t)tile_u * (KT * D)), 0, left, 0x00020000);
    unsigned char* sb = ring + stage * PP_STAGE_B;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = w4 + u * 4;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (lds_ptr_t)(sb + i * 1024), 16, k_vo, u * (16 * D * 2), 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = w4 + u * 4;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lds_ptr_t)(sb + PP_TILE_B + i * 1024), 16, v_vo, u * (16 * D * 2), 0, 0);
    }
  };

  // ---- fragment addresses (bytes inside a stage) ---------------------------------------------------
  const int kx = n32 & 15;
  const int k_base = n32 * 256 + ((kx >> 1) << 5) + ((hi ^ (kx & 1)) << 4);
  // the address of a step's fragment, base ^ (step << 5), is kept in a register per step, except with 64 dims: the
  // probabilities of 128 keys leave no room, and the reload of a spilled register would wait for the loads in flight
  int k_rd[NKF];
#pragma unroll
  for (int ks = 0; ks < NKF; ++ks) k_rd[ks] = k_base ^ (ks << 5);
  auto k_at = [&](int base, int ks) __attribute__((always_inline)) { return KH == 2 ? base ^ (ks << 5) : base + k_rd[ks]; };
  auto k_stage = [&](int sb_off) __attribute__((always_inline)) {
    int base = sb_off;
    if (KH == 2) {
      base += k_base;                            // k_base < 16 KB, the stage's offset is a multiple of 32 KB
      asm volatile("" : "+v"(base));             // formed anew for every tile
    }
    return base;
  };
  const int vs = lane & 15, vG = lane >> 4;
  const int v_base = PP_TILE_B + (((vG >> 1) * 4 + (vs >> 2)) * 256) + ((vs >> 2) << 6) +
                     ((((vG & 1) << 1) + ((vs & 3) >> 1)) << 4) + ((vs & 1) << 3);
  // LDS byte addresses of stage 0 for the asm reads
  const uint32_t ring_lds = (uint32_t)(uintptr_t)(lds_u8_ptr)ring;
  uint32_t v_ad[NVF];
#pragma unroll
  for (int db = 0; db < NVF; ++db) v_ad[db] = ring_lds + (uint32_t)(v_base ^ (db << 6));

  bf16x8 kpre[PP_KPRE];                          // fragment f = ks * 2 + kb of the tile whose S block comes next
  auto prefetch_k = [&](int sb_off) __attribute__((always_inline)) {
    const int base = k_stage(sb_off);
#pragma unroll
    for (int f = 0; f < PP_KPRE; ++f) kpre[f] = *(const bf16x8*)(ring + k_at(base, f >> 1) + (f & 1) * 32 * 256);
  };

  // `mid` runs before the last `tail` MFMAs are issued (all fragment reads are out by then).  Fragment f: step f / 2 of
  // row block f % 2.
  auto s_block = [&](f32x16 (&sacc)[NKB], int sb_off, auto mid, auto tail_c) __attribute__((always_inline)) {
    constexpr int TAIL = decltype(tail_c)::value;    // 0: no split
    const int base = k_stage(sb_off);
    bf16x8 kf[NKF][2];
#pragma unroll
    for (int f = 0; f < 2 * NKF; ++f)
      kf[f >> 1][f & 1] = f < PP_KPRE ? kpre[f] : *(const bf16x8*)(ring + k_at(base, f >> 1) + (f & 1) * 32 * 256);
    auto mfma = [&](int f) __attribute__((always_inline)) {
      const int ks = (f >> 1) % NKS, kb = (f >> 1) / NKS * 2 + (f & 1);
      sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[f >> 1][f & 1], qf[ks], ks == 0 ? negm : sacc[kb], 0, 0, 0);   // the S chain starts from -(running max)
    };
#pragma unroll
    for (int f = 0; f < 2 * NKF - TAIL; ++f) mfma(f);
#pragma unroll
    for (int i = 0; i < 2 * NKF - PP_KPRE; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if (TAIL < PP_KPRE) __builtin_amdgcn_sched_group_barrier(0x008, PP_KPRE - TAIL, 0);
    if (TAIL > 0) {
      mid();
#pragma unroll
      for (int f = 2 * NKF - TAIL; f < 2 * NKF; ++f) mfma(f);
    }
  };

  // softmax and PV of one tile; the S accumulators are in sacc
  auto softmax_pv = [&](f32x16 (&sacc)[NKB], int tile, int sb_off) __attribute__((always_inline)) {
    const int base = tile * KT;
    uint32_t va[NVF];
#pragma unroll
    for (int db = 0; db < NVF; ++db) va[db] = v_ad[db] + (uint32_t)sb_off;
    // V^T fragment f = kc * NVF + db: two transposing 8-byte reads (rows +0..3 and +8..11 of the 16-row chunk kc)
    s16x4 vlo[4 * NVF], vhi[4 * NVF];
#pragma unroll
    for (int f = 0; f < PP_VPRE; ++f) {
      LOCRET_TR_READ(vlo[f], va[f % NVF], (f / NVF) * 4096);
      LOCRET_TR_READ(vhi[f], va[f % NVF], (f / NVF) * 4096 + 2048);
    }
    if (base + KT - 1 > n_c + tw0) {           // wave-uniform: tile crosses the diagonal
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int slot = base + kb * 32 + (r >> 2) * 8 + hi * 4 + (r & 3);
          if (slot > limit) sacc[kb][r] = -INFINITY;
        }
    }
    uint4 pb[2 * NKB];                          // probabilities of keys 16 kc .. + 15
    {
      float ps;
      auto exp_pack_sum = [&]() __attribute__((always_inline)) {
        float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          uint32_t w[8];
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            const float e0 = __builtin_amdgcn_exp2f(sacc[kb][r]), e1 = __builtin_amdgcn_exp2f(sacc[kb][r + 1]);
            w[r >> 1] = pack_bf16(e0, e1);
            ps0 += e0;
            ps1 += e1;
          }
          pb[kb * 2 + 0] = make_uint4(w[0], w[1], w[2], w[3]);
          pb[kb * 2 + 1] = make_uint4(w[4], w[5], w[6], w[7]);
        }
        ps = ps0 + ps1;
      };
      exp_pack_sum();
      if (fresh || __any(!(ps < RESCALE_SUM))) {     // rare: set or raise the running max
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[kb][r]);
        mx = max_across_halves(mx);
        // Cut items only: in the part that holds the diagonal a query may see none of the part's keys
        // (its row of the first tile is wholly masked, and every later tile lies further right).  Such a lane keeps
        // max 0 and sum 0, and the merge kernel drops partials whose sum is 0; without the test it would form
        // -inf - (-inf).  In unsplit launches every query sees key 0, which lies in the first tile.
        const float delta = fresh ? ((GENERAL && mx == -INFINITY) ? 0.f : mx) : fmaxf(mx, 0.f);
        const float alpha = fresh ? 0.f : __builtin_amdgcn_exp2f(-delta);
        m_run += delta;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) negm[r] = -m_run;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[kb][r] -= delta;
        fresh = false;
        exp_pack_sum();
      }
      l_run += ps;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < 4 * NVF; ++f) {
      constexpr int LASTF = 4 * NVF - 1;
      const int newest = f + PP_VPRE - 1 < LASTF ? f + PP_VPRE - 1 : LASTF;   // newest fragment already requested
      // reads issued after fragment f's: two per fragment
      static_assert(PP_VPRE <= 6, "lgkmcnt cases");
      switch (2 * (newest - f)) {
        case 10: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 10); break;
        case 8: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 8); break;
        case 6: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 6); break;
        case 4: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 4); break;
        case 2: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 2); break;
        default: LOCRET_LGKM_WAIT(vlo[f], vhi[f], 0); break;
      }
      const s16x8 both = __builtin_shufflevector(vlo[f], vhi[f], 0, 1, 2, 3, 4, 5, 6, 7);
      oacc[f % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both),
                                                              *(const bf16x8*)&pb[f / NVF + 4 * (f % NVF / NDB)],
                                                              oacc[f % NDB], 0, 0, 0);
      if (f + PP_VPRE < 4 * NVF) {
        const int fn = f + PP_VPRE;
        LOCRET_TR_READ(vlo[fn], va[fn % NVF], (fn / NVF) * 4096);
        LOCRET_TR_READ(vhi[fn], va[fn % NVF], (fn / NVF) * 4096 + 2048);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto wg_barrier = []() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // tiles this wavefront's queries can see (wave-uniform, <= n_tiles): later tiles only keep the barriers
  const int n_active = max(0, min(n_tiles, wave_last_slot / KT + 1 - t_lo));
  if (isB) {
    issue(t_lo, 0);
    issue(t_lo + 1, 1);
    issue(t_lo + 2, 2);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");            // tiles 0 and 1 have landed
    wg_barrier();
    for (int t = 0; t < n_active; ++t) {
      const int sb_off = (t & 3) * PP_STAGE_B;
      wg_barrier();                                              // X(t)
      issue(t_lo + t + 3, (t + 3) & 3);
      prefetch_k(sb_off);
      wg_barrier();                                              // Y(t)
      f32x16 sacc[NKB];
      s_block(sacc, sb_off, []() {}, IntC<0>());
      softmax_pv(sacc, t_lo + t, sb_off);
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");          // own loads of tile t+2 have landed
    }
    for (int t = n_active; t < n_tiles; ++t) {
      wg_barrier();
      issue(t_lo + t + 3, (t + 3) & 3);
      wg_barrier();
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    }
  } else {
    wg_barrier();
    prefetch_k(0);
    for (int t = 0; t < n_active; ++t) {
      const int sb_off = (t & 3) * PP_STAGE_B;
      wg_barrier();                                              // X(t)
      f32x16 sacc[NKB];
      s_block(sacc, sb_off, wg_barrier, IntC<pp_ytail(D, GENERAL)>());        // Y(t), passed that many MFMAs before the end of the block
      softmax_pv(sacc, t_lo + t, sb_off);
      prefetch_k(((t + 1) & 3) * PP_STAGE_B);
    }
    for (int t = n_active; t < n_tiles; ++t) {
      wg_barrier();
      wg_barrier();
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // trailing empty loads

  // ---- epilogue ---------------------------------------------------------------------------------
  {
    const int t = tw0 + n32;
    float l = l_run + __shfl_xor(l_run, 32, 64);
    if (GENERAL && n_parts > 1) {
      // partial result of this part: O un-normalised, running max (log2 units) and sum; a query that saw no key
      // leaves sum 0 and O 0 (its accumulators hold 0, or NaN where a key of the part that it must not see has a value that is
      // not finite: 0 times it).  The accumulators go out as they lie in the registers, 1 KB in a row per store.
      if (__any(l == 0.f)) {
        const bool none = l == 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[db][r] = none ? 0.f : oacc[db][r];
      }
      const int64_t slot = (int64_t)layer * cut.n_donors + item;
      float4* op = (float4*)part + (slot * NW + wave) * (NDB * 4 * 64) + lane;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
          op[(db * 4 + rq) * 64] =
              make_float4(oacc[db][rq * 4 + 0], oacc[db][rq * 4 + 1], oacc[db][rq * 4 + 2], oacc[db][rq * 4 + 3]);
      if (hi == 0) ((float2*)(part + (int64_t)cut.n_slots * (NW * 32) * D))[slot * (NW * 32) + wave * 32 + n32] = make_float2(m_run, l);
    } else if (t < Tn) {
      const float inv = 1.f / l;
      bf16_t* op = out + ((int64_t)t * h + j) * D;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          uint2 w;
          w.x = pack_bf16(oacc[db][rq * 4 + 0] * inv, oacc[db][rq * 4 + 1] * inv);
          w.y = pack_bf16(oacc[db][rq * 4 + 2] * inv, oacc[db][rq * 4 + 3] * inv);
          *(uint2*)(op + db * 32 + rq * 8 + hi * 4) = w;
        }
    }
  }
}

// out[t][j][:] = sum_p w_p O_p / sum_p w_p l_p with w_p = 2^(m_p - max m) over the parts of a cut item.  A part whose
// sum is 0 saw no key of that row (a sum that is NaN makes the row NaN).  One workgroup per (donor, 32 dims), its threads as
// in the attention kernel.
template <int D>
__global__ __launch_bounds__(PP_NW * 64) void attn_pp_merge_kernel(const float* __restrict__ part, bf16_t* __restrict__ out,
                                                                   int Tn, int h, int g, int n_c_common, int hpw, PPOrder order,
                                                                   HeadLens n_c_h, PPCut cut) {
  constexpr int NW = PP_NW, NDB = D / 32, KT = pp_tile_keys(D);
  const int item = blockIdx.x, db = blockIdx.y;
  int hgroup, tt;
  pp_item(order, order.spread, item, hgroup, tt);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n32 = lane & 31, hi = lane >> 5;
  const int wph = NW / hpw, TW = wph * 32;
  const int n_c = head_len(n_c_h, (hgroup * hpw) / g, n_c_common);
  const int n_parts = cut.parts(item, (n_c + min(Tn, (tt + 1) * TW) + KT - 1) / KT);
  if (n_parts == 1) return;
  const float2* ml = (const float2*)(part + (int64_t)cut.n_slots * (NW * 32) * D) + wave * 32 + n32;
  const float4* op = (const float4*)part + (int64_t)wave * (NDB * 4 * 64) + db * (4 * 64) + lane;
  float M = -INFINITY;
  for (int p = 0; p < n_parts; ++p) {
    const float2 x = ml[((int64_t)p * cut.n_donors + item) * (NW * 32)];
    if (x.y > 0.f) M = fmaxf(M, x.x);
  }
  float acc[16], den = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  for (int p = 0; p < n_parts; ++p) {
    const int64_t slot = (int64_t)p * cut.n_donors + item;
    const float2 x = ml[slot * (NW * 32)];
    float4 o[4];
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) o[rq] = op[slot * (NW * NDB * 4 * 64) + rq * 64];
    const float w = x.y > 0.f ? __builtin_amdgcn_exp2f(x.x - M) : 0.f;     // such a part's O is 0 too
    den = fmaf(w, x.y, den);
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      acc[rq * 4 + 0] = fmaf(w, o[rq].x, acc[rq * 4 + 0]);
      acc[rq * 4 + 1] = fmaf(w, o[rq].y, acc[rq * 4 + 1]);
      acc[rq * 4 + 2] = fmaf(w, o[rq].z, acc[rq * 4 + 2]);
      acc[rq * 4 + 3] = fmaf(w, o[rq].w, acc[rq * 4 + 3]);
    }
  }
  const int t = tt * TW + (wave % wph) * 32 + n32;
  if (t >= Tn) return;
  const float inv = 1.f / den;      // every query sees at least its own key
  bf16_t* dst = out + ((int64_t)t * h + hgroup * hpw + wave / wph) * D + db * 32 + hi * 4;
#pragma unroll
  for (int rq = 0; rq < 4; ++rq) {
    uint2 w;
    w.x = pack_bf16(acc[rq * 4 + 0] * inv, acc[rq * 4 + 1] * inv);
    w.y = pack_bf16(acc[rq * 4 + 2] * inv, acc[rq * 4 + 3] * inv);
    *(uint2*)(dst + rq * 8) = w;
  }
}

static bool pp_head_dim(int d) { return d == 128 || d == 96 || d == 64; }

static int pp_heads_per_wg(int g) { return g % 8 == 0 ? 8 : g % 4 == 0 ? 4 : g % 2 == 0 ? 2 : 1; }

// Floats of workspace for the partial results of cut items: room for every item of the longest chunk in 8 parts, up to
// PP_MAX_SLOTS (34 MB at 128 dims).  0: this shape never cuts.
size_t attention_pp_split_floats(const Dims& Dm, int chunk_max) {
  if (!pp_head_dim(Dm.d) || !Dm.bf16) return 0;
  const int hpw = pp_heads_per_wg(Dm.g), TW = PP_NW / hpw * 32;
  const int64_t slots = (int64_t)8 * (Dm.h / hpw) * ((chunk_max + TW - 1) / TW);
  return (size_t)(slots < PP_MAX_SLOTS ? slots : PP_MAX_SLOTS) * (PP_NW * 32) * (Dm.d + 2);
}

// Which items of a launch to cut.  The unit is the key tile (1.7 us of a workgroup).  Workgroups occupy a CU each, so a
// short chunk, whose I items are at most half as many as the P CUs (both per XCD where the order deals items to XCDs),
// leaves most of the chip idle: the items longer than tau, about the mean load of a CU, are cut there, and the
// remainders come last in the launch and go to the CUs that had nothing or are done first.
// A cut costs the writing, reading and merging of partial results and a second prologue, about PP_CUT_COST tiles at
// the end of a launch; without that much gain nothing is cut.  With more items nothing is cut either, however
// uneven they are: the chip is limited by power there, the busy CUs of an uneven launch run faster, and cutting 256
// items of 97 ... 128 tiles to equal loads (or 256 items of 32 ... 256 tiles) took as long as leaving them whole
// (222 us against 215, 298 against 300), plus 9-13 us for the merge.
// Tuning::pp_split: 0 = never, k = every item into k parts (both bounded by the buffer).
constexpr int PP_CUT_COST = 6;
static PPCut plan_cut(const Dims& Dm, const PPOrder& o, const HeadLens& hl, int T, int n_c, int TW, size_t floats) {
  PPCut cut = {};
  const int lists = o.spread || (o.n_hgroups & 7) == 0 ? 8 : 1;           // item lists that share no CU
  const int P = lists == 8 ? PP_XCD_CUS : PP_CUS;
  const int KT = pp_tile_keys(Dm.d);
  cut.n_items = o.n_hgroups * o.n_ttiles;
  const int max_slots = (int)(floats / ((size_t)(PP_NW * 32) * (Dm.d + 2)));
  if (max_slots == 0 || Dm.tune.pp_split == 0 || Dm.tune.pp_split == 1) return cut;
  if (Dm.tune.pp_split > 1) {
    int k = Dm.tune.pp_split < PP_MAX_PARTS ? Dm.tune.pp_split : PP_MAX_PARTS;
    while (k > 1 && (int64_t)k * cut.n_items > max_slots) --k;
    if (k > 1) { cut.k = k; cut.n_donors = cut.n_items; cut.n_slots = k * cut.n_items; }
    return cut;
  }
  const int I = (cut.n_items + lists - 1) / lists;
  auto tiles = [&](int nc, int tt) { const int e = (tt + 1) * TW; return (nc + (T < e ? T : e) + KT - 1) / KT; };
  auto rank_len = [&](int r) { return hl.ragged ? hl.v[o.spread ? o.heads.v[r] : r] : n_c; };     // r-th KV head of the order
  const int heads = hl.ragged ? Dm.h_kv : 1;
  int64_t sum = 0;                          // tiles of all items (a KV head has gph head groups)
  int longest = 0;
  for (int r = 0; r < heads; ++r)
    for (int tt = 0; tt < o.n_ttiles; ++tt) {
      const int c = tiles(rank_len(r), tt);
      sum += c;
      longest = c > longest ? c : longest;
    }
  sum *= hl.ragged ? o.gph : o.n_hgroups;
  const int mean = (int)((sum + (int64_t)lists * P - 1) / ((int64_t)lists * P));        // load of a CU
  if (2 * I <= P) {
    int tau = mean + 2 > 8 ? mean + 2 : 8;
    if (tau < (longest + PP_MAX_PARTS - 1) / PP_MAX_PARTS) tau = (longest + PP_MAX_PARTS - 1) / PP_MAX_PARTS;
    for (;; tau += 1 + tau / 8) {
      if (longest < tau + PP_CUT_SLACK + PP_CUT_COST) return cut;
      int donors = 0;
      if (o.spread) {                       // whole heads of the order, up to the last one with an item to cut
        for (int r = 0; r < heads; ++r)
          if (tiles(rank_len(r), o.n_ttiles - 1) > tau + PP_CUT_SLACK) donors = (r + 1) * o.gph * o.n_ttiles;
      } else {                              // the order goes through the token tiles from the longest on
        int nt = 0;
        for (int r = 0; r < heads; ++r)
          for (int tt = 0; tt < o.n_ttiles; ++tt)
            if (tiles(rank_len(r), tt) > tau + PP_CUT_SLACK) { nt = nt > o.n_ttiles - tt ? nt : o.n_ttiles - tt; break; }
        donors = nt * o.n_hgroups;
      }
      const int parts = (longest - PP_CUT_SLACK + tau - 1) / tau;
      if ((int64_t)parts * donors > max_slots) continue;
      cut.tau = tau; cut.n_donors = donors; cut.n_slots = parts * donors;
      return cut;
    }
  }
  return cut;
}

// `tab` non-null: q holds un-rotated queries and the kernel rotates them (table row n_c + t).
bool attention_pp_fuses_select(const Dims& Dm, int n_cand) {
  if (!pp_head_dim(Dm.d) || (int64_t)Dm.cap * Dm.d * 2 >= (1ll << 31)) return false;
  const int wseg = ((n_cand + PP_NW - 1) / PP_NW + 63) & ~63;
  return wseg <= PP_SEL_MAXR * 64;
}

// The selection's workgroups sum the partials as long as that hides behind the attention: a thread walks n_parts partials for
// each of its tokens.  A step with 8 KV heads, summed there or reduced before it: T = 3072, 64 partials (384 a thread): 128 dims
// 458.5, 475.5 us, 64 dims 272.5, 282.4; T = 4096, 64 partials (512 a thread): 128 dims 658.5, 629.8 us, 64 dims 385.1, 366.7.
bool attention_bf16_sums_partials(int n_parts, int T) { return (T + PP_NW * 64 - 1) / (PP_NW * 64) * n_parts <= 384; }

// `sel` non-null (and attention_pp_fuses_select true): the launch also performs that selection.
bool launch_attention_bf16_pp(const Dims& Dm, LaunchTimer tm, const void* q, const float2* tab, const void* Kx, const void* V, void* out,
                              int T, int n_c, float scale, hipStream_t st, const SelectArgs* sel,
                              const HeadLens* n_c_h, float* split_part, size_t split_floats) {
  if (!pp_head_dim(Dm.d)) return false;
  if ((int64_t)Dm.cap * Dm.d * 2 >= (1ll << 31)) return false;   // 32-bit byte offsets inside one head
  constexpr int NW = PP_NW;
  const int g = Dm.g;
  const int hpw = pp_heads_per_wg(g);
  const int TW = NW / hpw * 32;
  const int n_hgroups = Dm.h / hpw;
  const int n_ttiles = (T + TW - 1) / TW;
  const float c_log2 = scale * 1.4426950408889634f;
  const int n_sel = sel ? Dm.h_kv : 0;
  const HeadLens hl = head_lens_or_common(n_c_h);
  const SelectArgs sa = sel ? *sel : SelectArgs{};
  PPOrder order;
  order.n_hgroups = n_hgroups;
  order.n_ttiles = n_ttiles;
  order.gph = g / hpw;
  order.n_sel = n_sel;
  // (equal lengths take the spread order only when told to, and the order lists MAX_HEAD_BUDGETS heads)
  order.spread = (hl.ragged && Dm.tune.pp_spread != 0) || (Dm.tune.pp_spread == 1 && Dm.h_kv <= MAX_HEAD_BUDGETS);
  order.heads = longest_first(hl, Dm.h_kv);
  const PPCut cut = plan_cut(Dm, order, hl, T, n_c, TW, split_part ? split_floats : 0);
  const bool parted = cut.n_donors > 0;
  const unsigned n_wg = (unsigned)(n_sel + cut.n_items + (parted ? cut.n_slots - cut.n_donors : 0));
#define LOCRET_PP_LAUNCH(SP)                                                                                          \
  do {                                                                                                                 \
    if (Dm.d == 64) LOCRET_PP_LAUNCH_D(64, SP);                                                                         \
    else if (Dm.d == 96) LOCRET_PP_LAUNCH_D(96, SP);                                                                    \
    else LOCRET_PP_LAUNCH_D(128, SP);                                                                                   \
  } while (0)
#define LOCRET_PP_LAUNCH_D(DD, SP)                                                                                    \
  hipExtLaunchKernelGGL((attn_pp_kernel<DD, SP>), dim3(n_wg), dim3(NW * 64), 0, st, tm.start,                          \
                        parted ? nullptr : tm.stop, 0, (const bf16_t*)q, tab, (const bf16_t*)Kx, (const bf16_t*)V,      \
                        (bf16_t*)out, T, Dm.h, g, Dm.cap, n_c, c_log2, hpw, order, sa, n_sel, hl, cut, split_part)
  if (parted || order.spread || hl.ragged) LOCRET_PP_LAUNCH(true); else LOCRET_PP_LAUNCH(false);
#undef LOCRET_PP_LAUNCH
#undef LOCRET_PP_LAUNCH_D
  if (parted) {
    const dim3 grid((unsigned)cut.n_donors, (unsigned)(Dm.d / 32));
#define LOCRET_PP_MERGE(DD)                                                                                            \
  hipExtLaunchKernelGGL(attn_pp_merge_kernel<DD>, grid, dim3(NW * 64), 0, st, nullptr, tm.stop, 0, (const float*)split_part,   \
                        (bf16_t*)out, T, Dm.h, g, n_c, hpw, order, hl, cut)
    if (Dm.d == 64) LOCRET_PP_MERGE(64);
    else if (Dm.d == 96) LOCRET_PP_MERGE(96);
    else LOCRET_PP_MERGE(128);
#undef LOCRET_PP_MERGE
  }
  return true;
}

}  // namespace locret
