// Stabilizer-masked top-k per KV head (Section 3.4; Algorithm 1: "+inf on the last n_s, top-b"),
// with an optional pinned prefix (the first n_pin units are kept as well: Locret-Q keeps the query,
// placed at the start of the sequence, visible to every eviction).
//
// One 1024-thread workgroup per KV head.  Scores become order-preserving 32-bit keys (NaN lowest,
// -0 == +0); a radix select finds the key tau of the k-th best candidate and how many units equal to
// tau still fit; a ballot-based ordered compaction then emits the kept indices ascending, taking equal
// keys from the lowest index up.  Integer work only, so the result is exact and deterministic.
//
// The keys are held in registers (select_reg_kernel): wavefront w owns a contiguous index range,
// lane-interleaved in rounds of 64, so every global read is a 256-byte line, the radix passes touch LDS
// only for the histogram, and the final ordered compaction is ballots over registers.  16 wavefronts
// on one CU have 128 registers each, which is 36 keys a thread (36864 candidates per head); 48 or 64 keys do not fit
// beside the rest and spill to scratch memory.  What is beyond 36 keys is read again by every pass, in groups of 8 loads.
// A step of 4096 tokens with eviction alone, 64-dim heads, in this form, with 48 or 64 spilling keys, with all keys
// read again: 8 heads x 40960 candidates 84, 86, 115 us; 8 x 65536 132, 131, 177 us; 1 x 49152 54, 48, 89 us.
// (Up to 36864 candidates: 48000 tokens into 8 budgets of 32768 units take 760 us where more than 24576 are read
// again, 538 us with all of them in registers.)
#include "device_util.h"
#include "kernels.h"
#include "select_body.h"

namespace locret {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / 64;

// ------------------------------------------------------------------------------------------------
// MAXR keys per thread in registers, TAIL: more candidates than that (select_body.h).
template <int MAXR, bool TAIL>
__global__ __launch_bounds__(SEL_THREADS) void select_reg_kernel(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t smem[select_body_smem_words(SEL_THREADS, 2)];
  select_reg_body<MAXR, SEL_THREADS, 2, TAIL>(a, blockIdx.x, smem);
}

// One token a thread: the thread's chain of loads is then the one a thread of the reduction has, and its launch (4 us) is
// saved.  With a second token a thread it is lost again.  A step, selection in a launch of its own, summed there or
// reduced before it: float32, 2 heads, T = 512: 32 partials 88.0, 89.1 us, 128 partials 199.4, 202.1; T = 1024, 32 partials 144.8,
// 146.1; T = 1500, 4 partials 159.2, 156.8; T = 2048, 32 partials 306.7, 299.6.  bf16, 8 heads x 64, T = 1024, 32 partials
// 105.8, 107.0 us; T = 1500, 8 partials 96.3, 95.5; T = 3072, 8 partials 158.8, 155.8, 32 partials 240.0, 226.4.
bool select_sums_partials(int T) { return T <= SEL_THREADS; }

// The form is chosen for the longest head; every form takes shorter heads as they come.
void launch_select(const SelectArgs& a, int h_kv, hipStream_t st) {
  const int rounds = select_rounds(a, SEL_WAVES);
#define LOCRET_SEL_REG(R)                                                                         \
  if (rounds <= R) {                                                                              \
    launch_kernel((select_reg_kernel<R, false>), dim3(h_kv), dim3(SEL_THREADS), 0, st, a);                 \
    return;                                                                                       \
  }
  LOCRET_SEL_REG(12)
  LOCRET_SEL_REG(24)
  LOCRET_SEL_REG(36)
#undef LOCRET_SEL_REG
  launch_kernel((select_reg_kernel<36, true>), dim3(h_kv), dim3(SEL_THREADS), 0, st, a);
}

// Nothing is over its budget: every head's kept list is 0, 1, 2, ... (only a caller's copy wants it).
__global__ __launch_bounds__(256) void keep_all_kernel(int32_t* __restrict__ out, int stride, int L_common, HeadLens L_h) {
  const int m = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  if (i < head_len(L_h, m, L_common)) out[(int64_t)m * stride + i] = i;
}

void launch_keep_all(int32_t* out, int stride, int h_kv, int L, const HeadLens& L_h, hipStream_t st) {
  launch_kernel(keep_all_kernel, dim3((L + 255) / 256, h_kv), dim3(256), 0, st, out, stride, L, L_h);
}

}  // namespace locret
