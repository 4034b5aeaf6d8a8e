// Rules by which launches are shaped, as plain functions of sizes (host code without HIP: tests compile them on their own).
#pragma once
#include <stdint.h>

namespace locret {

constexpr int RULE_CUS = 256;

// ---- decode step: keys per split -------------------------------------------------------------------------------------
// All workgroups of a launch run at once, so what counts is the CU with the most work: it has the keys of
// ceil(workgroups / 256) splits and their fixed share (query, first wait, merge: about what 64 keys cost).  One workgroup over a
// multiple of 256 costs most: 8 heads x 16.4K units x 128 dims take 15.9 us at 256 keys (520 workgroups), 14.1 at 192 (696), 14.0
// at 320 (424); 8 x 6.1K 7.5 us at 256 (200), 8.8 at 192 (264), 8.3 at 128 (392); 4 x 16.4K 8.8 us at 320 (212), 10.4 at 256 (260).
// Splits longer than 320 keys only as far as some 700 workgroups are left: on much data a workgroup or two a CU have too few
// loads in flight (32 x 8.2K x 96 dims: 16.7 us at 384 keys, 736 workgroups, 19.6 at 1056 keys, 256).
// float32 rows: some 700 workgroups of at least 128 keys.  A workgroup has half as many rows in flight and takes the longer for
// them, so two short ones on a CU cost less than a long one.  A token, caches from HBM, by this and by the search: 8 heads x 4.1K x
// 128 dims 20.4, 22.8 us, 8.2K 24.7, 34.1; 32 x 2K x 128 21.1, 24.6; 8 x 8.2K x 64 13.9, 15.1.  (bf16 rows of 16 dims, the same
// kernel: 8 heads x 8.2K 12.2, 10.3.)
constexpr int DEC_KEYS_MIN = 128, DEC_KEYS_SHORT = 320, DEC_KEYS_SHARE = 64, DEC_KEYS_MAX = 65536;
inline int decode_split_keys(bool bf16, int h_kv, int n_keys) {
  int64_t want = (((int64_t)h_kv * n_keys + 703) / 704 + 63) / 64 * 64;
  if (want > DEC_KEYS_MAX) want = DEC_KEYS_MAX;        // (both ends of the search below follow it)
  if (!bf16) return (int)(want < DEC_KEYS_MIN ? DEC_KEYS_MIN : want);
  const int64_t most = want < DEC_KEYS_SHORT ? DEC_KEYS_SHORT : want;
  int64_t best = DEC_KEYS_MIN, best_cost = INT64_MAX;
  for (int64_t k = DEC_KEYS_MIN > want / 2 ? DEC_KEYS_MIN : want / 128 * 64; k <= most; k += 64) {
    const int64_t wgs = (int64_t)h_kv * ((n_keys + k - 1) / k + 1), cost = (wgs + RULE_CUS - 1) / RULE_CUS * (k + DEC_KEYS_SHARE);
    if (cost < best_cost) { best_cost = cost; best = k; }
  }
  return (int)best;
}

// ---- retaining head, float32: hidden units of a workgroup ------------------------------------------------------------------
// 32 while that leaves at most one workgroup (of 16 tokens) a CU, else 64, which reads the tokens half as often.  `room`: floats
// that the partial scores may take.  locret_score on 768 inputs x 256 hidden units, 64 against 32 units: 512 tokens 12.6, 9.4 us, 611
// tokens (312 workgroups of 32) 12.5, 13.2, 900 12.7, 13.2; 1536 inputs: 512 19.2, 13.2, 611 19.5, 22.0; 6144 inputs x 1024: 100 tokens 64.1,
// 39.6, 200 64.2, 73.1.
inline int f32_hidden_units(int T, int h_kv, int d_R, int64_t room) {
  const int64_t wgs = (int64_t)((T + 15) / 16) * ((d_R + 31) / 32), partials = (int64_t)((d_R + 31) / 32) * h_kv * T;
  return wgs <= RULE_CUS && partials <= room ? 32 : 64;
}

}  // namespace locret
