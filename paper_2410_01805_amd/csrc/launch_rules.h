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

// ---- retaining head, bf16: tiles, slices of the contraction, order of the workgroups -------------------------------------------
// mt hidden units x nt tokens a workgroup, n_z slices of the contraction (1: none; the finish kernel sums more).  A launch without
// slices leaves d_R / mt partial scores.
struct ScorePlan {
  int mt, nt, n_z;
  bool hidden_first;      // neighbouring workgroups take the same tokens and the next hidden units (false: the other way round)
};

constexpr int SCORE_STAGE = 64;       // contraction elements of a stage of the kernel

// Slices: as many as give every CU a workgroup, of 8 stages at least, none of them empty.  zpart_floats: room for
// the partial pre-activations, 0: no slices.  forced (Tuning::score_split): -1 this rule, 0 never, k always k.
inline int score_slices(int64_t tiles, int stages, int T, int d_R, int64_t zpart_floats, int forced) {
  if (zpart_floats == 0) return 1;
  int64_t n = forced >= 0 ? forced : RULE_CUS / tiles >= 2 ? RULE_CUS / tiles : 1;
  if (n > 8) n = 8;
  auto last_empty = [&](int64_t k) { return (k - 1) * ((stages + k - 1) / k) >= stages; };      // slices are ceil(stages / k) long
  while (n > 1 && (n * T * d_R > zpart_floats || (forced < 0 && stages / n < 8) || last_empty(n))) --n;
  return n < 1 ? 1 : (int)n;
}

// Every XCD has an L2 of its own and takes every eighth workgroup.  Of slow x fast tiles (neighbouring workgroups differ in `fast`)
// those of one XCD need about this much of one stage; w_slow, w_fast: a row's and a column's share of it.
inline double score_xcd_load(int64_t slow, int64_t fast, double w_slow, double w_fast) {
  const double n = slow * fast / 8. > 1 ? slow * fast / 8. : 1;              // its workgroups
  const double f = (double)(fast / (fast % 8 == 0 ? 8 : fast % 4 == 0 ? 4 : fast % 2 == 0 ? 2 : 1));
  return (f < n ? f : n) * w_fast + (slow < n ? slow : n) * w_slow;
}

// About what a launch with these tiles costs, in us, a mean over what callers meet (inputs in the last-level cache and in HBM, locret_score
// and steps whose selection sums the partials beside the attention): the longer of a workgroup's chain of stages and of
// what the L2s have to fetch (MB), then the finish kernel (8 KV heads a workgroup, whole eights by a faster path) or the sum.
inline double score_cost(const ScorePlan& p, double xcd_load, int stages, int h_kv) {
  const double chain = (p.mt == 128 ? 0.38 : 0.212) * ((stages + p.n_z - 1) / p.n_z), fetch = xcd_load * 8 * stages / 1024 / 7.7;
  const double finish = p.n_z == 1 ? 1.9 : (h_kv % 8 == 0 ? 5.5 : 10.5) + 4.8 * ((h_kv + 7) / 8 - 1) + 0.45 * p.n_z;
  return (chain > fetch ? chain : fetch) + finish;
}

// Token tile: 64 when 128-token tiles would leave at least half of the CUs without one (2048 tokens at d_R = 1024).
// 32q/8kv x 128, d_R = 1024 (hot caches): chunks of 2048 tokens 42.4 us with 128-token tiles, 37.3 with 64-token tiles, 49.6 with those
// and two slices; chunks of 3072 or 4096 tokens are a third slower with 64-token tiles (more LDS traffic per MFMA).
//
// Order, for 64 x 64 tiles: the one by which an XCD needs fewer different tiles.  Tokens first against hidden units first,
// 32q/8kv x 128, d_R = 512, 900 tokens (15 x 8 tiles) 27.4 / 27.4, 21.8 / 22.9 us (inputs in the last-level cache / from HBM), 1024 tokens
// (16 x 8) 19.8 / 22.5, 23.0 / 23.4.
//
// Hidden tile: 128, or 64 where 64 x 64 tiles are at most one a CU and their partials fit: then there are twice as many workgroups
// for half as many slices.  locret_score with 128 x 64 tiles against 64 x 64, 32q/8kv x 128, d_R = 1024: 300 tokens 21.9 / 21.6, 15.3 /
// 16.9 us, 900 35.5 / 35.9, 25.7 / 32.6; 32q/32kv x 96: 900 65.7 / 66.5, 39.1 / 47.8; 16q/4kv x 128, d_R = 512: 2048 25.1 / 25.7, 15.9 / 19.2.
// But a slice also gets longer by that, a chain of stages that may take more than the finish kernel saved, and 64-unit tiles ask
// the L2s for more: d_R = 512: 1100 tokens (3 slices, 1) 24.2 / 25.0, 23.9 / 32.3, 1300 (3, 1) 26.4 / 27.1, 24.9 / 33.4; d_R = 384: 900 (4, 2)
// 19.9 / 21.2, 21.7 / 22.4.  So both are estimated.  Over 450 launches (16 layouts, d_R 128 .. 2048, 64 .. 4096 tokens) the choice takes
// 0.86 (last-level cache) and 0.92 (HBM) of the time of 128 x 64 tiles, 0.2 % more than the better form of each would in the mean.  It is the
// slower one for locret_score from HBM where the slices of 64 x 64 tiles are long: d_R = 1024, 611 tokens (3, 1) 27.1 / 27.0, 23.9 / 31.9; in a
// prompt, where the append or the attention has read the inputs before, that launch is the faster one (a 611-token prompt and
// 8 scored tokens 126.7, 121.4 us).
// (Tuning::score_nt: 0 = these rules, 64 / 128 = tokens of a workgroup, with 128 hidden units.)
inline ScorePlan plan_score(int T, int h_kv, int K, int d_R, int64_t zpart_floats, int64_t fine_floats, int tune_nt, int tune_split) {
  const int stages = K / SCORE_STAGE;
  const int64_t tiles128 = ((int64_t)T + 127) / 128 * (d_R / 128), t64 = ((int64_t)T + 63) / 64, h64 = d_R / 64, h128 = d_R / 128;
  const int nt = tune_nt == 64 || tune_nt == 128 ? tune_nt : tiles128 <= RULE_CUS / 2 ? 64 : 128;
  const ScorePlan wide = {128, nt, score_slices(((int64_t)T + nt - 1) / nt * h128, stages, T, d_R, zpart_floats, tune_split), false};
  if (nt != 64 || tune_nt != 0 || tune_split >= 0 || t64 * h64 > RULE_CUS || h64 * h_kv * T > fine_floats) return wide;
  const double tokens_first = score_xcd_load(h64, t64, 8, 8), hidden_first = score_xcd_load(t64, h64, 8, 8);      // KB
  const ScorePlan fine = {64, 64, score_slices(t64 * h64, stages, T, d_R, zpart_floats, -1), hidden_first < tokens_first};
  const double wide_us = score_cost(wide, score_xcd_load(h128, t64, 16, 8), stages, h_kv) - (wide.n_z == 1 && h128 == 1 ? 3 : 0);   // (a single partial is the score)
  return score_cost(fine, fine.hidden_first ? hidden_first : tokens_first, stages, h_kv) <= wide_us ? fine : wide;
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
