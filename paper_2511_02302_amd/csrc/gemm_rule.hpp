// Which tiles a grouped product takes, by its sizes: host code only.
#pragma once

#include "gemm_shared.hpp"

namespace ff8 {

// Workgroups of the small tiles' kernel that one CU runs at once, of the per_cu that registers allow:
// the tables of the experts' offsets take LDS, and above 360 experts only two of the three with TQ 64
// fit.  Groups sized for three there leave a third of each waiting for a CU (16 rows, 512 x 1024: 512
// experts, fprop 74 us, sized for two 71; 1024 experts 171 / 161).
constexpr int kLdsPerCU = 160 * 1024;
inline int small_per_cu(int per_cu, int lds) { return lds * per_cu <= kLdsPerCU ? per_cu : kLdsPerCU / lds; }

// wgrad on the small tiles: 256 (K) x 128 (N) ones, or 128 x 128.  Two of either run on a CU.  Where at
// most two of the first come to a CU, all run at once and need no second round as twice as many of the
// others do, which pays from about four K stages on (us, 128 x 128 / 256 x 128: two per CU, 4 experts of
// 2048 x 2048, 512 tokens 28 / 23, 768 33 / 27, 16 of 1024 x 1024 30 / 24, 35 / 28; 1.5 per CU, 8 experts of
// 768 x 2048, 512 tokens 20 / 21, 12 of 512 x 2048, 1024 tokens 29 / 28).  A part of a second round costs
// them a whole one (9 experts of 1024 x 2048, 2.25 per CU, 512 tokens 27 / 30; 10 of them, 2.5 per CU, 256
// tokens 23 / 25); from three per CU on they move a quarter less (12 of 1024 x 2048, 512 tokens 37 / 33;
// 15: 46 / 40; 16 of 2048 x 2048, 640 tokens 82 / 69; 32 of 4096 x 7168, 512 tokens 1024 / 920).
inline int64_t wgrad_tiles256(int E, int64_t N, int64_t K) { return E * (N / 128) * ((K + 255) / 256); }
inline bool wgrad_wide(int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  const int64_t n = wgrad_tiles256(E, N, K);
  return n >= 3 * cus || (n > cus && n <= 2 * cus && M_cap >= (4 * n >= 7 * cus ? 512 : 640) * (int64_t)E);
}
// wgrad on the small tiles or on 256 x 256 ones: six K stages of 128 tokens do not hide a 256 KB output
// tile, eight nearly do.  M_cap / E is the tokens per expert.  Times: us, 256 x 256 / small tiles.
//  * At most one 256 x 128 tile per CU: the small ones, whose products spread over twice the CUs (8
//    experts of 640 x 1024, 256 tokens 20 / 11, 4096 60 / 44).
//  * Below four per CU, up to 1024 tokens: the small ones (5 experts of 2048 x 1024, 1024 tokens 29 /
//    26, 2048 40 / 38, 4096 61 / 64; 15 of 1024 x 2048, 1024 tokens 53 / 53).
//  * Above, up to 1024 tokens, the cheaper by two lines in the K stages, us: 12.9 + 1.33 per stage for
//    a round of the CUs with the large tiles, which take whole rounds, and for 512 of the 256 x 128
//    ones 11.5 + 1.6, or 9.4 + 1.57 for outputs of at least 3584 columns.  7168 x 2048, 32 experts:
//    384 tokens 467 / 436, 512 509 / 512, 640 550 / 569, 768 583 / 613; 64 of 2816 x 2048: 384 383 /
//    344, 512 413 / 399, 768 471 / 477, 766 on average 474 / 510; 16 of 2816 x 2048 (5.5 rounds): 512 116 /
//    106, 768 131 / 122; 64 of 2048 x 1408: 768 262 / 246; 32 of 4096 x 7168: 512 1059 / 872, 768 1212 /
//    1050, 1024 1358 / 1226; of 7168 x 4096: 640 1165 / 959, 896 1329 / 1134.  Above 1024 tokens the
//    gain under even routing (1280 tokens, 4096 x 7168: 1509 / 1405) is a loss under skewed
//    (1443 / 1483).
inline bool wgrad_small(int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  const int64_t n = wgrad_tiles256(E, N, K);
  if (n <= cus) return true;
  if (M_cap > 1024 * (int64_t)E) return false;
  if (n < 4 * cus) return true;
  const int64_t rows = M_cap / E;  // 128 per stage; hundredths of a microsecond below
  const int64_t large = ((N + 255) / 256) * ((K + 255) / 256) * E;
  const int64_t t_large = (large + cus - 1) / cus * (1290 + 133 * rows / 128) + 600;
  const int64_t per_round = K >= 3584 ? 940 + 157 * rows / 128 : 1150 + 160 * rows / 128;
  return E * (N / 128) * (K / 128) * per_round / (4 * cus) + 540 < t_large;  // K / 128 / 2 tiles, half ones as halves
}

// The tq of the small tiles (64 or 128; wgrad: 128), or 0 for the 256 x 256 tiles; cus: compute
// units of the device.  M_cap / E bounds the mean rows of a group from above (it counts the
// padding), the rest is known exactly.  Times below: us, 256 x 256 tiles / these tiles, on normally
// distributed operands (random bytes draw more power, which slows the large tiles most) that no
// cache holds.
//  * fprop, dgrad, up to 96 rows per group, so one tile of rows per expert: both kernels stream the
//    weights, the large tiles in whole rounds of one tile per CU (1.45 us per K stage, 3.5 us per
//    round and 4.5 us once), these at 5.6 MB/us (fprop) or 4.75 (dgrad, whose loads are 128-byte
//    runs of the weight's rows) with TQ 64 and 4.7 or 4.25 with TQ 128, which groups above 64 rows
//    need.  The cheaper of the two: 16 rows, 32 experts of 4096 x 7168: fprop 174 / 166, dgrad 205 /
//    205; 8 of them: 74 / 47, 53 / 59; 32 of 7168 x 2048: 106 / 90, 95 / 101; 64 of 2816 x 2048: 85 / 75,
//    77 / 86; of 2048 x 1408: 46 / 40, 56 / 40; 64 rows: 183 / 175, 213 / 214; 79 / 49, 56 / 59; 109 /
//    94, 95 / 104; 87 / 79, 79 / 88; 48 / 42, 58 / 42.  With tokens for a few of the experts only, the
//    small ones do less where a large tile's K loop is as long (28 of 4096 x 2048, 58 tokens, dgrad 43 /
//    26); where a few experts hold most tokens, they read those weights once per 64 rows (32 of 4096 x
//    7168, 256 tokens x 4, Zipf(1.2): 97 / 107, 104 / 125).
//  * fprop, dgrad on grids of at most three 256 x 256 tiles per CU, where whole rounds of such
//    tiles leave CUs idle: the same model of the large tiles against 1.42 us (dgrad 1.55) per stage
//    of a round of 512 small ones.  16 experts of 2048 x 2048, fprop: 192 rows 37 / 31, 256 40 / 32, 384
//    34 / 40; 8 of 4096 x 7168: 192 rows 96 / 84; dgrad: 192 rows 67 / 105.  The groups' last, partial
//    tiles are an eighth of one per expert on average, but none where M_cap is whole tiles for every
//    expert, and then the share can be a round too many (512 rows each, fprop: 8 experts of 4096 x 7168
//    97 / 148, 16 of 2048 x 2048 39 / 52).  Experts share no tile, so up to 256 rows there are as many
//    as experts that have any; on that count the small ones, whose own is then low as well, have to
//    win by an eighth (dgrad a quarter): 64 experts of 2048 x 1408, dgrad of 128 rows 61 / 50; 49 of
//    1792 x 3456, 9 tokens, fprop 39 / 26; closer, 32 of 7168 x 2048, fprop of 128 rows on average 121 /
//    138, 30 of 1024 x 5120, one token x 7, dgrad 21 / 25.  TQ 64 when even 128 x 128 tiles do not reach
//    every CU, or reach it once for a few stages (8 experts of 1024 x 1024, 256 rows: 14.0 with TQ 128,
//    12.1 with 64).
//  * wgrad: see wgrad_small.
inline int small_gemm_tile(GemmMode mode, int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  if (mode == kWgrad) return wgrad_small(E, M_cap, N, K, cus) ? 128 : 0;
  const int64_t Np = mode == kFprop ? N : K, Kd = mode == kFprop ? K : N, nk = Kd / kBK;
  const bool f = mode == kFprop;
  const int64_t n_pt = (Np + 255) / 256;
  // hundredths of a microsecond for q tiles of 256 rows
  auto t_large = [&](int64_t q) { return (q * n_pt + cus - 1) / cus * (145 * nk + 350) + 450; };
  if (M_cap <= 96 * (int64_t)E) {
    const int tq = M_cap <= 64 * (int64_t)E ? 64 : 128;
    const int64_t rate = tq == 64 ? (f ? 56000 : 47500) : (f ? 47000 : 42500);  // bytes per 0.01 us
    return E * Np * Kd / rate + 200 < t_large(E) ? tq : 0;
  }
  const int64_t q_tiles = M_cap / 256 + (E + 7) / 8;
  const int64_t small = (M_cap / 128 + (E + 7) / 8) * (Np / 128);
  const int64_t t_small = small * (f ? 142 : 155) * nk / (2 * cus) + 700;
  const bool whole = M_cap % (256 * (int64_t)E) == 0;
  const bool wins = t_small < t_large(q_tiles) && !(whole && t_small >= t_large(M_cap / 256));
  const bool wins_by_experts = q_tiles < E && t_small + t_small / (f ? 8 : 4) < t_large(E);
  if (q_tiles * n_pt > 3 * cus || !(wins || wins_by_experts)) return 0;
  return small < cus || (small < 2 * cus && nk <= 8) ? 64 : 128;
}

}  // namespace ff8
