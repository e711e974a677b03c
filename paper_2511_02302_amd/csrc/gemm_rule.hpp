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

// 256 (K) x 128 (N) tiles of wgrad's output.
inline int64_t wgrad_tiles256(int E, int64_t N, int64_t K) { return E * (N / 128) * ((K + 255) / 256); }

// The small tiles of wgrad are 256 x 128, a quarter less DMA per product, from four of them per CU on (us,
// 128 x 128 / 256 x 128: 16 experts of 2048 x 2048, 640 tokens 82 / 69; 32 of 4096 x 7168, 512 tokens
// 1024 / 920).  Below, 128 x 128 ones: which are faster there depends on the routing, which is not known
// here, and under skewed routing they are by far (even: 15 experts of 1024 x 2048, 768 tokens 56 / 46, 16
// of 1024 x 1024, 512 tokens 30 / 24; Zipf(1.2): 31 of 1024 x 1024, 523 tokens 63 / 78, 21 of 1024 x 512,
// 519 tokens 29 / 40, 43 of 2816 x 256, 488 tokens 93 / 148).
inline bool wgrad_wide(int E, int64_t N, int64_t K, int64_t cus) { return wgrad_tiles256(E, N, K) >= 4 * cus; }

// wgrad on the small tiles or on 256 x 256 ones.  M_cap / E bounds the tokens per expert (its K) from
// above.  Times: us, 256 x 256 / small tiles.
//  * Where 256 x 256 tiles fill less than 5/8 of the CUs: the small ones (8 experts of 1024 x 256, 640
//    tokens 19 / 9; 18 of 2048 x 128, 1026 tokens, Zipf(1.2), 40 / 26; only even routing and very long K
//    turn that round: 6 of 1024 x 1536, 5522 tokens 69 / 90, but 3204 tokens, Zipf(1.2), 77 / 60).
//  * Otherwise up to 832 tokens: six K stages of 128 do not hide a 256 KB output tile (32 experts of 4096
//    x 7168: 512 tokens 1059 / 872, 768 1212 / 1050; of 7168 x 4096: 640 1165 / 959; 64 of 2816 x 2048:
//    384 383 / 344, 512 413 / 399, 768 471 / 477; 16 of 2816 x 2048: 768 131 / 122).  Above, the small
//    ones still gain under even routing (896 tokens, 4096 x 7168: 1286 / 1137), but lose under skewed (11
//    experts of 3072 x 5632, 874 tokens, Zipf(1.2) 273 / 326).
//  * But for outputs of up to 3072 columns and at least 128 of the large tiles per expert, whose small
//    tiles take longer, the cheaper by two lines in the K stages, us: 12.9 + 1.33 per stage for a round of
//    the CUs with the large tiles, which take whole rounds, and 11.5 + 1.6 for 512 of the 256 x 128 ones.
//    32 experts of 7168 x 2048: 384 tokens 467 / 436, 512 509 / 512, 640 550 / 569, 768 583 / 613, 625 on
//    average 561 / 610, 800 on average, Zipf(1.2) 617 / 653; of 4096 x 2560: 384 356 / 323, 640 414 / 407.
inline bool wgrad_small(int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  const int64_t per_expert = ((N + 255) / 256) * ((K + 255) / 256), large = E * per_expert;
  if (8 * large <= 5 * cus) return true;
  if (M_cap > 832 * (int64_t)E) return false;
  if (K >= 3584 || per_expert < 128 || wgrad_tiles256(E, N, K) < 4 * cus) return true;
  const int64_t rows = M_cap / E;  // 128 per stage; hundredths of a microsecond below
  const int64_t t_large = (large + cus - 1) / cus * (1290 + 133 * rows / 128) + 600;
  return wgrad_tiles256(E, N, K) * (1150 + 160 * rows / 128) / (2 * cus) + 540 < t_large;
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
//    tiles count as an eighth of one per expert, which fits random routings (63 experts of 1024 x 1024,
//    236 rows on average, fprop 47 / 38; exactly even groups of whole tiles have none and can get the
//    slower: 8 experts of 4096 x 7168, 512 rows each, fprop 97 / 148).  Experts share no tile, so up to
//    256 rows there are as many as experts that have any; on that count the small ones, whose own is
//    then low as well, have to win by a quarter: 64 experts of 2048 x 1408, dgrad of 128 rows 61 / 50; 49
//    of 1792 x 3456, 9 tokens, fprop 39 / 26; closer, 32 of 7168 x 2048, fprop of 128 rows on average
//    121 / 138, 30 of 1024 x 5120, one token x 7, dgrad 21 / 25.  TQ 64 when even 128 x 128 tiles do not
//    reach every CU, or reach it once for a few stages (8 experts of 1024 x 1024, 256 rows: 14.0 with TQ
//    128, 12.1 with 64).
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
  const bool wins_by_experts = q_tiles < E && t_small + t_small / 4 < t_large(E);
  if (q_tiles * n_pt > 3 * cus || !(t_small < t_large(q_tiles) || wins_by_experts)) return 0;
  return small < cus || (small < 2 * cus && nk <= 8) ? 64 : 128;
}

}  // namespace ff8
