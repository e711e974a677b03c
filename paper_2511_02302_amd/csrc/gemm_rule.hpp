// Which tiles a grouped product takes, by its sizes: host code only.
#pragma once

#include "gemm_shared.hpp"

namespace ff8 {

// The tq of the small tiles (64 or 128; wgrad: 128), or 0 for the 256 x 256 tiles; cus: compute
// units of the device.  M_cap / E bounds the mean rows of a group from above (it counts the
// padding), the rest is known exactly.  Times below: us, 256 x 256 tiles / these tiles, on normally
// distributed operands (random bytes draw more power, which slows the large tiles most) that no
// cache holds.
//  * fprop, dgrad, up to 96 rows per group, so one tile of rows per expert: both kernels stream the
//    weights, the large tiles in whole rounds of one tile per CU (1.45 us per K stage, 3.5 us per
//    round and 4.5 us once), these at 5.6 MB/us (fprop) or 4.75 (dgrad, whose loads are 128-byte
//    runs of the weight's rows) with TQ 64 and 4.7 or 4.25 with TQ 128, which groups above 64 rows
//    need.  The cheaper of the two, for dgrad by a sixteenth (where they come closer the small tiles
//    gain nothing, and a skewed routing costs them more: 32 experts of 4096 x 7168, 256 tokens x 4,
//    Zipf(1.2): 104 / 125): 16 rows, 32 experts of 4096 x 7168: fprop 174 / 166, dgrad 205 / 205; 8 of
//    them: 74 / 47, 53 / 59; 32 of 7168 x 2048: 106 / 90, 95 / 101; 64 of 2816 x 2048: 85 / 75, 77 / 86;
//    of 2048 x 1408: 46 / 40, 56 / 40; 64 rows: 183 / 175, 213 / 214; 79 / 49, 56 / 59; 109 / 94, 95 /
//    104; 87 / 79, 79 / 88; 48 / 42, 58 / 42.
//  * fprop, dgrad on grids of at most three 256 x 256 tiles per CU, where whole rounds of such
//    tiles leave CUs idle: the same model of the large tiles against 1.42 us (dgrad 1.55) per stage
//    of a round of 512 small ones.  How many tiles the groups' last, partial ones add is not known
//    here: none if the groups are whole tiles, so the small ones have to win on that count too (it
//    can be a whole round: 8 experts of 4096 x 7168, fprop of 512 rows: 97 / 148; 16 of 2048 x 2048:
//    39 / 52).  16 experts of 2048 x 2048, fprop: 192 rows 37 / 31, 256 40 / 32, 384 34 / 40; 8
//    of 4096 x 7168: 192 rows 96 / 84; dgrad: 192 rows 67 / 105.  TQ 64 when even 128 x 128 tiles do not
//    reach every CU, or reach it once for a few stages (8 experts of 1024 x 1024, 256 rows: 14.0 with
//    TQ 128, 12.1 with 64).
//  * wgrad up to 832 tokens per expert (its K): six K stages do not hide a 256 KB output tile.
//    32 experts of 4096 x 7168: 128 tokens 727 / 682, 256 795 / 686, 512 1112 / 920, 768 1287 /
//    1166, 1024 1437 / 1364; 7168 x 2048: 512 538 / 505, 768 614 / 617, 1024 685 / 737; also where
//    256 x 256 tiles fill less than 5/8 of the CUs (8 experts of 1024 x 256, 640 tokens: 19.2 / 8.5).
inline int small_gemm_tile(GemmMode mode, int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  if (mode == kWgrad) {
    const int64_t tiles = E * ((N + 255) / 256) * ((K + 255) / 256);  // 256 x 256
    return M_cap <= 832 * (int64_t)E || 8 * tiles <= 5 * cus ? 128 : 0;
  }
  const int64_t Np = mode == kFprop ? N : K, Kd = mode == kFprop ? K : N, nk = Kd / kBK;
  const bool f = mode == kFprop;
  // hundredths of a microsecond for n tiles of 256 x 256
  auto t_large = [&](int64_t n) { return (n + cus - 1) / cus * (145 * nk + 350) + 450; };
  if (M_cap <= 96 * (int64_t)E) {
    const int tq = M_cap <= 64 * (int64_t)E ? 64 : 128;
    const int64_t rate = tq == 64 ? (f ? 56000 : 47500) : (f ? 47000 : 42500);  // bytes per 0.01 us
    const int64_t small = E * Np * Kd / rate + 200, large = t_large(E * ((Np + 255) / 256));
    return (f ? small : small + small / 16) < large ? tq : 0;
  }
  // q tiles: the rows' own, and a share of one per expert for the groups' last, partial tiles
  const int64_t q_large = (M_cap + 255) / 256, n_pt = (Np + 255) / 256;
  const int64_t large = (M_cap / 256 + (E + 7) / 8) * n_pt;
  const int64_t small = (M_cap / 128 + (E + 7) / 8) * (Np / 128);
  const int64_t t_small = small * (f ? 142 : 155) * nk / (2 * cus) + 700;
  if (large > 3 * cus || t_small >= t_large(large) || t_small >= t_large(q_large * n_pt)) return 0;
  return small < cus || (small < 2 * cus && nk <= 8) ? 64 : 128;
}

}  // namespace ff8
