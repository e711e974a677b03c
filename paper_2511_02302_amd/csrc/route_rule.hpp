// How many launches a routing takes, by its sizes: host code only.
#pragma once

#include "ff8_launch.hpp"

namespace ff8 {

// By what a chunk's workgroup would have to sum by itself.  Times: us with the permute of 128 columns
// behind them, one / two / three launches.
//  * All the pairs, up to 4096: one (7 tokens x 6: 10.7 / 12.6 / 13.9; 1024 x 2: 9.2 / 10.5 / 13.1;
//    1024 x 8: 16.8 / 15.1 / 17.7).
//  * All the counts, up to 8192: two (16384 tokens, 64 experts: 25.3 with two, 28.8 with three; 256
//    experts, 16384 counts: 36.1 / 34.1).
//  * Up to 32768 counts above 512 experts, where one workgroup's threads each mark the padding rows of
//    an expert, one by one, in the separate scan: two where those are many, that is with 128-row
//    padding (8192 tokens, 1024 experts: 50 / 94, all tokens to one expert 48 / 31), but three with
//    16-row padding (48 / 35).
inline int route_launches(int64_t T, int k, int E, int align) {
  const int64_t counts = (T + kRouteChunk - 1) / kRouteChunk * E;
  if (T * k <= 4096) return 1;
  return counts <= 8192 || (E > 512 && align >= 128 && counts <= 32768) ? 2 : 3;
}

}  // namespace ff8
