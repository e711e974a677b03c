// Tile order of the 256 x 256 grouped GEMM (gemm.hip): which workgroup runs which tiles, and the
// grid that holds them all.  Integer code only, compiled for the host too, where the tests walk
// the order workgroup by workgroup.
#pragma once

#include "gemm_shared.hpp"

namespace ff8 {

constexpr int kTP = 256;   // p tile
constexpr int kTQ = 256;   // q tile
constexpr int kBQ = 8;     // q tiles per XCD block
constexpr int kBP = 4;     // p tiles per XCD block
constexpr int kPersistSlots = kBQ * kBP;  // workgroups per XCD and group
static_assert(kPersistSlots == 32, "an XCD block is the 32 workgroups one XCD runs at once");

// Semi-persistent: the grid is a sequence of groups of S workgroups per XCD (S = 32 on
// 256 CUs, one workgroup per CU), and each workgroup runs kRoundsPerWg tiles.  Workgroups
// are dispatched round-robin over the 8 XCDs, and in order within an XCD.  XCD x owns XCD
// blocks x, x + 8, x + 16, ... (kBQ x kBP tiles each, p fastest); its work list is their
// tiles in that order, item i = k S + s going to slot s of the group that owns round k.
// With S = 32, slot s takes tile s of every block, so the 32 workgroups of an XCD work on
// one block at a time and share its 8 q panels and 4 p panels per K step in their L2, while
// the 8 XCDs together sweep one 16 x 16-tile window (about one expert).  Bounding a
// workgroup to a few rounds keeps an XCD's workgroups from drifting apart (which costs L2
// sharing) and lets faster CUs take more groups.
// wgrad under skewed routing: every expert has the same tile count, so an expert's blocks
// rarely divide evenly over the 8 XCDs, and the largest experts' extra blocks pile up on a
// few of them.  When the largest expert has more than twice the mean rows (decided in every
// workgroup from the offsets, identically), each XCD instead takes one of 8 equal rectangles
// of every expert's tile grid (at least one round of 32 tiles each), which balances the XCDs
// exactly; with near-uniform routing the blocks, which share more operand panels per round,
// are kept.
constexpr int kRoundsPerWg = 4;           // work rounds (tiles) per workgroup

// A workgroup-uniform value in a scalar register.
__host__ __device__ __forceinline__ int uniform(int v) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}
// The same value, recomputed from here on by what uses it instead of being hoisted.
__host__ __device__ __forceinline__ int opaque_uniform(int v) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(v));
#endif
  return v;
}

// One tile of the grouped product: expert e, q rows [q0, q_end) of a 256-row tile, p
// columns from p0, contraction from k0 over nk stages.
struct TileInfo {
  int e, blk;
  int q0, q_end, k0, p0, nk;  // rows, columns and stages all stay below 2^31
  int k_lo, k_hi;             // wgrad: valid K bytes of the first / last stage
};

// wgrad: the K range of expert e's tiles.  K runs over whole 128-token blocks from the one
// holding offsets[e]; with groups padded to 16 the first and last may be shared with
// neighbouring experts (masked in their DMAs).
__host__ __device__ __forceinline__ void wgrad_k_range(const GemmArgs& g, int e, TileInfo& t) {
  const int o0 = uniform(g.offsets[e]);
  const int o1 = uniform(g.offsets[e + 1]);
  const int kb0 = o0 & ~(kBK - 1);
  t.k0 = kb0;
  t.nk = o1 > o0 ? (o1 - kb0 + kBK - 1) / kBK : 0;
  t.k_lo = o0 - kb0;
  t.k_hi = o1 > o0 ? o1 - (kb0 + (t.nk - 1) * kBK) : kBK;
}

// XCD blocks, or chunks of packed tiles, of a launch with n_qg q tiles.
__host__ __device__ __forceinline__ int order_blocks(int n_pt, int n_qg, bool packed) {
  return packed ? (n_qg * n_pt + kPersistSlots - 1) / kPersistSlots
                : ((n_pt + kBP - 1) / kBP) * ((n_qg + kBQ - 1) / kBQ);
}

// Whether packing saves a sweep over the XCDs, or half of one where the last can be split.  Where it
// does not, the blocks' tiles stay together and spread over more XCDs (us, packed / blocks: 16 experts
// of 450 rows, 1536 x 4096, fprop 60 / 56; 8 of 700 rows, 1408 x 2048, 37 / 34; wgrad of 8 experts of
// 1024 x 640, 1100 tokens 29 / 26; but under skewed routing wgrad's sweeps are as long as their longest
// tiles, and packing can spread those better: 8 of 2048 x 2560, 1100 tokens, Zipf(1.2) 89 / 122).  Over
// 539 products of odd widths packing gains 8% on average, by this rule 9%.
__host__ __device__ __forceinline__ bool packing_saves(int n_pt, int n_qg, bool split) {
  const int chunks = order_blocks(n_pt, n_qg, true), rest = chunks & 7;
  const int halves = 2 * (chunks >> 3) + (rest == 0 ? 0 : split && rest <= 4 ? 1 : 2);
  return halves < 2 * ((order_blocks(n_pt, n_qg, false) + 7) >> 3);
}

// Tile w_in of XCD block blk (kBQ x kBP tiles, p fastest).  False for tiles past the
// edges.  fprop/dgrad: q tiles are 256-row tiles of the expert groups (cum / off:
// cumulative tile counts and row offsets per expert, in LDS); n_qg: q tiles of the launch.
// kPack (p tiles not a multiple of kBP), packed: every third or so block would be cut by the p edge
// and leave its XCD a part of the work, so the blocks' tiles are packed into chunks of 32 in block
// order, and blk is a chunk; every chunk but the last is full.  64 experts of 1024 rows, 2048 x
// 1408 (6 p tiles): dgrad 236 -> 200 us, wgrad 371 -> 302.  With whole blocks only, the longer
// lookup between two tiles costs 1-2%, so those keep the short one.
template <int MODE, bool kPack>
__host__ __device__ __forceinline__ bool decode_tile(const GemmArgs& g, const int* cum, const int* off, int n_qg,
                                                     bool packed, int blk, int w_in, TileInfo& t) {
  int qg, pt;  // global q-tile index, p tile
  if (kPack && packed) {
    const int l = blk * kPersistSlots + w_in;
    if (l >= n_qg * g.n_pt) return false;
    const int row = l / (kBQ * g.n_pt), l_q = l - row * kBQ * g.n_pt;  // row of blocks
    const int nq = min(kBQ, n_qg - row * kBQ);
    const int pb = l_q / (kBP * nq), l_p = l_q - pb * kBP * nq;
    const int np = min(kBP, g.n_pt - pb * kBP);
    const int lq = l_p / np;
    qg = row * kBQ + lq;
    pt = pb * kBP + l_p - lq * np;
  } else {
    const int n_pb = (g.n_pt + kBP - 1) / kBP;
    const int qb = blk / n_pb, pb = blk - qb * n_pb;
    qg = qb * kBQ + w_in / kBP;
    pt = pb * kBP + w_in % kBP;
    if (pt >= g.n_pt) return false;
  }
  t.blk = blk;
  t.p0 = (int64_t)pt * kTP;
  if (MODE != kWgrad) {
    if (qg >= cum[g.E]) return false;
    int lo = 0, hi = g.E - 1;  // largest e with cum[e] <= qg
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cum[mid] <= qg) lo = mid; else hi = mid - 1;
    }
    const int e = uniform(lo);
    t.e = e;
    t.q0 = uniform(off[e] + (qg - cum[e]) * kTQ);  // uniform (LDS values)
    t.q_end = uniform(off[e + 1]);
    t.k0 = 0;
    t.nk = g.Kdim / kBK;
    t.k_lo = 0;
    t.k_hi = kBK;
  } else {
    if (qg >= g.E * g.n_qt) return false;
    const int e = qg / g.n_qt;
    t.e = e;
    t.q0 = (int64_t)(qg - e * g.n_qt) * kTQ;
    t.q_end = g.Nq;
    wgrad_k_range(g, e, t);
  }
  return true;
}

// A row-wise tile with at most 128 rows runs on half the q panel (Sched<2>) and stores rows
// [q0, q_end); the others store up to 256.
__host__ __device__ __forceinline__ bool half_tile(const TileInfo& t) { return t.q_end - t.q0 <= kTQ / 2; }

// wgrad, expert-share schedule: item i of XCD x is tile l = i % share of expert e = i / share
// in XCD x's rectangle (p fastest).  Every expert's tiles are split evenly over the 8 XCDs,
// so the XCDs' loads stay equal however skewed the routing is (with XCD blocks, an expert's
// block count is rarely a multiple of 8, and the largest experts' extra blocks pile up on a
// few XCDs).
__host__ __device__ __forceinline__ void decode_share_tile(const GemmArgs& g, int xcd, int i, TileInfo& t) {
  const int e = i / g.share, l = i - e * g.share;
  const int lq = l / g.rect_p, lp = l - lq * g.rect_p;
  const int rq = xcd / g.rect_b, rp = xcd - rq * g.rect_b;
  t.blk = 0;
  t.e = e;
  t.p0 = (rp * g.rect_p + lp) * kTP;
  t.q0 = (rq * g.rect_q + lq) * kTQ;
  t.q_end = g.Nq;
  wgrad_k_range(g, e, t);
}

// Next tile of this workgroup from round k on, below round k_end (k advances past empty
// edge tiles).  kPack: packed in wgrad (decided on the host), in fprop / dgrad by the entry behind
// cum's last (the groups are known on the device only).  There, where the last sweep over the XCDs
// has at most four chunks left, two XCDs take each, a half of every tile's rows (Sched<2>) each:
// fprop of 2816 x 2048, 64 experts, 4096 tokens x 6 (44 chunks) 183 -> 172 us; 16 experts, 2048
// tokens x 2 (11 or 12 chunks) 57 -> 53.
template <int MODE, bool kPack>
__host__ __device__ __forceinline__ bool next_tile(const GemmArgs& g, const int* cum, const int* off, int block_idx,
                                                   int n_blocks, bool use_share, int& k, TileInfo& t) {
  // fprop / dgrad: from the opaque block index, so that none of it stays in registers across the
  // K loop (dgrad spilled two; wgrad has room, and is 1% slower with this)
  const int bid = MODE != kWgrad ? opaque_uniform(block_idx) : block_idx;
  const int n_slots = g.n_slots, group_size = 8 * n_slots;
  const int group = bid / group_size, in_group = bid - group * group_size;
  const int xcd = in_group & 7, slot = in_group >> 3, k_end = (group + 1) * kRoundsPerWg;
  const int n_qg = !kPack ? 0 : MODE == kWgrad ? g.E * g.n_qt : uniform(cum[g.E]);
  const bool packed = kPack && (MODE == kWgrad || uniform(cum[g.E + 1]) != 0);
  for (; k < k_end; ++k) {
    const int i = k * n_slots + slot;
    if (MODE == kWgrad && use_share) {
      if (i >= g.E * g.share) return false;
      decode_share_tile(g, xcd, i, t);
      return true;
    }
    const int sweep = (i / kPersistSlots) * 8;
    if (packed && MODE != kWgrad && sweep == (n_blocks & ~7) && (n_blocks & 7) <= 4) {
      if (xcd >= 2 * (n_blocks & 7)) return false;
      if (!decode_tile<MODE, kPack>(g, cum, off, n_qg, packed, sweep + (xcd >> 1), i % kPersistSlots, t)) continue;
      // q_end is the group's end, not the tile's: the odd half ends with the tile
      t.q0 += (xcd & 1) * (kTQ / 2);
      t.q_end = min(t.q_end, t.q0 + kTQ / 2);
      if (t.q0 < t.q_end) return true;
      continue;
    }
    const int blk = sweep + xcd;
    if (blk >= n_blocks) return false;
    if (decode_tile<MODE, kPack>(g, cum, off, n_qg, packed, blk, i % kPersistSlots, t)) return true;
  }
  return false;
}

// Grid: groups of n_slots workgroups per XCD (one per CU, the same number on each of the
// 8 XCDs, at most kPersistSlots), enough groups of kRoundsPerWg rounds for `items` tiles per
// XCD, or for n_blocks_max XCD blocks (workgroups past the work actually present exit at once).
inline unsigned grid_items(int64_t items, int cus, int& n_slots) {  // items: work items (tiles) per XCD
  cus = (cus / 8) * 8;
  if (cus > 8 * kPersistSlots) cus = 8 * kPersistSlots;
  if (cus < 8) cus = 8;
  n_slots = cus / 8;
  const int64_t rounds = (items + n_slots - 1) / n_slots;
  const int64_t groups = (rounds + kRoundsPerWg - 1) / kRoundsPerWg;
  return (unsigned)((groups > 0 ? groups : 1) * 8 * n_slots);
}
inline unsigned grid_blocks(int64_t n_blocks_max, int cus, int& n_slots) {
  return grid_items((n_blocks_max + 7) / 8 * kPersistSlots, cus, n_slots);
}
inline int64_t blocks_of(int n_pt, int64_t n_qg) { return (int64_t)((n_pt + kBP - 1) / kBP) * ((n_qg + kBQ - 1) / kBQ); }

}  // namespace ff8
