// Host side of the grouped GEMMs' tiles and of the routing's launches, for test_tile_order.py: the
// choice of the tile shape and of the launches, and a walk of the 256 x 256 tiles' order, every tile of every workgroup of a launch, as the kernel's own
// functions give them.
#include "gemm_order.hpp"
#include "gemm_rule.hpp"
#include "route_rule.hpp"

namespace {

template <int MODE, bool kPack>
long walk(ff8::GemmArgs g, const int* cum, const int* off, unsigned grid, int n_qg, int* out, long cap) {
  const bool packed = kPack && (MODE == ff8::kWgrad || cum[g.E + 1]);
  const int n_blocks = ff8::order_blocks(g.n_pt, n_qg, packed);
  long n = 0;
  for (unsigned b = 0; b < grid; ++b) {
    int k = (int)(b / (8 * g.n_slots)) * ff8::kRoundsPerWg;
    ff8::TileInfo t;
    while (ff8::next_tile<MODE, kPack>(g, cum, off, (int)b, n_blocks, false, k, t)) {
      if (n == cap) return -1;
      const int rows = MODE != ff8::kWgrad && ff8::half_tile(t) ? ff8::kTQ / 2 : ff8::kTQ;
      int* o = out + 6 * n++;  // the rows the tile's epilogue stores
      o[0] = t.e; o[1] = t.q0; o[2] = t.q0 + rows < t.q_end ? t.q0 + rows : t.q_end;
      o[3] = t.p0; o[4] = t.blk; o[5] = (int)b;
      ++k;
    }
  }
  return n;
}

}  // namespace

// Tiles (expert, first row, end row, first column, block, workgroup) of a launch over E groups at
// `offsets` and n_pt column tiles; n_qt: wgrad's row tiles, 0 for the row-wise products.  Returns
// their number, -1 if out is too small.
extern "C" long tile_order_walk(int E, const int* offsets, int m_cap, int n_pt, int n_qt, int cus, int* out, long cap) {
  ff8::GemmArgs g{};
  g.E = E; g.offsets = offsets; g.n_pt = n_pt; g.n_qt = n_qt; g.Kdim = ff8::kBK; g.Nq = n_qt * ff8::kTQ;
  static int cum[1026];
  cum[0] = 0;
  for (int e = 0; e < E; ++e) cum[e + 1] = cum[e] + (offsets[e + 1] - offsets[e] + ff8::kTQ - 1) / ff8::kTQ;
  const int n_qg = n_qt ? E * n_qt : cum[E];
  const long bound = n_qt ? (long)E * n_qt : (m_cap + ff8::kTQ - 1) / ff8::kTQ + E;
  const unsigned grid = ff8::grid_blocks(ff8::blocks_of(n_pt, bound), cus, g.n_slots);
  cum[E + 1] = ff8::packing_saves(n_pt, n_qg, true);
  const bool pack = n_pt % ff8::kBP != 0 && (!n_qt || ff8::packing_saves(n_pt, n_qg, false));
  if (n_qt) return pack ? walk<ff8::kWgrad, true>(g, cum, offsets, grid, n_qg, out, cap)
                        : walk<ff8::kWgrad, false>(g, cum, offsets, grid, n_qg, out, cap);
  return pack ? walk<ff8::kFprop, true>(g, cum, offsets, grid, n_qg, out, cap)
              : walk<ff8::kFprop, false>(g, cum, offsets, grid, n_qg, out, cap);
}

extern "C" int tile_rule(int mode, int E, int64_t M_cap, int64_t N, int64_t K, int64_t cus) {
  return ff8::small_gemm_tile((ff8::GemmMode)mode, E, M_cap, N, K, cus);
}
extern "C" int tile_rule_wide(int E, int64_t N, int64_t K, int64_t cus) { return ff8::wgrad_wide(E, N, K, cus); }
extern "C" int tile_per_cu(int per_cu, int lds) { return ff8::small_per_cu(per_cu, lds); }
extern "C" int route_launch_count(int64_t T, int k, int E, int align) { return ff8::route_launches(T, k, E, align); }
