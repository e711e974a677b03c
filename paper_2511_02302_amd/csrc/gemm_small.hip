// The grouped GEMMs for small expert groups and short contractions: the same products, operand
// layouts and MFMA as gemm.hip, on 128-wide tiles with two or three workgroups per CU.
//
// What bounds these shapes is not the matrix core but the stream around it: with a few rows per
// expert the weights are read once and barely multiplied, and with a few K stages per tile the
// output and the first loads are most of a tile's time.  A 256 x 256 tile with one workgroup per
// CU does these in turn (first loads, K loop, output) and multiplies padding rows; here
//   * tiles are 128 (p) x TQ (q) with TQ = 64 or 128, so a group of few rows wastes little (wgrad,
//     whose sizes do not depend on the routing, also 256 x 128: a quarter less DMA per product);
//   * two or three workgroups share a CU (51 to 70 KB of LDS each, and 4 or 8 bytes per expert), so
//     one's loads and output run under the other's products;
//   * each workgroup walks its tiles as one stream of K stages: the DMA runs two stages ahead of
//     the products across tile boundaries, so no tile waits for its first loads.
// A stage's fragments are all read into registers, a barrier then frees its buffer and the DMA
// of the stage after next goes into it while the MFMAs run: two buffers keep two stages in flight
// (256 x 128: one buffer, refilled under 1024 cycles of MFMAs and the other workgroup's).
// The MFMA takes the q rows as its A operand, so a lane holds one output column and a store
// instruction writes whole 128-byte runs of output rows straight from the accumulators.

#include "gemm_rule.hpp"
#include "gemm_shared.hpp"

namespace ff8 {

namespace {

constexpr int kThreads = 256;
constexpr int kBW = 8;    // p tiles per block of the tile order

template <int MODE, int TP, int TQ, typename SC>
struct Shape {
  static constexpr bool kE8 = sizeof(SC) == 1;
  static constexpr int FP = TP / 64, FQ = TQ / 64;  // 32-wide fragments per wave, 2 x 2 waves
  static constexpr int kBufs = TP == 256 ? 1 : 2;   // stage buffers
  static constexpr int kPB = TP * kBK, kQB = TQ * kBK, kStage = kPB + kQB;
  static constexpr int kDmaP = TP / 32, kDmaQ = TQ / 32, kDma = kDmaP + kDmaQ;  // per wave and stage
  // scale area of one batch (fprop / dgrad: four K blocks) or stage (wgrad): [P | Q]
  static constexpr int kScaleP = (MODE == kWgrad) ? TP * 4 : 256;
  static constexpr int kScaleQ = (MODE == kWgrad) ? 512 : TQ * 16;
  static constexpr int kScale = kScaleP + kScaleQ;
  static constexpr int kScaleOff = kBufs * kStage, kTabOff = kScaleOff + 2 * kScale;
  static constexpr int kPerCU = TQ == 128 ? 2 : 3;
  static constexpr int kStores = FQ * FP * (MODE == kWgrad ? 16 : 8);  // output stores of a wave's whole tile
};

// Wait until at most `dma` (next) plus `stores` (out) vector memory operations are in flight (at
// most 63 can be counted), then the workgroup's barrier.
template <int DMA, int STORES>
__device__ __forceinline__ void wait_younger(bool next, bool out) {
  constexpr int both = DMA + STORES < 63 ? DMA + STORES : 63, only = STORES < 63 ? STORES : 63;
  if (next && out)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(both) : "memory");
  else if (next)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DMA) : "memory");
  else if (out)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(only) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  asm volatile("s_barrier" ::: "memory");
}

// One tile: expert e, q rows [q0, q_end), p columns from p0, nk K stages; wgrad: first token k0
// and the valid K bytes [k_lo, 128) of the first and [0, k_hi) of the last stage.
struct TileAt {
  int e, q0, q_end, p0, nk, k0, k_lo, k_hi;
};

extern __shared__ __attribute__((aligned(1024))) uint8_t g_lds[];

// Tile t (0 <= t < n) of the launch: experts in order, inside one blocks of kBW p tiles, each
// block q tile by q tile, p fastest, so that workgroups running together share panels in L2.
template <int MODE, int TP, int TQ>
__device__ __forceinline__ TileAt tile_at(const GemmArgs& g, const int* cum, const int* off, int t) {
  TileAt a;
  int nq, rem;
  if (MODE == kWgrad) {
    const int per = g.n_qt * g.n_pt;
    if (__builtin_amdgcn_readfirstlane(cum[0]) == 0) {
      a.e = t / per;
      rem = t - a.e * per;
    } else {
      // Shares: every XCD takes an eighth of every expert's tiles, so that their loads stay equal
      // however the tokens are spread; eight experts in a row give each XCD another eighth (the
      // parts are not exactly equal), which makes its tiles of a period one run, modulo per.
      const int xcd = blockIdx.x & 7, period = t / per;
      const int r0 = (xcd * per >> 3) + t - period * per;
      rem = r0 < per ? r0 : r0 - per;
      a.e = 8 * period + (((8 * rem + 7) / per - xcd) & 7);
    }
    nq = g.n_qt;
    if (a.e >= g.E) {  // shares, past the last expert of the last period
      a.nk = 0;
      return a;
    }
  } else {
    int e = 0;  // experts whose tiles all come before t
    const int lane = threadIdx.x & 63;
    for (int base = 0; base < g.E; base += 64) {
      const bool before = base + lane < g.E && (int64_t)cum[base + lane + 1] * g.n_pt <= t;
      const unsigned long long m = __ballot(before);
      e += __popcll(m);
      if (m != ~0ull) break;
    }
    a.e = __builtin_amdgcn_readfirstlane(e);
    const int c0 = __builtin_amdgcn_readfirstlane(cum[a.e]);
    nq = __builtin_amdgcn_readfirstlane(cum[a.e + 1]) - c0;
    rem = t - c0 * g.n_pt;
  }
  const int pb = rem / (kBW * nq);
  rem -= pb * kBW * nq;
  const int w = min(kBW, g.n_pt - pb * kBW);
  const int qt = rem / w;
  a.p0 = (pb * kBW + rem - qt * w) * TP;
  a.k0 = 0;
  a.k_lo = 0;
  a.k_hi = kBK;
  if (MODE == kWgrad) {
    a.q0 = qt * TQ;
    a.q_end = g.Nq;
    // K runs over whole 128-token blocks from the one holding the expert's first row
    const int o0 = __builtin_amdgcn_readfirstlane(off[a.e]);
    const int o1 = __builtin_amdgcn_readfirstlane(off[a.e + 1]);
    a.k0 = o0 & ~(kBK - 1);
    a.nk = o1 > o0 ? (o1 - a.k0 + kBK - 1) / kBK : 0;
    a.k_lo = o0 - a.k0;
    a.k_hi = o1 > o0 ? o1 - (a.k0 + (a.nk - 1) * kBK) : kBK;
  } else {
    a.q0 = __builtin_amdgcn_readfirstlane(off[a.e]) + qt * TQ;
    a.q_end = __builtin_amdgcn_readfirstlane(off[a.e + 1]);
    a.nk = g.Kdim / kBK;
  }
  return a;
}

// The DMA side of a workgroup's stage stream.
template <int MODE, int TP, int TQ, typename SC>
struct Stream {
  using S = Shape<MODE, TP, TQ, SC>;
  i32x4 p_rsrc, q_rsrc, sp_rsrc, sq_rsrc;
  uint32_t p_voff, q_voff, sp_voff, sq_voff;  // lane offsets at the tile's K block 0
  uint32_t p_kstep, q_kstep, p_istep, q_istep, sp_kstep, sq_kstep;
  int c16;                // wgrad: first of this lane's 16 tokens in a K block
  int t, t_step, t_end;   // current tile, stride, end of the XCD's range
  int ks, nk, k_lo, k_hi;
  int produced, batches;  // stages and scale batches issued so far
  int wave, lane;

  __device__ __forceinline__ void init(const GemmArgs& g) {
    constexpr uint32_t sb = sizeof(SC);
    const uint32_t Np = g.Np, Kd = g.Kdim, M = g.M_cap, E = g.E, Nq = g.Nq;
    if (MODE == kWgrad) {
      p_rsrc = make_rsrc(g.P, Np * M);
      q_rsrc = make_rsrc(g.Q, Nq * M);
      sp_rsrc = make_rsrc(g.sP, (M / kTile) * Np * sb);
      sq_rsrc = make_rsrc(g.sQ, (M / kTile) * Nq * sb);
      p_kstep = Np * kBK;
      q_kstep = Nq * kBK;
      p_istep = q_istep = 32 * kBK;
      sp_kstep = Np * sb;
      sq_kstep = Nq * sb;
    } else {
      p_rsrc = make_rsrc(g.P, E * Np * Kd);
      q_rsrc = make_rsrc(g.Q, M * Kd);
      sp_rsrc = make_rsrc(g.sP, E * (Np / kTile) * (Kd / kTile) * sb);
      sq_rsrc = make_rsrc(g.sQ, M * (Kd / kTile) * sb);
      p_kstep = (MODE == kDgrad) ? kBK * Np : kBK;
      p_istep = 32 * ((MODE == kDgrad) ? Np : Kd);
      q_kstep = kBK;
      q_istep = 32 * Kd;
      sp_kstep = ((MODE == kDgrad) ? Np / kTile : 1) * sb;
      sq_kstep = sb;
    }
  }
  // Sources of the current tile.  Instruction i of wave w carries the 8 rows of group w + 4 i;
  // lane l row l / 8 of them, LDS chunk l % 8, so memory chunk (l % 8) ^ swizzle(row).
  __device__ __forceinline__ void setup(const GemmArgs& g, const int* cum, const int* off) {
    constexpr uint32_t sb = sizeof(SC);
    const TileAt a = tile_at<MODE, TP, TQ>(g, cum, off, t);
    ks = 0;
    nk = a.nk;
    k_lo = a.k_lo;
    k_hi = a.k_hi;
    const uint32_t Np = g.Np, Kd = g.Kdim, Nq = g.Nq, e = a.e, p0 = a.p0, q0 = a.q0;
    const uint32_t r = 8 * wave + (lane >> 3);
    const uint32_t c = 16 * ((lane & 7) ^ kswz((int)r));
    if (MODE == kWgrad) {
      const uint32_t b0 = (uint32_t)a.k0 / kBK;
      p_voff = (b0 * Np + p0 + r) * kBK + c;
      q_voff = (b0 * Nq + q0 + r) * kBK + c;
      c16 = (int)c;
      // one dword per lane: 64 rows of float32 scales per wave (each wave repeats another's past the
      // tile), all rows of UE8M0 bytes (repeated likewise)
      const uint32_t pr = S::kE8 ? 4 * (lane & (TP / 4 - 1)) : (64 * wave + lane) & (TP - 1);
      const uint32_t qr = S::kE8 ? 4 * (lane & (TQ / 4 - 1)) : (64 * wave + lane) & (TQ - 1);
      sp_voff = (b0 * Np + p0 + pr) * sb;
      sq_voff = (b0 * Nq + q0 + qr) * sb;
      return;
    }
    q_voff = (q0 + r) * Kd + c;
    if (MODE == kFprop) {
      p_voff = (e * Np + p0 + r) * Kd + c;
    } else {  // W_e [n][p]: 128 n rows x 128 bytes, chunk ^ (n & 6)
      p_voff = (e * Kd + r) * Np + p0 + 16 * ((lane & 7) ^ (r & 6));
    }
    const uint32_t kb = Kd / kTile, nb = Np / kTile, pb = p0 / kTile, j = lane & 3;
    if (S::kE8) {
      sq_voff = (q0 + 64 * (TQ == 128 ? wave & 1 : 0) + lane) * kb;
      sp_voff = (MODE == kFprop) ? (e * nb + pb) * kb : (e * kb + j) * nb + (pb & ~3u);
    } else {
      sq_voff = ((q0 + 16 * (wave & (TQ / 16 - 1)) + (lane >> 2)) * kb + j) * sb;
      sp_voff = ((MODE == kFprop) ? (e * nb + pb) * kb + j : (e * kb + j) * nb + pb) * sb;
    }
  }
  // Issue the next stage of the stream (if there is one) into buffer produced % 2.
  __device__ __forceinline__ void produce(const GemmArgs& g) {
    if (t >= t_end) return;
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_u8*)g_lds;
    const uint32_t stage = lds + (S::kBufs == 1 ? 0 : (uint32_t)(produced & 1) * S::kStage);
    if (MODE == kWgrad || (ks & 3) == 0) {
      const uint32_t sc = lds + S::kScaleOff + (uint32_t)(batches & 1) * S::kScale;
      const uint32_t k = (uint32_t)ks;
      if (MODE == kWgrad) {
        const uint32_t pw = S::kE8 ? 0 : wave & (TP / 64 - 1), qw = S::kE8 ? 0 : wave & (TQ / 64 - 1);
        dma4(sp_rsrc, sp_voff + k * sp_kstep, sc + pw * 256);
        dma4(sq_rsrc, sq_voff + k * sq_kstep, sc + S::kScaleP + qw * 256);
      } else {
        dma4(sp_rsrc, sp_voff + k * sp_kstep, sc);
        if (S::kE8) {
          dma4(sq_rsrc, sq_voff + k, sc + S::kScaleP + (TQ == 128 ? wave & 1 : 0) * 256);
        } else {
          dma4(sq_rsrc, sq_voff + k * sq_kstep, sc + S::kScaleP + (wave & (TQ / 16 - 1)) * 256);
          if (TQ == 128)
            dma4(sq_rsrc, sq_voff + k * sq_kstep + 64u * (uint32_t)(g.Kdim / kTile) * 4u, sc + S::kScaleP + (wave + 4) * 256);
        }
      }
      ++batches;
    }
    uint32_t pv = p_voff + (uint32_t)ks * p_kstep, qv = q_voff + (uint32_t)ks * q_kstep;
    uint32_t pi = p_istep, qi = q_istep;
    if (MODE == kWgrad) {  // tokens of other experts in the first and last block read zeros
      const bool drop = (ks == 0 && c16 < k_lo) || (ks == nk - 1 && c16 >= k_hi);
      if (drop) {
        pv = (uint32_t)p_rsrc[2];
        qv = (uint32_t)q_rsrc[2];
        pi = qi = 0;
      }
    }
#pragma unroll
    for (int i = 0; i < S::kDmaP; ++i) dma16(p_rsrc, pv + i * pi, stage + (uint32_t)(wave + 4 * i) * 1024u);
#pragma unroll
    for (int i = 0; i < S::kDmaQ; ++i)
      dma16(q_rsrc, qv + i * qi, stage + S::kPB + (uint32_t)(wave + 4 * i) * 1024u);
    ++produced;
    ++ks;
  }
  // Move on to the next tile with K once the current one's stages are all issued.
  __device__ __forceinline__ void advance(const GemmArgs& g, const int* cum, const int* off) {
    while (t < t_end && ks >= nk) {
      t += t_step;
      if (t < t_end) setup(g, cum, off);
    }
  }
};

template <int MODE, int TP, int TQ, typename SC>
__global__ __launch_bounds__(kThreads, (Shape<MODE, TP, TQ, SC>::kPerCU)) void grouped_gemm_small_kernel(GemmArgs g) {
  using S = Shape<MODE, TP, TQ, SC>;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave >> 1, wq = wave & 1;
  const int l31 = lane & 31, h = lane >> 5;
  int* const off = reinterpret_cast<int*>(g_lds + S::kTabOff);  // row offsets of the experts
  int* const cum = off + g.E + 1;  // fprop / dgrad: cumulative q tiles; wgrad: one flag, shares

  int n;  // tiles of the launch
  bool shares = false;
  if (MODE != kWgrad) {
    if (tid < 64) {
      int carry = 0;
      for (int base = 0; base < g.E; base += 64) {
        const int i = base + tid;
        const int o0 = i < g.E ? g.offsets[i] : 0, o1 = i < g.E ? g.offsets[i + 1] : 0;
        int v = i < g.E ? (o1 - o0 + TQ - 1) / TQ : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int u = __shfl_up(v, d);
          if (tid >= d) v += u;
        }
        if (i < g.E) {
          cum[i + 1] = carry + v;
          off[i + 1] = o1;
        }
        carry += __shfl(v, 63);
      }
      if (tid == 0) {
        cum[0] = 0;
        off[0] = g.offsets[0];
      }
    }
    __syncthreads();
    n = __builtin_amdgcn_readfirstlane(cum[g.E]) * g.n_pt;
  } else {
    for (int i = tid; i <= g.E; i += kThreads) off[i] = g.offsets[i];
    __syncthreads();
    // Shares when the largest expert has over 64 rows more than 1.5 times the mean (every workgroup
    // finds the same).  Zipf(1.2), 512 rows on average, 32 experts of 4096 x 7168: 1506 us by
    // contiguous eighths, 892 by shares (256 x 256 tiles: 976).  With even routing the eighths share
    // more panels in L2: 64 experts of 2816 x 2048, 256 rows each, 240 and 281.
    if (tid < 64) {
      int mx = 0;
      for (int i = tid; i < g.E; i += 64) mx = max(mx, off[i + 1] - off[i]);
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) mx = max(mx, __shfl_xor(mx, d));
      if (tid == 0) cum[0] = 2 * (int64_t)mx * g.E > 3 * (int64_t)(off[g.E] - off[0]) + 128 * (int64_t)g.E;
    }
    __syncthreads();
    shares = __builtin_amdgcn_readfirstlane(cum[0]) != 0;
    n = (shares ? (g.E + 7) / 8 : g.E) * g.n_qt * g.n_pt;  // shares: of one XCD
  }
  // XCD x (workgroups are dispatched round-robin over the 8) takes a contiguous eighth of the
  // tiles, group by group of `rounds` tiles for each of its n_slots running workgroups.
  // (shares: its own tiles, an eighth of every expert's, see tile_at).
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int group = local / g.n_slots, slot = local - group * g.n_slots;
  const int first = shares ? 0 : xcd * (n >> 3) + min(xcd, n & 7);
  const int end = shares ? n : first + (n >> 3) + (xcd < (n & 7) ? 1 : 0);
  const int lo = first + group * g.n_slots * g.rounds, hi = min(end, lo + g.n_slots * g.rounds);
  if (lo + slot >= hi) return;

  Stream<MODE, TP, TQ, SC> st;
  st.wave = wave;
  st.lane = lane;
  st.t = lo + slot;
  st.t_step = g.n_slots;
  st.t_end = hi;
  st.produced = st.batches = 0;
  st.init(g);
  st.setup(g, cum, off);
  st.advance(g, cum, off);
  for (int i = 0; i < S::kBufs; ++i) {
    st.produce(g);
    st.advance(g, cum, off);
  }

  // lane addresses of the fragment reads within a stage
  int ra[4];  // K-major: 16-byte chunk 2 h + i of row l31 (i = 4 half-step + piece)
#pragma unroll
  for (int i = 0; i < 4; ++i) ra[i] = l31 * kBK + (((2 * h + 4 * (i >> 1) + (i & 1)) ^ kswz(l31)) << 4);
  int rt[S::FP];  // dgrad P: 8-byte transposing reads
  if (MODE == kDgrad) {
    const int gg = lane >> 4, hh = lane & 1, ii = (lane & 15) >> 1;
#pragma unroll
    for (int a = 0; a < S::FP; ++a) {
      const int chunk = 2 * (wp * S::FP + a) + (gg & 1);
      rt[a] = (32 * (gg >> 1) + ii) * kBK + ((chunk ^ (ii & 6)) << 4) + 8 * hh;
    }
  }

  int stage_no = 0, batch_no = 0;
  int since = 2;  // stages consumed since this wave's last full output (2: two or more)
  TileAt a = tile_at<MODE, TP, TQ>(g, cum, off, lo + slot);
  for (int t = lo + slot; t < hi; t += g.n_slots) {
    f32x16 acc[S::FQ][S::FP];
#pragma unroll
    for (int b = 0; b < S::FQ; ++b)
#pragma unroll
      for (int p = 0; p < S::FP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][p][v] = 0.0f;
    uint32_t sp_pack = 0, sq_pack[S::FQ];  // E8M0 bytes of the batch's four K blocks
    for (int ks = 0; ks < a.nk; ++ks) {
      // this wave's DMA of the stage has landed when only younger ones are in flight (loads and
      // stores retire in order): the next stage's, and the previous tile's output if all its
      // stores were issued after the stage's DMA, which is so for the kBufs stages that follow it
      wait_younger<S::kDma, S::kStores>(st.produced > stage_no + 1, since < S::kBufs);
      if (since < 2) ++since;
      const uint8_t* const P = g_lds + (S::kBufs == 1 ? 0 : (stage_no & 1) * S::kStage);
      const uint8_t* const Q = P + S::kPB;
      i32x8 fp[2][S::FP], fq[2][S::FQ];
#pragma unroll
      for (int hs = 0; hs < 2; ++hs) {
#pragma unroll
        for (int b = 0; b < S::FQ; ++b)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            fq[hs][b] = with_half(fq[hs][b],
                                  *reinterpret_cast<const u32x4*>(Q + ra[2 * hs + i] + (wq * S::FQ + b) * 32 * kBK), i);
#pragma unroll
        for (int p = 0; p < S::FP; ++p) {
          if constexpr (MODE == kDgrad) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
              const i32x2 x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                  (i32x2 __attribute__((address_space(3)))*)((lds_u8*)(P + rt[p] + (64 * hs + 8 * rr) * kBK)));
              fp[hs][p][2 * rr] = x[0];
              fp[hs][p][2 * rr + 1] = x[1];
            }
          } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
              fp[hs][p] = with_half(fp[hs][p],
                                    *reinterpret_cast<const u32x4*>(P + ra[2 * hs + i] + (wp * S::FP + p) * 32 * kBK), i);
          }
        }
      }
      // scales: one E8M0 byte per row and K block (the float32 exponent field or the stored byte)
      uint32_t cp[S::FP], cq[S::FQ];
      if constexpr (MODE == kWgrad) {
        const uint8_t* const sc = g_lds + S::kScaleOff + (stage_no & 1) * S::kScale;
#pragma unroll
        for (int p = 0; p < S::FP; ++p) {
          const int row = 32 * (wp * S::FP + p) + l31;
          cp[p] = S::kE8 ? sc[row] : reinterpret_cast<const uint32_t*>(sc)[row] >> 23;
        }
#pragma unroll
        for (int b = 0; b < S::FQ; ++b) {
          const int row = 32 * (wq * S::FQ + b) + l31;
          cq[b] = S::kE8 ? sc[S::kScaleP + row] : reinterpret_cast<const uint32_t*>(sc + S::kScaleP)[row] >> 23;
        }
      } else {
        if ((ks & 3) == 0) {
          const uint8_t* const sc = g_lds + S::kScaleOff + (batch_no & 1) * S::kScale;
          const u32x4 v = *reinterpret_cast<const u32x4*>(sc);
          if constexpr (!S::kE8) {
            sp_pack = (v[0] >> 23) | (v[1] >> 23) << 8 | (v[2] >> 23) << 16 | (v[3] >> 23) << 24;
          } else if constexpr (MODE == kFprop) {
            sp_pack = v[0];
          } else {
            const int sh = 8 * ((a.p0 / kTile) & 3);
            sp_pack = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) sp_pack |= ((v[j] >> sh) & 0xffu) << (8 * j);
          }
#pragma unroll
          for (int b = 0; b < S::FQ; ++b) {
            const int row = 32 * (wq * S::FQ + b) + l31;
            if constexpr (S::kE8) {
              sq_pack[b] = reinterpret_cast<const uint32_t*>(sc + S::kScaleP)[row];
            } else {
              const u32x4 q = reinterpret_cast<const u32x4*>(sc + S::kScaleP)[row];
              sq_pack[b] = ((q[0] >> 23) & 0xffu) | ((q[1] >> 23) & 0xffu) << 8 | ((q[2] >> 23) & 0xffu) << 16 |
                           (q[3] >> 23) << 24;
            }
          }
          ++batch_no;
        }
        const int sh = 8 * (ks & 3);
#pragma unroll
        for (int p = 0; p < S::FP; ++p) cp[p] = sp_pack >> sh;
#pragma unroll
        for (int b = 0; b < S::FQ; ++b) cq[b] = sq_pack[b] >> sh;
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every wave has read the stage
      ++stage_no;
      st.produce(g);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int hs = 0; hs < 2; ++hs)
#pragma unroll
        for (int b = 0; b < S::FQ; ++b)
#pragma unroll
          for (int p = 0; p < S::FP; ++p)
            acc[b][p] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[hs][b], fp[hs][p], acc[b][p], 0, 0, 0,
                                                                        (int)cq[b], 0, (int)cp[p]);
      __builtin_amdgcn_sched_barrier(0);
      st.advance(g, cum, off);  // under the MFMAs
    }
    const TileAt done = a;
    if (t + g.n_slots < hi) a = tile_at<MODE, TP, TQ>(g, cum, off, t + g.n_slots);
    if (MODE == kWgrad && done.nk == 0 && (g.accumulate || done.e >= g.E)) continue;
    since = done.q0 + 32 * S::FQ * (wq + 1) <= done.q_end ? 0 : 2;
    if (TP == 256 && done.p0 + 128 * wp >= g.Np) {  // the wave's columns lie past the edge
      since = 2;
      continue;
    }
    // Output: lane column p, register i row 8 (i / 4) + 4 h + i % 4 of a 32 x 32 fragment.  Group
    // ends are multiples of 16, so the 8 rows of a register quad are all inside or all outside.
#pragma unroll
    for (int b = 0; b < S::FQ; ++b) {
      const int q = done.q0 + 32 * (wq * S::FQ + b);
#pragma unroll
      for (int gr = 0; gr < 4; ++gr) {
        if (q + 8 * gr >= done.q_end) break;
        const int col = done.p0 + 32 * wp * S::FP;
        if (MODE == kWgrad) {
          float* const o = static_cast<float*>(g.out) + ((size_t)done.e * g.Nq + q + 8 * gr) * g.Np + col;
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int p = 0; p < S::FP; ++p) {
              float* const d = o + (uint32_t)(4 * h + j) * (uint32_t)g.Np + 32 * p + l31;
              const float v = acc[b][p][4 * gr + j];
              __builtin_nontemporal_store(g.accumulate ? *d + v : v, d);
            }
        } else {
          // pairs of columns share a dword: even lanes take row 2 i of both, odd lanes row 2 i + 1
          uint16_t* const o = static_cast<uint16_t*>(g.out) + (size_t)(q + 8 * gr) * g.Np + col;
          const int odd = lane & 1;
          const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            uint32_t v[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
              const uint32_t mine = pack_bf16x2(acc[b][p][4 * gr + 2 * j], acc[b][p][4 * gr + 2 * j + 1]);
              const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xF, 0xF, false);
              v[p] = __builtin_amdgcn_perm(other, mine, sel);
            }
            // swap halves: x[0] = rows 2 j (+ odd) of both fragments' columns, x[1] = rows 4 + 2 j
            const auto x = __builtin_amdgcn_permlane32_swap(v[0], v[1], false, false);
            const int c = 32 * h + (l31 & ~1);
            __builtin_nontemporal_store(x[0], reinterpret_cast<uint32_t*>(o + (uint32_t)(2 * j + odd) * (uint32_t)g.Np + c));
            __builtin_nontemporal_store(x[1],
                                        reinterpret_cast<uint32_t*>(o + (uint32_t)(4 + 2 * j + odd) * (uint32_t)g.Np + c));
          }
        }
      }
    }
  }
}

template <int MODE, int TP, int TQ, typename SC>
hipError_t run_small(GemmArgs g, int64_t tiles_max, hipStream_t st) {
  using S = Shape<MODE, TP, TQ, SC>;
  const int lds = S::kTabOff + (MODE == kWgrad ? g.E + 2 : 2 * (g.E + 1)) * (int)sizeof(int);
  const int64_t per_xcd = (tiles_max + 7) / 8;
  int64_t slots = (int64_t)(device_cu_count() / 8) * small_per_cu(S::kPerCU, lds);
  if (slots < 1) slots = 1;
  if (slots > per_xcd) slots = per_xcd;
  g.n_slots = (int)slots;
  const int64_t groups = (per_xcd + slots * g.rounds - 1) / (slots * g.rounds);
  grouped_gemm_small_kernel<MODE, TP, TQ, SC><<<(unsigned)(groups * slots * 8), kThreads, lds, st>>>(g);
  return hipGetLastError();
}

template <typename SC>
hipError_t grouped_gemm_small_impl(GemmMode mode, int tq, const uint8_t* a, const SC* a_s, const uint8_t* b,
                                   const SC* b_s, const int32_t* offsets, int E, int64_t M_cap, int64_t N, int64_t K,
                                   void* out, int accumulate, hipStream_t st) {
  GemmArgs g{};
  g.P = b; g.sP = b_s; g.Q = a; g.sQ = a_s;
  g.offsets = offsets;
  g.out = out;
  g.E = E;
  g.M_cap = (int)M_cap;
  g.accumulate = accumulate;
  g.Np = (int)(mode == kFprop ? N : K);
  g.Nq = (int)N;
  g.Kdim = (int)(mode == kFprop ? K : N);
  if (mode == kWgrad) {
    g.n_qt = (int)(N / 128);
    const bool w256 = wgrad_wide(E, N, K, device_cu_count());
    g.rounds = M_cap <= 128 * (int64_t)E ? 1 : 4;
    g.n_pt = (int)(w256 ? (K + 255) / 256 : K / 128);
    const int64_t n = (int64_t)(E + 7) / 8 * 8 * g.n_qt * g.n_pt;  // whole periods of eight experts
    return w256 ? run_small<kWgrad, 256, 128, SC>(g, n, st) : run_small<kWgrad, 128, 128, SC>(g, n, st);
  }
  g.n_pt = g.Np / 128;
  g.rounds = 2;
  const int64_t n = ((M_cap + tq - 1) / tq + E) * g.n_pt;  // every expert adds at most one partial q tile
  if (mode == kFprop)
    return tq == 64 ? run_small<kFprop, 128, 64, SC>(g, n, st) : run_small<kFprop, 128, 128, SC>(g, n, st);
  return tq == 64 ? run_small<kDgrad, 128, 64, SC>(g, n, st) : run_small<kDgrad, 128, 128, SC>(g, n, st);
}

}  // namespace

int small_gemm_tile(GemmMode mode, int E, int64_t M_cap, int64_t N, int64_t K) {
  return small_gemm_tile(mode, E, M_cap, N, K, device_cu_count());
}

hipError_t launch_grouped_gemm_small(GemmMode mode, int tq, const uint8_t* a, const float* a_s, const uint8_t* b,
                                     const float* b_s, const int32_t* offsets, int E, int64_t M_cap, int64_t N,
                                     int64_t K, void* out, int accumulate, hipStream_t st) {
  return grouped_gemm_small_impl(mode, tq, a, a_s, b, b_s, offsets, E, M_cap, N, K, out, accumulate, st);
}
hipError_t launch_grouped_gemm_small(GemmMode mode, int tq, const uint8_t* a, const e8m0_t* a_s, const uint8_t* b,
                                     const e8m0_t* b_s, const int32_t* offsets, int E, int64_t M_cap, int64_t N,
                                     int64_t K, void* out, int accumulate, hipStream_t st) {
  return grouped_gemm_small_impl(mode, tq, a, a_s, b, b_s, offsets, E, M_cap, N, K, out, accumulate, st);
}

}  // namespace ff8
