// What the grouped GEMM kernels share: launch arguments, the K-major LDS tile swizzle and the
// LDS DMA.
#pragma once

#include "ff8_device.hpp"
#include "ff8_launch.hpp"

namespace ff8 {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;

constexpr int kBK = 128;        // k per stage (one scale block)
constexpr int kScaleBatch = 4;  // K blocks per scale batch

struct GemmArgs {
  const uint8_t* P;   // fprop: w; dgrad: w; wgrad: xT
  const void* sP;     // scales: float, or UE8M0 bytes
  const uint8_t* Q;   // fprop: a; dgrad: g; wgrad: gT
  const void* sQ;
  const int32_t* offsets;
  void* out;
  int E;
  int M_cap;          // dimensions are below 2^31 (byte offsets below 2^32 are checked on the host)
  int Np;             // extent of p (output columns)
  int Nq;             // wgrad: extent of q (N); fprop/dgrad: unused
  int Kdim;           // fprop/dgrad: contraction length; wgrad: unused (per group)
  int n_pt, n_qt;     // p tiles; q tiles (wgrad only)
  int accumulate;
  int n_slots;        // workgroups per XCD in one group of the grid
  // wgrad expert shares (share = 0: none fit): each XCD takes one rect_q x rect_p-tile
  // rectangle of every expert's n_qt x n_pt tiles, the 8 rectangles tiling it (rect_b along p)
  int share, rect_q, rect_p, rect_b;
  int rounds;         // small-group kernel: tiles per workgroup
};

// K-major stage tile: rows x 128 bytes, 16-byte chunk c of row r at c ^ kswz(r).  Any
// 16 consecutive rows take the 16 distinct (r % 2, chunk) slots of a 256-byte bank window,
// and the swizzle repeats every 16 rows, so fragment rows 32 apart share one address
// register (plus an immediate offset).
__device__ __forceinline__ int kswz(int r) { return (r >> 1) & 7; }

// LDS DMA (buffer_load ... lds): each lane loads 16 (or 4) bytes at resource base +
// soff + voff into LDS at M0 + 16 * lane (or 4 * lane).  The resources cover exactly
// their tensor, and every operand offset is in voffset, which the hardware range-checks:
// rows past a tensor's end read zeros, so tiles at the edges need no clamping (K-blocked
// wgrad operands: rows past the end read the next block's rows, or zeros after the last
// block; those rows' accumulators are never stored).  Issued
// through inline asm so that the compiler does not serialize the pipeline with
// conservative waits; the kernel waits for its own DMA (vmcnt) before the barrier that
// publishes a stage.  The compiler's hazard checks do not look inside asm.  A buffer
// instruction needs 5 wait states after a VALU write of an SGPR it reads (the resource or M0
// may come straight from v_readfirstlane, or from v_readlane when the compiler reloads a
// spilled SGPR), and an LDS DMA 1 after an SALU write of M0; with fewer, the load can use the
// register's old value.  The DMAs issued right after a tile's setup (kLoop false) carry all 5.
// Inside the K loop the resources are loop-invariant and M0 is set by s_mov, so the DMAs there
// carry 1 (4 issue cycles fewer per DMA, 1-2% on every GEMM); the hazard scan of the compiled
// kernels checks that no VALU write of an SGPR they read comes closer.
// Raw (stride 0) buffer resource: loads at offsets >= `bytes` return zeros.
__device__ __forceinline__ i32x4 make_rsrc(const void* base, uint32_t bytes = 0xFFFFFFFFu) {
  const uint64_t a = (uint64_t)base;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu));  // stride 0
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;   // raw 32-bit data format
  return r;
}
template <bool kLoop = false>
__device__ __forceinline__ void dma16(const i32x4& rsrc, uint32_t voff, uint32_t lds_off) {
  if constexpr (kLoop)
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "{m0}"(lds_off), "v"(voff), "s"(rsrc)
                 : "memory");
  else
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "{m0}"(lds_off), "v"(voff), "s"(rsrc)
                 : "memory");
}
// 4-byte form (scales).  The scale DMAs, like the operand DMAs, keep their whole offset in
// the range-checked voffset, so a lane past a scale tensor's end reads zeros.
template <bool kLoop = false>
__device__ __forceinline__ void dma4(const i32x4& rsrc, uint32_t voff, uint32_t lds_off) {
  if constexpr (kLoop)
    asm volatile("s_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" : : "{m0}"(lds_off), "v"(voff), "s"(rsrc)
                 : "memory");
  else
    asm volatile("s_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds" : : "{m0}"(lds_off), "v"(voff), "s"(rsrc)
                 : "memory");
}

__device__ __forceinline__ i32x8 with_half(i32x8 f, const u32x4& x, int half) {
  f[4 * half + 0] = (int)x[0];
  f[4 * half + 1] = (int)x[1];
  f[4 * half + 2] = (int)x[2];
  f[4 * half + 3] = (int)x[3];
  return f;
}

// Lane index as an opaque value: lane-dependent tile setup and epilogue arithmetic built
// on it is recomputed per tile instead of being hoisted out of the tile loop, where it
// would stay live (in registers) through the main loop.
__device__ __forceinline__ int opaque_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

}  // namespace ff8
