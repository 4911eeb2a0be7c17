// The attend kernel (one persistent workgroup per compute unit), shared by
// the translation units that instantiate it (attend_*.hip).
//
//  * Work unit = (query row n with all H heads, page range).  Under a fold
//    plan each worker runs its own run of units; otherwise the planner's
//    queue (longest unit first) is dealt to the workers in a snake.  Neither
//    takes an atomic, so a worker knows its next unit ahead and issues that
//    unit's query and first steps before its current epilogue.
//  * 4 waves, one per SIMD.  Heads come in blocks of 16 (kHeadBlocks of
//    them: 8, 4 or 2).  For QK^T and the softmax wave w owns two head blocks
//    (one with at most 4 blocks), whose query rows stay in VGPRs for the
//    whole unit; for PV it owns output columns [128w, +128) of all heads, up
//    to 256 accumulation registers per lane.
//  * KV is staged 32 rows (half a page, one "step") at a time straight from
//    HBM into LDS with 16-byte direct-to-LDS loads, through a ring of four
//    slots: step j (QK), step j-1 (PV) and two steps in flight (three slots
//    and one step in flight for bf16 top-k, whose resolved rows need the
//    room).  A unit's page ids sit in one VGPR, 64 pages at a time.
//  * Iteration j, behind one workgroup barrier: the PV MFMAs of step j-2
//    carried past it; S^T[32 keys x heads] = K Q^T for step j (K read from
//    LDS as the A operand) with the loads of step j+2 spread through it; then
//    the softmax of step j interleaved with the PV MFMAs of step j-1; then P
//    of step j is written to LDS for every wave's PV.  Steady-state iterations
//    are compiled without the checks for a unit's first and last steps.
//  * All MFMAs are 16x16 tiles (x32 bf16, x128 fp8).  They take the same
//    cycles per flop as 32x32 ones but move half the accumulator data per
//    flop, and the chip, whose clock these kernels hold down by power, runs
//    faster.  Measured: a loop of a step's MFMAs and LDS reads alone takes
//    1,276 ns with 16x16x32 against 1,400 ns with 32x32x16 (1.93 against 1.65
//    GHz); whole passes, same box, all 16x16 against all 32x32: 256 short bf16
//    histories 204.6 -> 197.5 us, 4 long ones 114.2 -> 110.7, chunk 8 over fp8
//    531.7 -> 503.7, 2,048 listed positions 158.2 -> 149.5.
//  * Softmax in base 2 against a reference fixed at the unit's first-step
//    max, so O is never rescaled in the loop; a logit more than 64 above the
//    reference makes the workgroup redo the unit from its true max (at most
//    two passes).  Numerator and denominator share the reference, so the
//    result is the same function.
//  * O^T[512 x heads] += V^T P^T on MFMA: P^T fragments come from the P
//    exchange area in LDS and V^T is read from the same staged rows with
//    ds_read_b64_tr_b16 (bf16) or ds_read_b64_tr_b8 (fp8) transposing loads.
//  * Epilogue: O/l goes through LDS as bf16 (fp16 for a split unit's partial,
//    with a power-of-two scale per 128 columns) so that every store writes
//    whole 256-byte row pieces.
//  * fp8 cache: for QK, K's codes go to the fp8 pipe as they are (exact QK:
//    they convert exactly to bf16, a fragment ahead of its MFMAs); V's codes
//    convert exactly to bf16; the per-token scale is applied in fp32 to the
//    score and to P before P is rounded for PV.
//  * fp8 latent-row cache (656-byte rows: E4M3 latent with a power-of-two
//    scale per 128 columns, bf16 RoPE): K takes each tile's scale as its block
//    scale (exact QK: in the conversion); for PV, wave w's output columns are
//    tile w, so its P weights take the keys' tile-w scales.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"
#include "splash_common.hpp"
#include "device_types.hpp"

namespace splash {

// s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt[3:0], [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Workgroup barrier that does not drain outstanding global->LDS loads (a
// __syncthreads() would wait for every in-flight load).  LDS writes of this
// wave are completed first; the compiler may not move memory accesses across.
__device__ __forceinline__ void lds_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt((0x3F & 15) | (7 << 4) | (0 << 8) | ((0x3F >> 4) << 14));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Opaque copy: keeps the compiler from hoisting work derived from v out of a loop.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// 8 E4M3 codes (two dwords) -> 8 bf16 times `scale`, of which the
// instruction uses only the exponent (latent rows: the tile's scale, which
// the format keeps a power of two; otherwise 1).  Exact.
__device__ __forceinline__ bf16x8 fp8x8_to_bf16(u32x2 raw, float scale = 1.0f) {
  u32x4 r;
  r[0] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)raw[0], scale, false));
  r[1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)raw[0], scale, true));
  r[2] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)raw[1], scale, false));
  r[3] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)raw[1], scale, true));
  return __builtin_bit_cast(bf16x8, r);
}

// Reductions over the four lanes that share a head (lane n16 + 16 g).
__device__ __forceinline__ float head_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float head_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// ---- QK^T of the fp8 caches on the fp8 matrix pipe.  A bf16 query value
// has 8 significant bits and an E4M3 code 4, so after scaling a head's row
// by a power of two that puts its largest |q| in [128, 256), each value x is
// the sum of two codes: hi = rne(x), then lo = rne(x - hi), whose residual
// has at most 4 significant bits.  lo holds the residual times 2^4 and its
// MFMA scales it back by 2^-4 (the B operand's block scale), so the split is
// exact for |x| >= 2^-6 (2^-14 of the row's largest value); below that each
// term is off by at most 2^-14.  K enters as the cache's own codes (latent
// rows: with each tile's power-of-two scale as the A operand's block
// scale).  S = scale * (K hi^T + 2^-4 K lo^T), two 16x16x128 MFMAs per 128
// dims and tile, with no per-step conversion of K.  Where the bf16 MFMA keeps
// fp32 (5e-8 of the magnitude sum at most), the fp8 MFMA aligns the products of
// a lane's K values to the largest of them and drops what lies below 2^-13 of
// it (32x32x64 alike).  Over 262,144 sums of 576 products, query N(0, 1) split
// in two and K N(0, 1) codes, it is off by up to 5.8e-6 of sum |q_i k_i|, 7.5e-7
// on average (32x32x64: up to 7.0e-6 and 7.5e-7 on the same rows).

// N pairs of bf16 values (one pair per dword of w, low half first) -> hi
// codes of the values over `unit` (a power of two) and lo codes (the residual
// over unit / 16), value v at byte v % 4 of dword v / 4.  The conversions
// apply the scales themselves and the residual is taken in the values' own
// units, halved (a hi code of 256 under the largest unit, 2^120, is 2^128,
// past fp32; half of it is not), where it is exact: seven operations a pair
// (eleven with the scalings on their own), all of it latency at a unit's start.
template <int N>
__device__ __forceinline__ void split_query_values(const int* w, int* hi, int* lo, float unit) {
  const float unit_half = unit * 0.5f, unit_lo = unit * 0.03125f;
  auto residual = [](uint32_t bits, float h) { return __builtin_fmaf(__uint_as_float(bits), 0.5f, -h); };
#pragma unroll
  for (int g = 0; g < N / 2; ++g) {
    const uint32_t d0 = (uint32_t)w[2 * g], d1 = (uint32_t)w[2 * g + 1];
    s16x2 a = {0, 0};
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(a, __builtin_bit_cast(bf16x2, d0), unit, false);
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(a, __builtin_bit_cast(bf16x2, d1), unit, true);
    const int hw = __builtin_bit_cast(int, a);
    const f32x2 h01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hw, unit_half, false);
    const f32x2 h23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hw, unit_half, true);
    s16x2 v = {0, 0};
    v = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(v, residual(d0 << 16, h01[0]), residual(d0 & 0xFFFF0000u, h01[1]), unit_lo,
                                                 false);
    v = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(v, residual(d1 << 16, h23[0]), residual(d1 & 0xFFFF0000u, h23[1]), unit_lo,
                                                 true);
    hi[g] = hw;
    lo[g] = __builtin_bit_cast(int, v);
  }
}

// The same codes from the values scaled by `inv` = 1 / unit first, which the
// latent-row kernel keeps: with the shorter form the compiler gives its step
// loop another register assignment, and the whole kernel measures slower (64
// requests x 2 rows of 2,048 listed positions: 112 against 130 us a pass; the
// per-token kernel gains from it, chunk 8: 504 -> 488 us).
template <int N>
__device__ __forceinline__ void split_query_values_scaled(const int* w, int* hi, int* lo, float inv) {
#pragma unroll
  for (int g = 0; g < N / 2; ++g) {
    const uint32_t d0 = (uint32_t)w[2 * g], d1 = (uint32_t)w[2 * g + 1];
    const float x0 = __uint_as_float(d0 << 16) * inv, x1 = __uint_as_float(d0 & 0xFFFF0000u) * inv;
    const float x2 = __uint_as_float(d1 << 16) * inv, x3 = __uint_as_float(d1 & 0xFFFF0000u) * inv;
    s16x2 a = {0, 0};
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, x0, x1, 1.0f, false);
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, x2, x3, 1.0f, true);
    const int hw = __builtin_bit_cast(int, a);
    const f32x2 h01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hw, 1.0f, false);
    const f32x2 h23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hw, 1.0f, true);
    s16x2 v = {0, 0};
    v = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(v, (x0 - h01[0]) * 16.f, (x1 - h01[1]) * 16.f, 1.0f, false);
    v = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(v, (x2 - h23[0]) * 16.f, (x3 - h23[1]) * 16.f, 1.0f, true);
    hi[g] = hw;
    lo[g] = __builtin_bit_cast(int, v);
  }
}

// One MFMA of a score tile's accumulation chain, through inline asm with a
// VGPR accumulator: the compiler picks one MFMA destination class per
// function, and the output accumulator already fills the 256 accumulation
// registers.  finish_scores covers the latency before VALU code reads the
// result.  VALU_SRC adds the wait states that operands written by the VALU
// just before need.
template <bool FIRST, bool VALU_SRC>
__device__ __forceinline__ void mfma_qk(f32x4& acc, const bf16x8& k, const bf16x8& q) {
  if constexpr (FIRST) {
    if constexpr (VALU_SRC)
      asm volatile("s_nop 2\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(k), "v"(q));
    else
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(k), "v"(q));
  } else {
    if constexpr (VALU_SRC)
      asm volatile("s_nop 2\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "v"(q));
    else
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "v"(q));
  }
}
// A PV MFMA whose operands were written long before (those carried past a
// barrier).  With all 256 accumulation registers taken (ALL_ACC) it is in asm,
// so that the accumulator is updated in place: the compiler moved all eight
// accumulators through temporaries every step (32 copies and their wait
// states).  Nothing reads its result for many MFMAs.
template <bool ALL_ACC>
__device__ __forceinline__ void mfma_pv_in_place(f32x4& o, const bf16x8& v, const bf16x8& p) {
  if constexpr (ALL_ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(v), "v"(p));
  else o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, p, o, 0, 0, 0);
}
// A score tile's MFMA on the fp8 pipe, with E8M0 block scales: byte 0 of `ks`
// scales the lane's K block, byte QB of `qs` its query block, each by
// 2^(byte - 127).  (qs holds every query scale that the kernel uses, one a
// byte: kQScaleOne, kQScaleLo, kQScaleRope.)
constexpr int kQScaleOne = 0, kQScaleLo = 1, kQScaleRope = 2;
#define SPLASH_MFMA8(NOP, C, SEL, ...) \
  asm volatile(NOP "v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, " C ", %3, %4 " SEL __VA_ARGS__)
template <bool FIRST, bool VALU_SRC, int QB>
__device__ __forceinline__ void mfma_qk8(f32x4& acc, const i32x8& k, const i32x8& q, int ks, int qs) {
  static_assert(QB == 0 || (!FIRST && !VALU_SRC), "combinations used");
  if constexpr (FIRST) {
    SPLASH_MFMA8("", "0", "op_sel_hi:[0,0,0]", : "=&v"(acc) : "v"(k), "v"(q), "v"(ks), "v"(qs));
  } else if constexpr (VALU_SRC) {
    SPLASH_MFMA8("s_nop 2\n\t", "%0", "op_sel_hi:[0,0,0]", : "+v"(acc) : "v"(k), "v"(q), "v"(ks), "v"(qs));
  } else if constexpr (QB == kQScaleOne) {
    SPLASH_MFMA8("", "%0", "op_sel_hi:[0,0,0]", : "+v"(acc) : "v"(k), "v"(q), "v"(ks), "v"(qs));
  } else if constexpr (QB == kQScaleLo) {
    SPLASH_MFMA8("", "%0", "op_sel:[0,1,0] op_sel_hi:[0,0,0]", : "+v"(acc) : "v"(k), "v"(q), "v"(ks), "v"(qs));
  } else {
    SPLASH_MFMA8("", "%0", "op_sel_hi:[0,1,0]", : "+v"(acc) : "v"(k), "v"(q), "v"(ks), "v"(qs));
  }
}

// LDS layout of one staged step (32 cache rows): rows are cut into line
// groups of 128 B (bf16) or 64 B (fp8); group l of row r sits at
//   bf16: l*4096 + r*128 + ((c8 ^ swz8(r)) * 16)     (c8 = 16-byte chunk in group)
//   fp8:  l*2048 + r*64  + ((c4 ^ swz4(r)) * 16)
// so every 1 KB direct-to-LDS instruction reads whole memory lines of 8 (16)
// rows.  The XORs spread the operand reads over the 64 banks.  A 16-byte read
// takes lanes {0-3, 12-15, 20-23, 24-27} together (then the others alike), an
// 8-byte transposing read 32 lanes: of K, rows {0-3, 12-15} of one chunk and
// {4-11} of its neighbour share a cycle; of V, rows {4g .. 4g+3} of two
// neighbouring g (fp8: and the rows 16 above).  Both tables give each of them
// a bank slot of its own: measured for 4 waves, 16.0 cycles per K read (1 KB;
// a table fit for V alone: 32) and 11.5 (fp8 9.7) cycles per V read against
// 16.0 with (r >> 1) & 7 alone.
__device__ __forceinline__ uint32_t swz8(uint32_t r) {
  return ((r & 2u)) | ((((r >> 2) ^ (r >> 3)) & 1u) << 2) | ((r >> 3) & 1u);
}
__device__ __forceinline__ uint32_t swz4(uint32_t r) {
  return ((((r >> 2) ^ (r >> 3)) & 1u) << 1) | (((r >> 3) ^ (r >> 4)) & 1u);
}

// Latent rows (LAT: 656 B = 512 E4M3 codes at 0 | 4 fp32 tile scales at 512
// | 64 bf16 RoPE at 528): in LDS the latent's 8 line groups as fp8, then the
// RoPE as one bf16 line group at kRopeOff, then the rows' tile scales (16 B
// per row) at kData, and at kScaleT the same scales tile-major ([tile][row],
// written by wave 0 once its loads landed).
template <bool FP8, bool LAT = false>
struct StepLayout {
  static constexpr int kRowBytes = LAT ? 656 : FP8 ? kDimQK : 2 * kDimQK;   // 656 / 576 / 1152
  static constexpr int kRopeOff = 8 * kStepKeys * 64;                      // LAT: 16384
  static constexpr int kData = LAT ? kRopeOff + kStepKeys * 128 : kStepKeys * kRowBytes;  // 20480 / 18432 / 36864
  static constexpr int kScaleT = kData + 1024;                                            // LAT
  static constexpr int kBuf = LAT ? kData + 1536 : FP8 ? kData + 256 : kData;             // + fp32 scales
  // per wave and step (LAT: wave 0; waves 1-3 issue one fewer)
  static constexpr int kLoadsPerStep = LAT ? 6 : FP8 ? 5 : 9;
};

// Ring slots of the attend kernel: the step being multiplied (QK), the
// previous one (PV), and kDist steps in flight.  Four slots (two steps in
// flight) everywhere except the bf16 top-k variant, whose resolved pool rows
// take the LDS the fourth slot would need.
template <bool FP8, bool TOPK>
struct Ring {
  static constexpr int kSlots = (FP8 || !TOPK) ? 4 : 3;
  static constexpr int kDist = kSlots - 2;
};

// LDS map beyond the ring (bytes): P of one step, one KB per head block
// (fragment order: lane l's 8 weights at 16 l)
constexpr int kPBytes = kMaxHeads * kStepKeys * 2;

// Element pairs of the softmax that run under the QK stream (of 8 a step)
constexpr int kSoftmaxPairs1 = 2;

// Direct global->LDS loads, issued through asm so that the compiler's wait
// insertion (which cannot tell which LDS bytes they write) does not drain
// them before every LDS read; the kernel waits for them explicitly.  The
// source is a uniform 64-bit base plus a per-lane 32-bit offset, or (_v) a
// per-lane 64-bit address; the LDS destination is `lds` + LDS_ADD + 16 * lane
// (4 * lane for the dword form).  SRC_ADD goes into the instruction's offset,
// which moves the LDS destination as well: M0 is set that much lower.  Three
// instructions a load: a lone wave on its SIMD pays an issue slot for each.
// (M0 is a reserved register: the compiler allocates nothing to it, writes it
// only for an instruction that takes it, and refuses it as a clobber.  It is
// not restored: nothing else in these kernels takes it, which their listing
// shows as no mention of m0 but these.)
// NT: the non-temporal hint ("nt" on gfx950), which streams the lines through
// the caches instead of keeping them; the attend kernel sets it when no other
// tile reads the same pages (one query row per request), so that the cache
// rows do not evict what is reused.
#define SPLASH_DMA(INSN, ADDR, HINT, ...)                                                                  \
  asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\t" INSN " %2, " ADDR " offset:%3" HINT               \
               ::"s"(lds), "n"(LDS_ADD - SRC_ADD), "v"(va), "n"(SRC_ADD), ##__VA_ARGS__ : "scc", "memory")
template <bool NT, int LDS_ADD, int SRC_ADD>
__device__ __forceinline__ void dma_b128(const void* sbase, uint32_t va, uint32_t lds) {
  if constexpr (NT) SPLASH_DMA("global_load_lds_dwordx4", "%4", " nt", "s"(sbase));
  else SPLASH_DMA("global_load_lds_dwordx4", "%4", "", "s"(sbase));
}
template <bool NT, int LDS_ADD, int SRC_ADD>
__device__ __forceinline__ void dma_b128_v(uint64_t va, uint32_t lds) {
  if constexpr (NT) SPLASH_DMA("global_load_lds_dwordx4", "off", " nt");
  else SPLASH_DMA("global_load_lds_dwordx4", "off", "");
}
template <bool NT, int LDS_ADD>
__device__ __forceinline__ void dma_b32(const void* sbase, uint32_t va, uint32_t lds) {
  constexpr int SRC_ADD = 0;
  if constexpr (NT) SPLASH_DMA("global_load_lds_dword", "%4", " nt", "s"(sbase));
  else SPLASH_DMA("global_load_lds_dword", "%4", "", "s"(sbase));
}
template <bool NT, int LDS_ADD>
__device__ __forceinline__ void dma_b32_v(uint64_t va, uint32_t lds) {
  constexpr int SRC_ADD = 0;
  if constexpr (NT) SPLASH_DMA("global_load_lds_dword", "off", " nt");
  else SPLASH_DMA("global_load_lds_dword", "off", "");
}

// lane id from an asm (volatile: recomputed where it is used, not held in a
// register across the loop)
__device__ __forceinline__ uint32_t fresh_lane() {
  uint32_t ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  return ln;
}

// Where a step's rows come from.  Dense: a uniform base and the lane's byte
// offset inside the step (for t = 0), token scales at a uniform base.  Top-k
// (gathered rows): the lane's row address (chunk included) and token-scale
// address; latent rows also need other rows of the step (step_rows: its 32
// resolved rows in LDS) and the pool.
struct StepSrc {
  const uint8_t* base;
  const float* scales;
  uint32_t lane_off;
  uint64_t row_addr, scale_addr;
  const int32_t LDS_AS* step_rows;
  const uint8_t* kv;
};

// Load t of one step, into the ring slot at LDS address `buf`; wdst is where
// the wave's part of a line group starts.
//  bf16: wave w loads rows [8w, 8w+8) of every line group g (t = g);
//  fp8:  instruction i = w + 4t (< 18) loads line group i >> 1, rows
//        [16 (i & 1), +16); waves 2 and 3 also load the 32 token scales.
//  LAT:  t < 4 as fp8 (the latent's 8 line groups); t = 4: wave w loads the
//        RoPE of rows [8w, 8w+8) into the bf16 layout; t = 5: wave 0 loads
//        the 32 rows' tile scales (lanes 32-63 repeat 0-31).
template <bool FP8, int t, bool LAT, bool NT, bool TOPK>
__device__ __forceinline__ void issue_one(const StepSrc& s, uint32_t buf, uint32_t wdst, int wave) {
  auto rows = [&]() {
    if constexpr (TOPK) dma_b128_v<NT, 4096 * t, 128 * t>(s.row_addr, buf + wdst);
    else dma_b128<NT, 4096 * t, 128 * t>(s.base, s.lane_off, buf + wdst);
  };
  if constexpr (LAT) {
    using L = StepLayout<true, true>;
    if constexpr (t < 4) {
      rows();
    } else if constexpr (t == 4) {
      const uint32_t ln = fresh_lane(), r = 8 * wave + (ln >> 3);
      const uint32_t in_row = 528 + (((ln & 7) ^ swz8(r)) * 16);
      if constexpr (TOPK)
        dma_b128_v<NT, L::kRopeOff, 0>(
            (uint64_t)(uintptr_t)s.kv + (uint64_t)(uint32_t)s.step_rows[r] * L::kRowBytes + in_row, buf + 1024 * wave);
      else
        dma_b128<NT, L::kRopeOff, 0>(s.base, r * L::kRowBytes + in_row, buf + 1024 * wave);
    } else if (wave == 0) {
      const uint32_t r = fresh_lane() & 31;
      if constexpr (TOPK)
        dma_b128_v<NT, L::kData, 0>((uint64_t)(uintptr_t)s.kv + (uint64_t)(uint32_t)s.step_rows[r] * L::kRowBytes + 512, buf);
      else
        dma_b128<NT, L::kData, 0>(s.base, r * L::kRowBytes + 512, buf);
    }
  } else if constexpr (!FP8) {
    rows();
  } else {
    if (t < 4 || wave + 4 * t < 18) rows();
    else if constexpr (TOPK) dma_b32_v<NT, 18432>(s.scale_addr, buf);
    else dma_b32<NT, 18432>(s.scales, (fresh_lane() & 31) * 4, buf);
  }
}
template <bool FP8, bool LAT, bool NT, bool TOPK, int t = 0>
__device__ __forceinline__ void issue_step(const StepSrc& s, uint32_t buf, uint32_t wdst, int wave) {
  if constexpr (t < StepLayout<FP8, LAT>::kLoadsPerStep) {
    issue_one<FP8, t, LAT, NT, TOPK>(s, buf, wdst, wave);
    issue_step<FP8, LAT, NT, TOPK, t + 1>(s, buf, wdst, wave);
  }
}

// Operand fragments as the LDS reads return them (fp8: the 8 codes) and
// their conversion to the MFMA's bf16.  The streams convert a fragment in
// the slot that uses it, so the read has the slots since its issue to land;
// converting right at the read would wait for it there.
template <bool FP8>
using FragRaw = typename std::conditional<FP8, u32x2, bf16x8>::type;
template <bool FP8>
__device__ __forceinline__ bf16x8 frag_bf16(const FragRaw<FP8>& r) {
  if constexpr (FP8) return fp8x8_to_bf16(r);
  else return r;
}
// K operand (A): dims 32ks + 8g + [0, 8) of key 16kb + n16.  kbase: the lane's
// address for (kb = 0, ks = 0); the chunk XORs of the others act on its bits.
template <bool FP8>
__device__ __forceinline__ FragRaw<FP8> load_k_raw(const uint8_t LDS_AS* buf, uint32_t kbase, int ks, int kb) {
  if constexpr (!FP8)
    return *(const bf16x8 LDS_AS*)(buf + (kbase ^ (64 * (ks & 1))) + 4096 * (ks >> 1) + 2048 * kb);
  else
    return *(const u32x2 LDS_AS*)(buf + (kbase ^ (32 * (ks & 1) + 16 * kb)) + 2048 * (ks >> 1) + 1024 * kb);
}
// V^T operand (A): the 16 columns of column block c of the wave's 8, keys
// {4g .. 4g+3, 16+4g .. 16+4g+3} in slot order.  vbuf includes the wave's
// column offset; vbase is the lane's address for c = 0.
template <bool FP8>
__device__ __forceinline__ FragRaw<FP8> load_v_raw(const uint8_t LDS_AS* vbuf, uint32_t vbase, int c) {
  if constexpr (!FP8) {
    const uint8_t LDS_AS* p = vbuf + (vbase ^ (32 * (c & 3))) + 4096 * (c >> 2);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 LDS_AS*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 LDS_AS*)(p + 2048));
    const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
    return __builtin_bit_cast(bf16x8, (u32x4){l2[0], l2[1], h2[0], h2[1]});
  } else {
    const i32x2 raw = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
        (i32x2 LDS_AS*)(vbuf + (vbase ^ (16 * (c & 3))) + 2048 * (c >> 2)));
    return __builtin_bit_cast(u32x2, raw);
  }
}

// Latent rows: a wave's PV covers output columns [128 wave, +128), one
// latent tile, so the tile scale of each key multiplies that key's P weight
// instead of V.  The scales are powers of two 2^e, so the product is the
// weight with e added to its bf16 exponent field: one packed 16-bit add per
// pair of weights (d holds e << 7 of both keys), and a packed max that
// turns an exponent pushed below the normal range into 0.  Exact while the
// result stays normal: weights are at most 2^64 in the pass that is kept
// and e <= 63 (a scale above 2^63 is outside the format); a weight pushed
// below 2^-126 contributes nothing the fp32 sum would keep.
__device__ __forceinline__ bf16x8 scale_p(bf16x8 p, const u32x4& d) {
  const u32x4 w = __builtin_bit_cast(u32x4, p);
  u32x4 r;
  u16x2 sum[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // (scalar copies first: a bit cast taken straight from a vector element
    // reads element 0 whatever the index)
    const unsigned wi = w[i], di = d[i];
    sum[i] = __builtin_bit_cast(u16x2, wi) + __builtin_bit_cast(u16x2, di);
    asm volatile("" : "+v"(sum[i]));  // (all sums, then all maxima: a maximum right after its sum waits)
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(i16x2, sum[i]), (i16x2){0, 0}));
  return __builtin_bit_cast(bf16x8, r);
}
// The exponent steps (e << 7, 16 bits per key) of the tile-`wave` scales of
// the 8 keys of a P^T fragment, in slot order, from the tile-major table.
__device__ __forceinline__ u32x4 load_p_scales(const uint8_t LDS_AS* scales_t, int g, int wave) {
  const uint8_t LDS_AS* base = scales_t + 2 * (32 * wave + 4 * g);
  const u32x2 a = *(const u32x2 LDS_AS*)base, b = *(const u32x2 LDS_AS*)(base + 32);
  return (u32x4){a[0], a[1], b[0], b[1]};
}

// TOPK: the top-k variant.  Row n attends the first topk_count[n] token
// positions of its list topk_idx[n] (of request b = n / q_chunk); a unit
// covers list entries [64 p0, 64 p1) instead of pages, and its prologue
// resolves every entry to its pool row, from which each lane loads its
// staged row.
// LAT: the fp8 latent-row cache (FP8 set too): latent tiles with their tile
// scale for QK, the RoPE read as bf16, and for PV each wave's P scaled by its
// tile's key scales.
// NT: non-temporal cache-row loads and result stores (one query row per
// request).  Q8 (fp8 caches): QK on the fp8 matrix pipe (split query, K's
// own codes); without it K is converted to bf16 for the bf16 MFMA.
// NB: head blocks of 16 multiplied: 8, or 4 / 2 for at most 64 / 32 heads.
template <bool FP8, bool TOPK, bool LAT, bool NT, bool Q8, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void attend_kernel(AttendLaunch a) {
  static_assert(!LAT || FP8, "latent rows are an fp8 variant");
  static_assert(!Q8 || FP8, "the fp8-pipe QK serves the fp8 caches");
  static_assert(NB == 8 || NB == 4 || NB == 2, "head blocks");
  using L = StepLayout<FP8, LAT>;
  constexpr int kSlots = Ring<FP8, TOPK>::kSlots, kDist = Ring<FP8, TOPK>::kDist;
  constexpr int kRing = kSlots * L::kBuf;
  constexpr int kHB = NB == 8 ? 2 : 1;   // head blocks a wave owns for QK
  constexpr int kKS = 18;                // 32-dim steps of the bf16 QK
  constexpr int kQT = 4;                 // 128-dim blocks on the fp8 pipe (then the RoPE 64)
  constexpr bool kExact = FP8 && !Q8;    // exact QK of the fp8 caches: K converted to bf16
  // (exact QK) K fragment f of a step is one that is converted
  constexpr auto converts = [](int f) { return f < 36 && !(LAT && f % kKS >= 16); };
  // Unit overlap (dense bf16 and per-token fp8): the next unit's query and
  // first kDist steps are issued before this unit's epilogue stores, so their
  // latency hides behind the epilogue.  (Latent rows: with it the 8-block
  // kernel's step loop spills a register, whose reload waits for the loads in
  // flight.)
  constexpr bool kOverlap = !TOPK && !LAT;
  // LDS map: the ring, then the P exchange area (two steps), then (top-k
  // only) the unit's resolved pool rows.  The epilogue's staging (the
  // per-head normalisers, then 4 KB per wave) uses LDS idle at that time:
  // dense bf16, whose ring and P area fill the 160 KB, the ring slots 0-1,
  // with a unit's step j in slot (j + 2) mod 4 so that the next unit's first
  // two steps land in slots 2-3 meanwhile; otherwise past everything else.
  constexpr int kPOff = kRing;
  constexpr int kBtOff = kPOff + 2 * kPBytes;
  constexpr int kEnd = kBtOff + (TOPK ? kTopkUnitPages * kPage * 4 : 0);
  constexpr int kStageBytes = 1024 + 4 * 4096;
  constexpr bool kStageInRing = !FP8 && !TOPK;
  constexpr int kStageOff = kStageInRing ? 0 : kEnd;
  constexpr int kSlotBase = kStageInRing ? 2 : 0;
  static_assert(!kStageInRing || kStageBytes <= 2 * L::kBuf, "bf16 staging fits in ring slots 0-1");
  constexpr int kSmem = kStageInRing ? kEnd : kEnd + kStageBytes;
  static_assert(kSmem <= 163840, "LDS budget");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kSmem];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform per wave
  const int n16 = lane & 15, g = lane >> 4;
  // QK and softmax role: head blocks kHB * wave + i; with two head blocks in
  // all, waves 2 and 3 have none
  const bool qk_on = NB >= 4 || wave < NB;
  const float c2 = a.softmax_scale * 1.4426950408889634f;  // log2(e)
  // fp8 caches (Q8): the query's power-of-two row scale joins the softmax constant
  float c2v[kHB];
#pragma unroll
  for (int i = 0; i < kHB; ++i) c2v[i] = c2;
  // block scales of the fp8 QK MFMAs (E8M0): 1, 2^-4 for the lo terms, and
  // the RoPE block's: its query operand holds the hi codes in each lane's
  // first 16 bytes and the lo codes in its second; the MFMA takes the scales
  // of first halves from lane groups 0 and 1, those of second halves from 2
  // and 3 (checked with a probe).  The constant 1 of K is byte 0 too.
  const int bs = (int)opaque(127u | (123u << 8) | ((g < 2 ? 127u : 123u) << 16));
  const uint8_t* __restrict__ kv = (const uint8_t*)a.kv;
  uint8_t LDS_AS* sm = (uint8_t LDS_AS*)smem;
  uint8_t LDS_AS* p_lds = sm + kPOff;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)sm);
  float LDS_AS* l_lds = (float LDS_AS*)(sm + kStageOff);
  int32_t LDS_AS* s_bt = (int32_t LDS_AS*)(sm + kBtOff);  // top-k only

  // ---- per-lane offsets (bytes), fixed for the kernel ----
  const uint32_t wdst = FP8 ? 2048 * (wave >> 1) + 1024 * (wave & 1) : 1024 * wave;  // (see issue_one)
  auto dma_row_of = [&](uint32_t ln) -> uint32_t { return FP8 ? 16 * (wave & 1) + (ln >> 2) : 8 * wave + (ln >> 3); };
  const uint32_t dma_row = dma_row_of(lane);
  // the lane's bytes of its row, and (dense) of the step
  const uint32_t row_lane = FP8 ? 64 * (wave >> 1) + (((lane & 3) ^ swz4(dma_row)) * 16) : ((lane & 7) ^ swz8(dma_row)) * 16;
  const uint32_t src_lane = dma_row * L::kRowBytes + row_lane;
  // K operand: row n16; bf16 chunk g, fp8 8 bytes at 8g (see load_k_raw).
  // Q8: 16-byte chunk g of a pair of line groups, and of the RoPE group (twice:
  // against the hi and the lo codes).  The RoPE's base (latent
  // rows: its bf16 line group, two 32-dim steps) is made each step.
  uint32_t kbase;
  if constexpr (!FP8) kbase = n16 * 128 + ((g ^ swz8(n16)) * 16);
  else if constexpr (!Q8) kbase = n16 * 64 + (((g >> 1) ^ swz4(n16)) * 16) + 8 * (g & 1);
  else kbase = n16 * 64 + ((g ^ swz4(n16)) * 16);
  auto rope_base = [](uint32_t n, uint32_t gg) -> uint32_t {
    return LAT ? L::kRopeOff + n * 128 + ((gg ^ swz8(n)) * 16) : 8 * 2048 + n * 64 + ((gg ^ swz4(n)) * 16);
  };
  // V operand (transposing reads), see load_v_raw
  const int i16 = lane & 15;
  uint32_t vbase;
  if constexpr (!FP8) {
    // source lane: row 16t + 4g + (i16>>2), 16-byte chunk (i16>>1)&1 of the block's two, 8*(i16&1) bytes in
    const uint32_t row = 4 * g + (i16 >> 2);
    vbase = row * 128 + ((((uint32_t)(i16 >> 1) & 1u) ^ swz8(row)) * 16) + 8 * (i16 & 1) + 8192 * wave;
  } else {
    // tr8 source lane: key k = i16>>1 of the slot order, 8 columns at 8(i16&1)
    const uint32_t k = i16 >> 1, row = 16 * (k >> 2) + 4 * g + (k & 3);
    vbase = row * 64 + (swz4(row) * 16) + 8 * (i16 & 1) + 4096 * wave;
  }

  // Schedule, without atomics so that a worker knows its next unit ahead:
  // under a fold plan made for this many workers, worker g runs its own
  // units [table[g], table[g + 1]); otherwise the queue, ordered longest unit
  // first, is dealt in a snake (pass k gives worker g position kG + g, or
  // kG + G-1-g on odd passes), which pairs the longest units of one pass with
  // the shortest of the next as a longest-first greedy schedule would.  The
  // plan, the records and the lengths are read through the scalar cache:
  // nothing writes them while the kernel runs.
  typedef const int32_t __attribute__((address_space(4))) ConstI32;
  typedef const i32x4 __attribute__((address_space(4))) ConstI32x4;
  ConstI32* hdr = (ConstI32*)a.ws.header;
  const int32_t G = (int32_t)gridDim.x, wg = (int32_t)blockIdx.x;
  const bool own_run = hdr[kHdrSchedule] == G;
  const int32_t run_begin = own_run ? hdr[kHdrWorkerTable + wg] : 0;
  const int32_t run_end = own_run ? hdr[kHdrWorkerTable + wg + 1] : hdr[kHdrUnits];
  // With query chunks, the rows of one request read the same pages: the
  // queue's neighbours (the longest-first order keeps a request's units
  // together) go to workers of one XCD, whose L2 then serves the pages to
  // all of them.  Workgroups are placed on the 8 XCDs round robin, so
  // queue slot l of a pass goes to worker (l mod G/8) * 8 + l / (G/8).
  const int32_t lg = (a.q_chunk > 1 && (G & 7) == 0) ? (wg & 7) * (G >> 3) + (wg >> 3) : wg;
  auto unit_rec = [&](int k) -> i32x4 {
    const int32_t u = own_run ? run_begin + k : k * G + ((k & 1) ? G - 1 - lg : lg);
    if (u < run_end) return ((ConstI32x4*)a.ws.units)[u];
    return (i32x4){-1, 0, 0, 0};
  };
  // A unit's keys: request b, pages [p0, p1) (a shard's count from its first
  // page), keys [key_begin, key_end) in nsteps steps of 32.
  struct Geo {
    int tile, slot, b, p0, p1, key_begin, key_end, nsteps;
  };
  auto geometry = [&](const i32x4 r) {
    Geo u;
    u.tile = r.x;
    u.slot = r.w;
    u.b = r.x / a.q_chunk;
    const int qi = r.x - u.b * a.q_chunk;
    int Lk = tile_keys(((ConstI32*)a.seq_lens)[u.b], a.q_chunk, qi);
    u.p0 = r.y;
    u.p1 = r.z;
    if (a.key_end) {
      const int first = ((ConstI32*)a.key_begin)[u.b] >> 6;
      u.p0 += first;
      u.p1 += first;
      Lk = min(Lk, ((ConstI32*)a.key_end)[u.b]);
    }
    if constexpr (TOPK) Lk = ((ConstI32*)a.topk_count)[r.x];  // entries of the row's list
    u.key_begin = u.p0 * kPage;
    u.key_end = min(u.p1 * kPage, Lk);
    u.nsteps = (u.key_end - u.key_begin + kStepKeys - 1) / kStepKeys;
    return u;
  };
  // The page ids of 64 pages of a unit, one per lane (pages past the unit's
  // end repeat its last one, so only entries of the unit's pages are read).
  auto load_pages = [&](const Geo& u, int chunk) -> int {
    const int32_t* bt = a.block_table + (size_t)u.b * a.bt_stride + u.p0;
    return bt[min(64 * chunk + (int)fresh_lane(), u.p1 - u.p0 - 1)];
  };
  // Query operands (B), row = head.  bf16: k = dims 32ks + 8g + [0, 8).
  // Padding heads (head >= H) take head 0's row: their scores stay finite and
  // nothing of theirs is stored.  (Nothing consumes the loaded values here,
  // so the loads stay in flight until the first QK MFMA.)
  // Q8: block t (128 dims), lane group g: dims 128t + 16g + [0, 16) and the
  // same 64 further on, as K's two 16-byte chunks; loaded as bf16 into qh
  // (first half) and ql, which split_query replaces by the hi and lo codes.
  // The RoPE block (qe): dims 512 + 16g + [0, 16).
  bf16x8 qf[Q8 ? 1 : kKS][kHB];
  i32x8 qh[Q8 ? kQT : 1][kHB], ql[Q8 ? kQT : 1][kHB], qe[(Q8 && !LAT) ? kHB : 1];
  bf16x8 qr[(Q8 && LAT) ? 2 : 1][kHB];  // latent rows: the RoPE fragments, bf16 (times the row scale's inverse)
  auto load_q = [&](int t) {
    if (!qk_on) return;
    // (lane coordinates made here: the row addresses are not hoisted out of
    // the unit loop, where they would be spilled)
    const int ln = (int)fresh_lane(), g = ln >> 4;
#pragma unroll
    for (int i = 0; i < kHB; ++i) {
      const int head = 16 * (kHB * wave + i) + (ln & 15);
      const uint16_t* qrow = (const uint16_t*)a.q + ((size_t)t * a.H + (head < a.H ? head : 0)) * kDimQK;
      auto pair = [&](int dim, int dim2) {
        const u32x4 f0 = *(const u32x4*)(qrow + dim), f1 = *(const u32x4*)(qrow + dim2);
        return __builtin_bit_cast(i32x8, __builtin_shufflevector(f0, f1, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      if constexpr (Q8) {
#pragma unroll
        for (int m = 0; m < kQT; ++m) {
          qh[m][i] = pair(128 * m + 16 * g, 128 * m + 16 * g + 8);
          ql[m][i] = pair(128 * m + 64 + 16 * g, 128 * m + 64 + 16 * g + 8);
        }
        if constexpr (LAT) {
#pragma unroll
          for (int p = 0; p < 2; ++p) qr[p][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + 512 + 32 * p + 8 * g));
        } else {
          qe[i] = pair(512 + 16 * g, 512 + 16 * g + 8);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qf[ks][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + 32 * ks + 8 * g));
      }
    }
  };
  // Q8: the head's row scale, then the split of every block; sets the lane's
  // softmax constant
  auto split_query = [&]() {
    // largest magnitude of both halves, as bf16 bit patterns (they order like
    // the magnitudes)
    auto bmax = [](uint32_t m, uint32_t w) -> uint32_t {
      const uint32_t mag = w & 0x7FFF7FFFu;
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_bit_cast(u16x2, mag)));
    };
    auto bmax_f = [](float m, uint32_t w) {
      return fmaxf(m, fmaxf(fabsf(__uint_as_float(w << 16)), fabsf(__uint_as_float(w & 0xFFFF0000u))));
    };
#pragma unroll
    for (int i = 0; i < kHB; ++i) {
      int biased;  // exponent field of the row's largest magnitude
      if constexpr (LAT) {
        float mx = 0.f;
#pragma unroll
        for (int m = 0; m < kQT; ++m)
#pragma unroll
          for (int d = 0; d < 8; ++d) mx = bmax_f(bmax_f(mx, (uint32_t)qh[m][i][d]), (uint32_t)ql[m][i][d]);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int d = 0; d < 4; ++d) mx = bmax_f(mx, __builtin_bit_cast(u32x4, qr[p][i])[d]);
        biased = (int)((__float_as_uint(head_max(mx)) >> 23) & 255u);
      } else {
        uint32_t mb = 0;
#pragma unroll
        for (int m = 0; m < kQT; ++m)
#pragma unroll
          for (int d = 0; d < 8; ++d) mb = bmax(bmax(mb, (uint32_t)qh[m][i][d]), (uint32_t)ql[m][i][d]);
#pragma unroll
        for (int d = 0; d < 8; ++d) mb = bmax(mb, (uint32_t)qe[i][d]);
        mb = (mb & 0xFFFFu) > (mb >> 16) ? mb & 0xFFFFu : mb >> 16;
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 16, 64));
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 32, 64));
        biased = (int)(mb >> 7);
      }
      int e = biased - 127;  // floor(log2 max), -127 for 0
      // (every finite bf16 has e <= 127, so the largest scaled value stays
      // under 256; rows below 2^-100 become zeros, their scores ~0 anyway)
      e = e < -100 ? -100 : (e > 127 ? 127 : e);
      const float inv = __uint_as_float((uint32_t)(127 + 7 - e) << 23);   // 2^(7 - e)
      const float unit = __uint_as_float((uint32_t)(127 - 7 + e) << 23);  // 2^(e - 7)
      c2v[i] = c2 * unit;
#pragma unroll
      for (int m = 0; m < kQT; ++m) {
        int w[16], hi[8], lo[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          w[d] = qh[m][i][d];
          w[8 + d] = ql[m][i][d];
        }
        if constexpr (LAT) split_query_values_scaled<16>(w, hi, lo, inv);
        else split_query_values<16>(w, hi, lo, unit);
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          qh[m][i][d] = hi[d];
          ql[m][i][d] = lo[d];
        }
      }
      if constexpr (LAT) {
        // the RoPE fragments times the same power of two (exact in bf16)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const u32x4 w = __builtin_bit_cast(u32x4, qr[p][i]);
          u32x4 o;
#pragma unroll
          for (int d = 0; d < 4; ++d)
            o[d] = pack_bf16x2(__uint_as_float(w[d] << 16) * inv, __uint_as_float(w[d] & 0xFFFF0000u) * inv);
          qr[p][i] = __builtin_bit_cast(bf16x8, o);
        }
      } else {
        // the RoPE block: dims 512 + 16g + [0, 16), hi codes then lo codes
        int w[8], hi[4], lo[4];
#pragma unroll
        for (int d = 0; d < 8; ++d) w[d] = qe[i][d];
        split_query_values<8>(w, hi, lo, unit);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          qe[i][d] = hi[d];
          qe[i][4 + d] = lo[d];
        }
      }
    }
  };

  i32x4 cur = unit_rec(0), nxt = unit_rec(1);
  bool pre = false;  // the current unit's query, pages and first steps were issued by the previous unit
  int pages = 0;     // page ids of the current unit (dense), 64 at a time
  for (int k = 0; cur.x >= 0; ++k) {
    const Geo U = geometry(cur);
    const int tile = U.tile, slot = U.slot, b = U.b, p0 = U.p0, p1 = U.p1;
    const int key_begin = U.key_begin, key_end = U.key_end, nsteps = U.nsteps;
    // the record after next, and what the next unit needs at this unit's
    // end, read now (scalar loads) and used there
    const i32x4 nxt2 = unit_rec(k + 2);
    Geo N = {};
    int n_phys = 0;
    if (kOverlap && nxt.x >= 0) {
      N = geometry(nxt);
      n_phys = ((ConstI32*)a.block_table)[(size_t)N.b * a.bt_stride + N.p0];
    }

    if constexpr (TOPK) {
      // pool row of every list entry of the unit (entries past the list end
      // read pool row 0, whose keys the tail mask removes)
      const int32_t* sel = a.topk_idx + (size_t)tile * a.topk;
      const int32_t* btr = a.block_table + (size_t)b * a.bt_stride;
      for (int e = tid; e < (p1 - p0) * kPage; e += 256) {
        int row = 0;
        if (key_begin + e < key_end) {
          const int pos = sel[key_begin + e];
          row = btr[pos >> 6] * kPage + (pos & (kPage - 1));
        }
        s_bt[e] = row;
      }
    }
    if (!pre) {
      if constexpr (!TOPK) pages = load_pages(U, 0);
      load_q(tile);
    }
    __syncthreads();  // (top-k) the resolved rows visible

    // the first page also through the scalar cache: the first steps need not
    // wait for the vector load of the page ids
    const int first_phys = TOPK ? 0 : ((ConstI32*)a.block_table)[(size_t)b * a.bt_stride + p0];
    // source of step j on page `phys` (two steps per page: key_begin is a
    // page boundary); top-k: from the lane's pool row and (fp8) token-scale row
    auto step_src = [&](int j, int phys) {
      StepSrc s = {};
      const int half = j & 1;
      s.base = kv + (size_t)phys * (kPage * L::kRowBytes) + (half ? kStepKeys * L::kRowBytes : 0);
      if constexpr (FP8 && !LAT) s.scales = a.kv_scales + (size_t)phys * kPage + half * kStepKeys;
      s.lane_off = src_lane;
      return s;
    };
    auto lane_row = [&](int j) { return s_bt[j * kStepKeys + dma_row_of(fresh_lane())]; };
    auto scale_row = [&](int j) { return FP8 ? s_bt[j * kStepKeys + (fresh_lane() & 31)] : 0; };
    auto topk_src = [&](int j, int row, int srow) {
      StepSrc s = {};
      s.row_addr = (uint64_t)(uintptr_t)kv + (uint64_t)(uint32_t)row * L::kRowBytes + row_lane;
      s.scale_addr = (uint64_t)(uintptr_t)a.kv_scales + (uint64_t)(uint32_t)srow * 4;
      s.step_rows = s_bt + j * kStepKeys;
      s.kv = kv;
      return s;
    };
    // ring slot of step j (byte offset); slots_at gives those of steps j-1,
    // j, ..., j + kDist, which the iterations rotate (laundered so that the
    // compiler keeps them in scalars)
    auto slot_off = [&](int j) { return (uint32_t)((j + kSlotBase + kSlots) % kSlots) * L::kBuf; };
    uint32_t ring[kSlots];

    // Softmax reference: fixed at the first step's max (O is still zero
    // there), never moved afterwards, so O is never rescaled inside the loop.
    // If a later logit exceeds it by more than 64 (base 2), P could overflow:
    // the workgroup then redoes the unit with the unit's true max, which is
    // known after the first pass.
    float m_init[kHB], m_ref[kHB], l_run[kHB], l_exact[kHB];
#pragma unroll
    for (int i = 0; i < kHB; ++i) m_init[i] = -INFINITY;
    f32x4 o[8][NB];     // [column block of the wave's 128][head block]
    bf16x8 pf[NB], d_v;  // P^T of the step being multiplied; V of the column block carried past a barrier
    for (int pass = 0;; ++pass) {
      // Pipeline: step j is staged kDist steps ahead; iteration j runs QK of
      // step j, then the softmax of step j together with PV of step j-1.
#pragma unroll
      for (int j = 0; j < kDist; ++j)
        if (j < nsteps && (pass > 0 || !pre)) {
          if constexpr (TOPK) issue_step<FP8, LAT, NT, TOPK>(topk_src(j, lane_row(j), scale_row(j)), lds0 + slot_off(j), wdst, wave);
          else issue_step<FP8, LAT, NT, TOPK>(step_src(j, first_phys), lds0 + slot_off(j), wdst, wave);
        }
      if constexpr (Q8) {
        if (pass == 0 && qk_on) split_query();
      }

#pragma unroll
      for (int x = 0; x < 8; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) o[x][y] = (f32x4){};
      d_v = (bf16x8){};
#pragma unroll
      for (int hb = 0; hb < NB; ++hb) pf[hb] = (bf16x8){};
      float tmax[kHB];  // largest t = z*log2(e) - m_ref of this pass, per lane and head
#pragma unroll
      for (int i = 0; i < kHB; ++i) {
        m_ref[i] = m_init[i];
        l_run[i] = l_exact[i] = 0.f;
        tmax[i] = -INFINITY;
      }

#pragma unroll
      for (int i = 0; i < kSlots; ++i) {
        ring[i] = slot_off(i - 1);
        asm volatile("" : "+s"(ring[i]));
      }
      // where the step staged next comes from, looked up one iteration early
      // (top-k: its rows, read from LDS per lane)
      auto page_of = [&](int j) {
        if ((j & 127) == 0 && j > 0) {  // uniform, once per 64 pages
          pages = load_pages(U, j >> 7);
          asm volatile("" : "+v"(pages));  // (waited for here: a wait after the branch would drain the loads in flight every step)
        }
        return __builtin_amdgcn_readlane(pages, (j >> 1) & 63);
      };
      if (!TOPK && pass > 0 && nsteps > 128) pages = load_pages(U, 0);
      StepSrc next = {};
      int next_row = 0, next_srow = 0;
      if (kDist < nsteps) {
        if constexpr (TOPK) {
          next_row = lane_row(kDist);
          next_srow = scale_row(kDist);
        } else {
          next = step_src(kDist, page_of(kDist));
        }
      }
      // One pipeline iteration.  pf_mode 1 (the steady state): step j + kDist
      // exists, so it is staged here, and step j is not the last one (no
      // history end inside it); 2: nothing left to stage; 0 (the first
      // step): decided at run time.
      auto iteration = [&](int j, auto with_pv, auto pf_mode) {
        constexpr bool kPV = decltype(with_pv)::value;
        constexpr int kPFM = decltype(pf_mode)::value;
        uint8_t LDS_AS* buf = sm + ring[1];                  // step j
        uint8_t LDS_AS* vbuf = sm + ring[0];                 // step j-1
        const uint32_t pf_buf = lds0 + ring[kSlots - 1];     // step j + kDist
        uint8_t LDS_AS* p_cur = p_lds + kPBytes * (j & 1);
        const uint8_t LDS_AS* p_prev = p_lds + kPBytes * ((j + 1) & 1);  // P of step j-1
        const int valid = key_end - (key_begin + j * kStepKeys);  // >= 1; >= 32 in the steady state
        const bool pf_next = kPFM == 1 ? true : kPFM == 2 ? false : (j + kDist < nsteps);
        const bool may_end = kPFM != 1;
        StepSrc src;
        if constexpr (TOPK) src = topk_src(j + kDist, next_row, next_srow);
        else src = next;
        if (kDist == 2 && (kPFM == 1 || j + 1 < nsteps)) {
          // step j + 1's loads may still be in flight (LAT: only wave 0 loads
          // the tile scales)
          if (LAT && wave != 0) wait_vmcnt<L::kLoadsPerStep - 1>();
          else wait_vmcnt<L::kLoadsPerStep>();
        } else {
          wait_vmcnt<0>();
        }
        if (may_end && valid < kStepKeys) {
          // rows past the history end: P is zero there, V must not be NaN
          const u32x4 z = {0, 0, 0, 0};
          const uint32_t ln = fresh_lane();
          if ((int)dma_row_of(ln) >= valid) {
#pragma unroll
            for (int t = 0; t < L::kLoadsPerStep; ++t)
              if (!FP8 || t < 4 || (!LAT && wave + 4 * t < 18)) *(u32x4 LDS_AS*)(buf + wdst + 16 * ln + 4096 * t) = z;
          }
          if constexpr (LAT) {
            // their RoPE and tile scales (each cleared by the wave that
            // loaded it, after its own loads landed): zero scales keep the
            // scaled P and K finite
            if ((int)(8 * wave + (ln >> 3)) >= valid) *(u32x4 LDS_AS*)(buf + L::kRopeOff + 1024 * wave + 16 * ln) = z;
            if (wave == 0 && (int)(ln & 31) >= valid) *(u32x4 LDS_AS*)(buf + L::kData + 16 * ln) = z;
          } else if constexpr (FP8) {
            // their token scales too (both waves that load the scales clear
            // them after their own loads landed, so a zero is written last)
            if (wave >= 2 && (int)(ln & 31) >= valid) *(float LDS_AS*)(buf + L::kData + 4 * ln) = 0.f;
          }
        }
        if constexpr (LAT) {
          // the tile-major table of the step's scale exponents (after the
          // zero fill): (bits >> 16) - (127 << 7) is e << 7 for 2^e; a
          // zeroed scale (rows past the end, whose weights are 0) gives a
          // step that keeps those weights 0
          const uint32_t ln = fresh_lane();
          if (wave == 0 && ln < 32) {
            const u32x4 v = *(const u32x4 LDS_AS*)(buf + L::kData + 16 * ln);
#pragma unroll
            for (int t = 0; t < 4; ++t)
              *(uint16_t LDS_AS*)(buf + L::kScaleT + 2 * (32 * t + ln)) = (uint16_t)(((v[t] >> 16) & 0x7F80u) - 0x3F80u);
          }
        }
        // step j staged; P of step j-1 visible; every wave is done with
        // iteration j-1, so the slot of step j-2 is free
        lds_barrier();

        // fp8: laundered copies of the lane's addresses, so that their XORed
        // variants are made here each step and not kept (and spilled)
        const uint32_t kbase_i = FP8 ? opaque(kbase) : kbase, vbase_i = FP8 ? opaque(vbase) : vbase;
        const uint32_t lane_i = FP8 ? fresh_lane() : (uint32_t)lane, lane16 = 16 * lane_i, n16_i = lane_i & 15, g_i = lane_i >> 4;
        const uint32_t kbase_r = rope_base(n16_i, g_i);
        auto load_pf = [&](int hb) { pf[hb] = *(const bf16x8 LDS_AS*)(p_prev + 1024 * hb + lane16); };
        // the MFMAs step j-2 carried past the barrier (column block 7), operands in registers
        auto deferred = [&]() {
#pragma unroll
          for (int hb = 0; hb < NB; ++hb) {
            mfma_pv_in_place<NB == 8>(o[7][hb], d_v, pf[hb]);
            __builtin_amdgcn_sched_barrier(0);
          }
          // (outside the steady state an accumulator may be spilled: its wait states)
          if constexpr (NB == 8 && kPFM != 1) asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
        };
        u32x4 psc;           // LAT: tile-`wave` scale exponent steps of the P fragments' keys
        FragRaw<FP8> vf[3];  // V fragments of three column blocks, as read
        bf16x8 vcur;         // that of the current column block, converted
        // PV MFMA q of step j-1: column block c = q / NB, head block q % NB;
        // the V fragment of column block c + 2 is read at the first MFMA of c
        constexpr int kNPV = 8 * NB;
        auto pv_slot = [&](auto qc) {
          if constexpr (kPV) {
            constexpr int q = decltype(qc)::value, c = q / NB, hb = q % NB;
            if constexpr (hb == 0 && c + 2 < 8) vf[(c + 2) % 3] = load_v_raw<FP8>(vbuf, vbase_i, c + 2);
            if constexpr (LAT) {
              if constexpr (c == 0) pf[hb] = scale_p(pf[hb], psc);
            }
            if constexpr (hb == 0) vcur = frag_bf16<FP8>(vf[c % 3]);
            if constexpr (c == 7) d_v = vcur;  // carried past the next barrier
            else o[c][hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vcur, pf[hb], o[c][hb], 0, 0, 0);
          }
        };

        // ---- the softmax of step j, base 2; lane = heads 16 (kHB wave + i) + n16, keys
        // 16kb + 4g + r; t = z*log2(e) - m_ref.  P is rounded to bf16 for the
        // PV MFMA.  The bf16 path normalises the output by the sum of the
        // rounded weights, so the weights applied to V sum to one and only the
        // spread of the rounding errors reaches the output; the LSE keeps the
        // exact fp32 sum.
        f32x4 sacc[2][kHB];  // scores [key block][head block]
        f32x4 sc[2];         // fp8: token scales
        auto load_sc = [&]() {
          if constexpr (FP8 && !LAT) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) sc[kb] = *(const f32x4 LDS_AS*)(buf + L::kData + 16 * (4 * kb + g_i));
          }
        };
        // scores of key block kb: token scales (fp8) and the history-end mask
        auto finish_scores = [&](int kb) {
#pragma unroll
          for (int i = 0; i < kHB; ++i) {
            asm volatile("" : "+v"(sacc[kb][i]));  // (no use before this point)
            if constexpr (FP8 && !LAT) sacc[kb][i] *= sc[kb];
            if (may_end && valid < kStepKeys) {
              // the last step of a history: keys past its end get no weight
              const int hk = (int)opaque(4 * g_i);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (hk + 16 * kb + r >= valid) sacc[kb][i][r] = -INFINITY;
            }
          }
        };
        float psum[kHB], pexact[kHB], el_t[2], el_p[2];
#pragma unroll
        for (int i = 0; i < kHB; ++i) psum[i] = pexact[i] = 0.f;
        unsigned pb[kHB][4];
        // Operation u of element pair n (n = (2 i + kb) * 2 + r / 2), each
        // pinned where it is called, between the MFMAs of its slot: a lone
        // wave issues a 16x16 MFMA every 16 cycles and has 8 of them for other
        // instructions (an exp takes 8, the others 4), so the softmax is dealt
        // out evenly instead of sunk below the streams.
        auto softmax_op = [&](auto nc, auto uc) {
          constexpr int n = decltype(nc)::value, u = decltype(uc)::value;
          constexpr int i = n >> 2, kb = (n >> 1) & 1, r = 2 * (n & 1), w = n & 3;
          if constexpr (u < 2) {
            el_t[u] = __builtin_fmaf(sacc[kb][i][r + u], c2v[i], -m_ref[i]);
            asm volatile("" : "+v"(el_t[u]));
          } else if constexpr (u < 4) {
            el_p[u - 2] = __builtin_amdgcn_exp2f(el_t[u - 2]);
            asm volatile("" : "+v"(el_p[u - 2]));
          } else if constexpr (u == 4) {
            // largest t of the pass, two per max3
            tmax[i] = fmaxf(tmax[i], fmaxf(el_t[0], el_t[1]));
            asm volatile("" : "+v"(tmax[i]));
          } else if constexpr (u == 5 || u == 7) {
            pexact[i] += el_p[(u - 5) / 2];
            asm volatile("" : "+v"(pexact[i]));
          } else if constexpr (u == 6) {
            // (fp8: the token scale multiplies V too: fold it into the weight)
            if constexpr (FP8 && !LAT) pb[i][w] = pack_bf16x2(el_p[0] * sc[kb][r], el_p[1] * sc[kb][r + 1]);
            else pb[i][w] = pack_bf16x2(el_p[0], el_p[1]);
            asm volatile("" : "+v"(pb[i][w]));
          } else {
            if constexpr (!(FP8 && !LAT)) {
              psum[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pb[i][w]), (bf16x2){1.0f, 1.0f}, psum[i], false);
              asm volatile("" : "+v"(psum[i]));
            }
            // the head block's P^T fragment is whole: publish it for every wave's PV
            if constexpr (w == 3)
              *(u32x4 LDS_AS*)(p_cur + 1024 * (kHB * wave + i) + lane16) = (u32x4){pb[i][0], pb[i][1], pb[i][2], pb[i][3]};
          }
        };
        constexpr int kOps = 9, kPairs = 4 * kHB;
        // operations [first, last) of slot k of S slots over which pairs
        // [n0, n1) are dealt, by issue cycles (44 a pair)
        auto softmax_slot = [&](auto n0c, auto n1c, auto kc, auto sc_) {
          constexpr int n0 = decltype(n0c)::value, n1 = decltype(n1c)::value, k = decltype(kc)::value, S = decltype(sc_)::value;
          static_for<(n1 - n0) * kOps>([&](auto oc) {
            constexpr int o_ = decltype(oc)::value, u = o_ % kOps;
            constexpr int before = (o_ / kOps) * 44 + (u < 3 ? 4 * u : u == 3 ? 16 : 8 + 4 * u);
            if constexpr (before * S / ((n1 - n0) * 44) == k)
              softmax_op(std::integral_constant<int, n0 + o_ / kOps>{}, std::integral_constant<int, u>{});
          });
        };

        // ---- stream 1: QK^T of step j for the wave's head blocks, key block
        // 0 then 1 (bf16: 36 slots of one K fragment each), with the loads of
        // step j + kDist, the P fragments and the first two V fragments of step
        // j-1 and the first kP1 pairs of the softmax among them
        constexpr int kSlots1 = (Q8 && !LAT) ? 40 : 36;
        constexpr int kP1 = kPV && kHB == 2 ? kSoftmaxPairs1 : 0;
        constexpr int kFrom1 = kSlots1 / 2 + 5;  // key block 0's scores are done: five slots of MFMAs and reads after its last
        auto stream1_rest = [&](auto ic) {
          constexpr int i = decltype(ic)::value;
          if constexpr (kPV) {
            if constexpr (i >= kSlots1 - 10 - NB && i < kSlots1 - 10) load_pf(i - (kSlots1 - 10 - NB));
            if constexpr (i == (kP1 > 0 ? kFrom1 - 5 : kSlots1 - 8)) load_sc();
            if constexpr (LAT && i == kSlots1 - 10) psc = load_p_scales(vbuf + L::kScaleT, g_i, wave);
            if constexpr (i == kSlots1 - 8) vf[0] = load_v_raw<FP8>(vbuf, vbase_i, 0);
            if constexpr (i == kSlots1 - 4) vf[1] = load_v_raw<FP8>(vbuf, vbase_i, 1);
          }
          if constexpr ((i & 3) == 2 && (i >> 2) < L::kLoadsPerStep) {
            if (pf_next) issue_one<FP8, (i >> 2), LAT, NT, TOPK>(src, pf_buf, wdst, wave);
          }
          if constexpr (kP1 > 0 && i >= kFrom1) {
            if constexpr (i == kFrom1) finish_scores(0);
            softmax_slot(std::integral_constant<int, 0>{}, std::integral_constant<int, kP1>{},
                         std::integral_constant<int, i - kFrom1>{}, std::integral_constant<int, kSlots1 - kFrom1>{});
          }
        };
        if (qk_on) {
          constexpr int kKPre = 4;  // K fragments in flight
          FragRaw<FP8> kf[Q8 ? 1 : kKPre];
          // Q8: K operands of 128-dim blocks, two in turn: a block is read after
          // the first MFMA of the block before it (the registers' last MFMA
          // has been issued before that one and has read them long before
          // the LDS returns)
          i32x8 k8[Q8 ? 2 : 1];
          constexpr int kF = LAT ? 4 : 5;   // Q8: blocks per key block
          auto load_k8 = [&](int f) {
            const int kb = f / kF, t = f % kF;
            u32x4 c0, c1;
            if (t < kQT) {
              const uint8_t LDS_AS* p = buf + (kbase_i ^ (16 * kb)) + 1024 * kb + 4096 * t;
              c0 = *(const u32x4 LDS_AS*)p;
              c1 = *(const u32x4 LDS_AS*)(p + 2048);
            } else {
              const uint8_t LDS_AS* p = buf + (kbase_r ^ (16 * kb)) + 1024 * kb;
              c0 = *(const u32x4 LDS_AS*)p;
              c1 = *(const volatile u32x4 LDS_AS*)p;  // (a second read is cheaper than four moves)
            }
            return __builtin_bit_cast(i32x8, __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7));
          };
          // latent rows: RoPE fragments of key block kb, 32 dims p, bf16 as staged
          auto load_kr = [&](int kb, int p) {
            return *(const bf16x8 LDS_AS*)(buf + (kbase_r ^ (64 * p)) + 2048 * kb);
          };
          // bf16 K fragment f = 18 kb + ks
          auto load_kf = [&](int f) { return load_k_raw<FP8>(buf, kbase_i, f % kKS, f / kKS); };
          bf16x8 kr[LAT ? 4 : 1];
          // LAT: tile scales of the lane's key row in each key block (Q8: their
          // biased exponents are the E8M0 bytes)
          f32x4 tsc[2];
          auto load_tsc = [&](int kb) { tsc[kb] = *(const f32x4 LDS_AS*)(buf + L::kData + 16 * (16 * kb + n16_i)); };
          if constexpr (LAT) {
            load_tsc(0);
            if constexpr (!Q8) load_tsc(1);
          }
          // exact QK of the fp8 caches: fragment f converted to bf16 (kc[f % 3];
          // latent RoPE fragments are bf16 as read), half of it a slot
          u32x4 kc[kExact ? 3 : 1];
          auto convert_half = [&](auto fc, auto hc) {
            constexpr int f = decltype(fc)::value, h = decltype(hc)::value;
            if constexpr (converts(f)) {
              const float scale = LAT ? tsc[f / kKS][(f % kKS) >> 2] : 1.0f;
              const int raw = (int)kf[f % kKPre][h];
              kc[f % 3][2 * h] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw, scale, false));
              kc[f % 3][2 * h + 1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw, scale, true));
              asm volatile("" : "+v"(kc[f % 3]));
            }
          };
          if constexpr (Q8) {
            if constexpr (LAT) {
#pragma unroll
              for (int f = 0; f < 4; ++f) kr[f] = load_kr(f & 1, f >> 1);
            }
            k8[0] = load_k8(0);
          } else {
#pragma unroll
            for (int f = 0; f < kKPre; ++f) kf[f] = load_kf(f);
          }
          if constexpr (kPV) deferred();
          if constexpr (LAT && Q8) {
            // the RoPE part first, on the bf16 pipe
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
              for (int i = 0; i < kHB; ++i) {
                if (f < 2) mfma_qk<true, false>(sacc[f & 1][i], kr[f], qr[f >> 1][i]);
                else mfma_qk<false, false>(sacc[f & 1][i], kr[f], qr[f >> 1][i]);
              }
            // an fp8 MFMA reads the accumulator a bf16 MFMA wrote: its wait states
            asm volatile("s_nop 7");
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (kExact) {
            convert_half(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            convert_half(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
            convert_half(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});
            kf[0] = load_kf(kKPre);
            __builtin_amdgcn_sched_barrier(0);
          }
          static_for<kSlots1>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (Q8) {
              // block f: 2 kHB MFMAs (hi, lo per head block), spread over four
              // slots; the RoPE block (per-token cache) kHB
              constexpr int f = i >> 2, part = i & 3;
              if constexpr (f < 2 * kF) {
                constexpr int kb = f / kF, t = f % kF;
                const int ksc = LAT ? (int)((__float_as_uint(tsc[kb][t & 3]) >> 23) & 255u) : bs;
                // (a scale written by the VALU just before needs wait states)
                constexpr bool kV = LAT && part == 0;
                if constexpr (t < kQT) {
                  if constexpr (part < kHB) {
                    if constexpr (t == 0 && !LAT) mfma_qk8<true, false, kQScaleOne>(sacc[kb][part], k8[f & 1], qh[t][part], ksc, bs);
                    else mfma_qk8<false, kV, kQScaleOne>(sacc[kb][part], k8[f & 1], qh[t][part], ksc, bs);
                  } else if constexpr (part < 2 * kHB) {
                    mfma_qk8<false, false, kQScaleLo>(sacc[kb][part - kHB], k8[f & 1], ql[t][part - kHB], ksc, bs);
                  }
                } else {
                  if constexpr (part < kHB) mfma_qk8<false, false, kQScaleRope>(sacc[kb][part], k8[f & 1], qe[part], ksc, bs);
                }
                if constexpr (part == 0 && f + 1 < 2 * kF) {
                  k8[(f + 1) & 1] = load_k8(f + 1);
                  if constexpr (LAT && f + 1 == kF) load_tsc(1);
                }
              }
            } else if constexpr (kExact) {
              // Bound by issue: a fragment's four conversions take about as
              // long as its two MFMAs (8 cycles each against 16), so they are
              // dealt out between the MFMAs of the two fragments before it and
              // neither pipe waits for the other.  Two or more instructions
              // (that slot's second MFMA, the next fragment's conversions)
              // separate the last one from the first MFMA that reads it; where
              // none follow, that MFMA brings its wait states.  Against all
              // four just before the fragment's MFMAs (and their wait states),
              // 128 heads: 64 requests of 1,024 to 4,096 positions 87.5 -> 79.8
              // us per-token, 94.8 -> 89.3 latent rows; 8 x 4 rows of 8,192 to
              // 32,768 positions 224 -> 196 and 252 -> 229 us.
              constexpr int kb = i / kKS, ks = i % kKS;
              bf16x8 ka;
              if constexpr (converts(i)) ka = __builtin_bit_cast(bf16x8, kc[i % 3]);
              else ka = kr[2 * kb + (ks & 1)];
              mfma_qk<ks == 0, converts(i) && !converts(i + 1)>(sacc[kb][0], ka, qf[ks][0]);
              __builtin_amdgcn_sched_barrier(0);
              convert_half(std::integral_constant<int, i + 1>{}, std::integral_constant<int, 1>{});
              __builtin_amdgcn_sched_barrier(0);
              if constexpr (kHB == 2) mfma_qk<ks == 0, false>(sacc[kb][1], ka, qf[ks][1]);
              __builtin_amdgcn_sched_barrier(0);
              convert_half(std::integral_constant<int, i + 2>{}, std::integral_constant<int, 0>{});
              if constexpr (i + 1 + kKPre < 36) {
                constexpr int n = i + 1 + kKPre;
                if constexpr (!converts(n)) kr[2 * (n / kKS) + (n & 1)] = load_kr(n / kKS, n & 1);
                else kf[n % kKPre] = load_kf(n);
              }
            } else {
              constexpr int kb = i / kKS, ks = i % kKS;
              const bf16x8 ka = kf[i % kKPre];
              if constexpr (i + kKPre < 36) kf[i % kKPre] = load_kf(i + kKPre);
#pragma unroll
              for (int x = 0; x < kHB; ++x) mfma_qk<ks == 0, false>(sacc[kb][x], ka, qf[ks][x]);
            }
            stream1_rest(ic);
            __builtin_amdgcn_sched_barrier(0);
          });
        } else {
          if constexpr (kPV) deferred();
          static_for<kSlots1>([&](auto ic) { stream1_rest(ic); });
        }

        // ---- stream 2: the PV MFMAs of step j-1 (all but column block 7)
        // with the rest of the softmax, after kLead of them (the QK chains
        // drain meanwhile), and the look-up of the step staged next
        constexpr int kLead = kPV ? (NB == 8 ? 8 : 4) : 0;
        constexpr int kN2 = kPV ? kNPV - NB : 0;
        constexpr int kS2 = kN2 - NB / 2 - kLead;  // softmax slots: P is written half a column block before the end
        const int jn = min(j + kDist + 1, nsteps - 1);
        int jphys = 0;
        auto look_up = [&](int stage) {
          if (kPFM == 2) return;
          if constexpr (TOPK) {
            if (stage == 0) {
              next_row = lane_row(jn);
              next_srow = scale_row(jn);
            }
          } else {
            if (stage == 0) jphys = page_of(jn);
            else next = step_src(jn, jphys);
          }
        };
        if (qk_on) {
          if constexpr (kPV) {
            static_for<kN2>([&](auto kc) {
              constexpr int k = decltype(kc)::value;
              pv_slot(kc);
              if constexpr (k == kLead - 1) {
                // the last MFMA results' 12 wait states, of which the lead MFMAs count kLead
                if constexpr (kLead == 8) asm volatile("s_nop 3");
                else asm volatile("s_nop 7");
                if constexpr (kP1 == 0) finish_scores(0);
                finish_scores(1);
              }
              if constexpr (k >= kLead)
                softmax_slot(std::integral_constant<int, kP1>{}, std::integral_constant<int, kPairs>{},
                             std::integral_constant<int, k - kLead>{}, std::integral_constant<int, kS2>{});
              if constexpr (k == kN2 / 2) look_up(0);
              if constexpr (k == kN2 - 2) look_up(1);
              __builtin_amdgcn_sched_barrier(0);
            });
          } else {
            load_sc();
            asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3");
            finish_scores(0);
            finish_scores(1);
            // first step of the pass: its largest score is the reference (a
            // restarted pass already has one)
#pragma unroll
            for (int i = 0; i < kHB; ++i) {
              if (m_ref[i] == -INFINITY) {
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                  for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sacc[kb][i][r] * c2v[i]);
                m_ref[i] = head_max(mx);
              }
            }
            softmax_slot(std::integral_constant<int, 0>{}, std::integral_constant<int, kPairs>{},
                         std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
            look_up(0);
            look_up(1);
          }
#pragma unroll
          for (int i = 0; i < kHB; ++i) {
            l_exact[i] += pexact[i];
            if constexpr (!(FP8 && !LAT)) l_run[i] += psum[i];
          }
        } else {
          look_up(0);
          look_up(1);
          static_for<kN2>([&](auto kc) {
            pv_slot(kc);
            __builtin_amdgcn_sched_barrier(0);
          });
        }
        pv_slot(std::integral_constant<int, 7 * NB>{});  // (converts column block 7's V, carried past the barrier)
        const uint32_t oldest = ring[0];
#pragma unroll
        for (int i = 0; i + 1 < kSlots; ++i) ring[i] = ring[i + 1];
        ring[kSlots - 1] = oldest;
      };

      iteration(0, std::false_type{}, std::integral_constant<int, 0>{});
      int j = 1;
      for (; j + kDist < nsteps; ++j) iteration(j, std::true_type{}, std::integral_constant<int, 1>{});
      for (; j < nsteps; ++j) iteration(j, std::true_type{}, std::integral_constant<int, 2>{});
      // PV of the last step, after what the step before it carried
      lds_barrier();
      {
        const uint8_t LDS_AS* vbuf = sm + ring[0];
        const uint8_t LDS_AS* p_last = p_lds + kPBytes * ((nsteps - 1) & 1);
        FragRaw<FP8> vf[3];
        vf[0] = load_v_raw<FP8>(vbuf, vbase, 0);
        vf[1] = load_v_raw<FP8>(vbuf, vbase, 1);
#pragma unroll
        for (int hb = 0; hb < NB; ++hb) mfma_pv_in_place<NB == 8>(o[7][hb], d_v, pf[hb]);
        if constexpr (NB == 8) asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
        u32x4 psc;
        const uint32_t ln = fresh_lane();
        if constexpr (LAT) psc = load_p_scales(vbuf + L::kScaleT, ln >> 4, wave);
#pragma unroll
        for (int hb = 0; hb < NB; ++hb) {
          pf[hb] = *(const bf16x8 LDS_AS*)(p_last + 1024 * hb + 16 * ln);
          if constexpr (LAT) pf[hb] = scale_p(pf[hb], psc);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (c + 2 < 8) vf[(c + 2) % 3] = load_v_raw<FP8>(vbuf, vbase, c + 2);
          const bf16x8 v = frag_bf16<FP8>(vf[c % 3]);
#pragma unroll
          for (int hb = 0; hb < NB; ++hb) o[c][hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pf[hb], o[c][hb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      bool over = false;
#pragma unroll
      for (int i = 0; i < kHB; ++i) {
        const float mt_max = head_max(tmax[i]);
        // (should the pass be redone: from the unit's true max)
        m_init[i] = m_ref[i] + mt_max;
        over = over || mt_max > 64.0f;
      }
      // Every wave votes in the P buffer the last step did not use: the last
      // PV reads only the other one.  It is written next by the P of the
      // first step of a second pass, behind that step's barrier, so every
      // wave has read the votes by then.
      int32_t LDS_AS* votes = (int32_t LDS_AS*)(p_lds + kPBytes * (nsteps & 1));
      if (fresh_lane() == 0) votes[wave] = __builtin_amdgcn_ballot_w64(over) ? 1 : 0;
      __syncthreads();
      const bool restart = (votes[0] | votes[1] | votes[2] | votes[3]) != 0;
      // the second pass starts from the unit's true max, so it never
      // overflows; it is the last one in any case
      if (!restart || pass > 0) break;
    }  // pass

    // ---- the next unit's query, page ids and first steps.  Every wave is
    // past its last PV (the vote barrier), so the ring is free; the epilogue
    // below stages in LDS these steps do not use.  Steps 0 and 1 are the two
    // halves of the unit's first page.
    pre = false;
    if constexpr (kOverlap) {
      if (nxt.x >= 0) {
        pages = load_pages(N, 0);
        load_q(N.tile);
#pragma unroll
        for (int j = 0; j < kDist; ++j)
          if (j < N.nsteps) issue_step<FP8, LAT, NT, TOPK>(step_src(j, n_phys), lds0 + slot_off(j), wdst, wave);
        pre = true;
      }
    }

    // ---- epilogue: normalise and store
    if (qk_on) {
      const int ln = (int)fresh_lane(), g = ln >> 4;
#pragma unroll
      for (int i = 0; i < kHB; ++i) {
        // normaliser: sum of the weights as applied (rounded); LSE: exact sum
        const float l_ex = head_sum(l_exact[i]);
        const float l_tot = (FP8 && !LAT) ? l_ex : head_sum(l_run[i]);
        const float lse_nat = (m_ref[i] + __log2f(l_ex)) * 0.6931471805599453f;
        const int head = 16 * (kHB * wave + i) + (ln & 15);
        // the reciprocal of each head's normaliser (1 ulp), by the wave that owns the head
        if (g == 0) l_lds[head] = __builtin_amdgcn_rcpf(l_tot);
        if (g == 0 && head < a.H) {
          if (slot < 0) {
            if (a.lse) a.lse[(size_t)tile * a.H + head] = lse_nat;
          } else {
            a.ws.part_lse[(size_t)slot * a.H + head] = lse_nat;
          }
        }
      }
    }
    __syncthreads();
    // Each head block of the wave's 128 columns is scaled in registers,
    // packed to 16 bits and passed through 4 KB of LDS of the wave's own, so
    // that the stores write 256-byte row pieces instead of the accumulators'
    // 8-byte ones: 16 heads x 256 B, 16-byte chunks XOR-permuted by head so
    // that writes (8 B of 16 heads) and reads (a row per 16 lanes) are free of
    // bank conflicts; the wave's LDS ops complete in order, so no barrier is
    // needed.  (The epilogue is bound by its stores:
    // every worker writes its 128 KB at about the same time.)
    // NT: the stores are non-temporal too.  Lines left dirty in the L2 are
    // written back at the kernel's end, after the last worker; streamed
    // stores shorten that drain, at the price of the combine reading the
    // partials from memory instead of the L2 (measured on the
    // one-row-per-request workloads: the kernel 2-7 us shorter, the combine
    // 2 us longer).
    // Accumulator lane: head 16hb + n16, columns 16c + 4g + [0, 4).
    {
      // (laundered, so that the addresses below are not hoisted out of the
      // unit loop and spilled)
      const uint32_t ll = fresh_lane(), nl = ll & 15, gl = ll >> 4;
      uint8_t LDS_AS* stage = sm + kStageOff + 1024 + 4096 * wave;
      const bool split = slot >= 0;
      uint16_t* obase = (split ? a.ws.part_half + (size_t)slot * a.H * kDimV : (uint16_t*)a.out + (size_t)tile * a.H * kDimV) +
                        128 * wave + 8 * (ll & 15);
      static_for<NB>([&](auto hbc) {
        constexpr int hb = decltype(hbc)::value;
        if (16 * hb >= a.H) return;  // uniform: H is a multiple of 16
        float rl = l_lds[16 * hb + nl];
        if (split) {
          // the (slot, head) quarter's scale, and its exponent in byte `wave` of the head's word
          float m = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(o[c][hb][r]));
          const uint32_t e = partial_exponent(head_max(m) * rl);
          rl *= __builtin_bit_cast(float, (127u - e) << 23);
          if (gl == 0) ((uint8_t*)(a.ws.part_exp + (size_t)slot * a.H + 16 * hb + nl))[wave] = (uint8_t)e;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const f32x4 v = o[c][hb] * rl;
          u32x2 w;
          if (split) w = (u32x2){pack_f16x2(v[0], v[1]), pack_f16x2(v[2], v[3])};
          else w = (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
          *(u32x2 LDS_AS*)(stage + 256 * nl + (((2 * c + (gl >> 1)) ^ nl) * 16) + 8 * (gl & 1)) = w;
        }
        u32x4 rows[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t row = 4 * k + (ll >> 4);
          rows[k] = *(const u32x4 LDS_AS*)(stage + 256 * row + (((ll & 15) ^ row) * 16));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          u32x4* dst = (u32x4*)(obase + (size_t)(16 * hb + 4 * k + (ll >> 4)) * kDimV);
          if constexpr (NT) __builtin_nontemporal_store(rows[k], dst);
          else *dst = rows[k];
        }
      });
    }
    cur = nxt;
    nxt = nxt2;
  }
}

// The kernel for a call's head count.  Up to 64 (32) heads only 4 (2) head
// blocks are multiplied, on waves that own one each, instead of 8 with
// padding (measured: 64 heads over bf16, three layers, 115 -> 99 us; 16 heads
// over fp8, 219 -> 176 us; exact QK, 64 heads over fp8, 82.6 -> 65.4 us, 16
// heads over latent rows, 305 -> 200 us).
// NT (non-temporal cache-row loads) when every request has one query row:
// then no two tiles read the same pages.
template <bool FP8, bool TOPK, bool LAT, bool Q8>
inline void launch_attend_heads(const AttendLaunch& a, int32_t workers, hipStream_t s) {
  auto go = [&](auto nb) {
    constexpr int NB = decltype(nb)::value;
    if (a.q_chunk == 1)
      hipLaunchKernelGGL((attend_kernel<FP8, TOPK, LAT, true, Q8, NB>), dim3(workers), dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((attend_kernel<FP8, TOPK, LAT, false, Q8, NB>), dim3(workers), dim3(256), 0, s, a);
  };
  if (a.H > 64) go(std::integral_constant<int, 8>{});
  else if (a.H > 32) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 2>{});
}

}  // namespace splash
