// Shared pieces of the matrix-core (MFMA) scan kernels for gfx950.
//
// Tiling.  The K rows of the state are independent recurrences that share only
// W, v_t and f_t (row i of H W + k v^T needs row i of H and the scalar k_i;
// this is the structure Theorem 1 of the paper uses).  A workgroup therefore
// owns RB blocks of 16 rows of one (batch, head) state and all V columns; each
// wavefront owns one 16 x 16 tile: lane l holds rows 4*(l/16)+r (r = 0..3) of
// column l%16 -- the accumulator layout of the 16x16 MFMA family.  A state of
// K rows is split over P = K/(16*RB) workgroups so that small batches still
// fill 256 CUs; sums over rows (y, dv, df, dW) are finished across workgroups
// in a fixed order by small epilogue kernels.
//
// Operand precision.  Gradients of this recurrence at T = 4096 are extremely
// sensitive to the forward trajectory (the backward amplifies a trajectory
// error of 2e-4 into gradient errors of several percent), so the state enters
// its contraction as an fp16 pair (hi, lo) with hi + lo = H' to ~21 bits.  The
// pair occupies two k-slots of the 16x16x32 MFMA (or two of its rows) and the W
// fragment holds each row of W twice.  All other matrix-core operands (dS, the stash
// copies of H and Z, q, k, v, dy) are single fp16 values.
//
// Scaled state.  tanh(x) = 1 - 2/(1 + 2^(c x)) with c = 2*log2(e).  The kernels
// carry H' = c*H in fp32 registers, so the fp16 operand cvt(H') makes the MFMA
// produce c*(H W) directly and the exponent needs no multiply; results that
// leave the chip (y, dq, dW, df, H_T, checkpoints) are scaled back by 1/c.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace m2rnn {

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef unsigned short bf16_raw;

constexpr float kC = 2.8853900817779268f;  // 2*log2(e)
constexpr float kInvC = 0.34657359027997264f;
constexpr int kLdsLimit = 160 * 1024;

__device__ __forceinline__ float bf16_to_f32(bf16_raw x) {
  return __builtin_bit_cast(float, (uint32_t)x << 16);
}
// round to nearest even; NaN stays NaN
__device__ __forceinline__ bf16_raw f32_to_bf16(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_raw)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_raw)(u >> 16);
}

// Two elements H' -> their fp16 (hi, lo) parts as two packed registers, {hi0, hi1} and {lo0, lo1}:
// hi is H' rounded towards zero to 11 significant bits, lo = fp16(H' - hi).  Four instructions for
// two elements: the mixed-precision FMA subtracts the fp16 hi in fp32, so hi needs no fp32 copy of
// its own.  (v_fma_mixlo/mixhi_f16 would round to fp16 in the same instruction, but take 8.3 cycles
// a wave where v_fma_mix_f32 and the packing conversion take 4.3.)
__device__ __forceinline__ u2_t split2_hi_lo(float h0, float h1) {
  typedef float f2_t __attribute__((ext_vector_type(2)));
  const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(h0, h1));
  float l0, l1;
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l0) : "v"(hi), "v"(h0));
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(l1) : "v"(hi), "v"(h1));
  const f2_t lo = {l0, l1};
  return u2_t{hi, __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, h2_t))};
}
// Four elements of a lane as the operand of a 16x16x32 MFMA that contracts 16 columns, hi and lo
// parts both: slots {hi0, hi1, lo0, lo1, hi2, hi3, lo2, lo3}.  Slot e meets W's row pair_row(e).
__device__ __forceinline__ u4_t split4_hi_lo(const float (&h)[4]) {
  const u2_t a = split2_hi_lo(h[0], h[1]), b = split2_hi_lo(h[2], h[3]);
  return u4_t{a.x, a.y, b.x, b.y};
}
__device__ __forceinline__ constexpr int pair_row(int e) { return 2 * (e >> 2) + (e & 1); }
// the first of the two slots that row r takes (the other one is 2 further)
__device__ __forceinline__ constexpr int pair_slot(int r) { return r + (r & 2); }

// One state element through the non-linearity and the gate of the recurrence equations, on the
// scaled state:  H' <- f H' + gp tanh(s),  gp = c (1 - f),  sp = c s = 2 log2(e) s.
//     tanh(s) = sign(s) (1 - e) / (1 + e),   e = 2^-|sp|  in (0, 1].
// Why this form and not 1 - 2 / (1 + 2^sp): the forward trajectory of this recurrence can be
// transiently chaotic (units whose transition matrix has gain above one amplify a
// perturbation of the state by 10^4 .. 10^6 over a few hundred steps, and the backward
// gradient of such a unit follows the trajectory), so the ABSOLUTE error of tanh near zero
// decides how far such units drift from an exact evaluation.  1 - 2/(1+e) carries the
// rounding of exp2, of the sum and of the reciprocal as absolute errors (measured 4.4e-8
// rms); here 1 - e is exact for e in [1/2, 1] and the reciprocal's error is relative to the
// result, which leaves half an ulp of e in [1/2, 1) (measured 0.7e-8 rms).  e <= 1 also
// cannot overflow, whatever the pre-activation.  Two more vector instructions per element.
__device__ __forceinline__ float gate_tanh_step(float f, float gp, float h, float sp) {
  const float e = __builtin_amdgcn_exp2f(-__builtin_fabsf(sp));
  const float rr = __builtin_amdgcn_rcpf(1.f + e);
  const float n = fmaf(-gp, e, gp);                      // gp (1 - e) >= 0
  const float ns = __builtin_copysignf(n, sp);
  return fmaf(ns, rr, f * h);
}

// dS = G ((1-f) - w) as an fp16 operand, from ug = -w = -(1-f) Z^2 in fp16: only the small term w
// is fp16, the leading term 1 - f and G stay fp32.  (With the whole factor (1-f)(1 - Z^2) in fp16 the
// rounded factor is biased: Z^2 is mostly below one fp16 ulp of 1 - f, so the factor rounds up to
// fp16(1 - f) more often than down, by 2.4e-5 on average; compounded through the W path of the
// Jacobian that is +1 % on a gradient carried over 4096 steps.)  The factor does not depend on G, so
// it is off the chain of the carried gradient; v_fma_mixlo/mixhi_f16, which would form and round
// (1-f) G - w G at once, take 8.3 cycles a wave against 4.3 here.
__device__ __forceinline__ h4_t ds_of(const float (&G)[4], h4_t ug, float gm) {
  typedef float f4v_t __attribute__((ext_vector_type(4)));
  const u2_t u = __builtin_bit_cast(u2_t, ug);
  const uint32_t u0 = u.x, u1 = u.y;
  float t[4];
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(t[0]) : "v"(u0), "v"(gm));
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t[1]) : "v"(u0), "v"(gm));
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(t[2]) : "v"(u1), "v"(gm));
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t[3]) : "v"(u1), "v"(gm));
  const f4v_t d = {G[0] * t[0], G[1] * t[1], G[2] * t[2], G[3] * t[3]};
  return __builtin_convertvector(d, h4_t);
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains
// the vector-memory counter, i.e. it would wait for every global load and store
// in flight (the staged q/k/v prefetch, the per-step y / dq / dk stores) at each
// of the one or two barriers a scan step needs.  Nothing is exchanged between
// waves through global memory inside these kernels, so only LDS must be settled.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS access as base register + compile-time byte offset (the offset lands in the
// instruction's 16-bit immediate).  `lchar` pointers are 32-bit LDS addresses.
typedef __attribute__((address_space(3))) char lchar;
template <typename T>
__device__ __forceinline__ T lds_ld(const lchar *p, int off) {
  return *(const __attribute__((address_space(3))) T *)(p + off);
}
template <typename T>
__device__ __forceinline__ void lds_st(lchar *p, int off, T v) {
  *(__attribute__((address_space(3))) T *)(p + off) = v;
}

__device__ __forceinline__ f4_t mfma_k32(h8_t a, h8_t b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4_t mfma_k16(h4_t a, h4_t b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

// Reads a just-finished MFMA chain's result into vector registers HERE, in the
// basic block that issued the MFMAs.  Without it the compiler may sink the first
// read of the result below a conditional block that follows the chain
// (MFMA; if (...) {long block}; use): the wait states an MFMA result needs before
// a vector-ALU read are then counted along the long path only, and the waves
// that skip the block read the accumulator too early (seen as wrong gradients).
// settle() alone only marks the spot: where a conditional block follows the chain, the first
// real consumer must also sit (and be pinned) in front of that block, as the backward's
// carry update does.  Guarded by tests/test_gpu_instantiations.py, which runs every tiling.
__device__ __forceinline__ void settle(f4_t &d) { asm volatile("" : "+v"(d)); }

// Maximum of a NON-NEGATIVE float over aligned groups of G = 2, 4, 8, 16, 32 or 64 consecutive
// lanes (result in every lane of the group), without LDS traffic: DPP steps inside each row
// of 16 lanes, then the rows through scalar registers.  Non-negative floats order like
// their bit patterns, so the maxima are taken on integers.
template <int G>
__device__ __forceinline__ float group_max_nonneg(float x) {
  static_assert(G == 2 || G == 4 || G == 8 || G == 16 || G == 32 || G == 64, "group size");
  int v = __builtin_bit_cast(int, x);
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  if constexpr (G > 2)
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  if constexpr (G > 4)
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  if constexpr (G > 8)
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false));  // row_mirror
  if constexpr (G > 16) {
    const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    if constexpr (G == 64)
      v = max(max(r0, r1), max(r2, r3));
    else
      v = (threadIdx.x & 32) ? max(r2, r3) : max(r0, r1);
  }
  return __builtin_bit_cast(float, v);
}
// Sum over each group of 16 lanes, in all of them.
__device__ __forceinline__ float row_sum(float x) {
  auto add = [](float y, int moved) { return y + __builtin_bit_cast(float, moved); };
  x = add(x, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // lane xor 1
  x = add(x, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // lane xor 2
  x = add(x, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xF, 0xF, true));  // rotated by 4
  x = add(x, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xF, 0xF, true));  // rotated by 8
  return x;
}
// eight bf16 values (one 16-byte load) widened to fp32
__device__ __forceinline__ void bf16x8_to_f32(const u4_t &w, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __builtin_bit_cast(float, w[i] << 16);
    x[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xFFFF0000u);
  }
}
// 2^e with e clamped to the normal range
__device__ __forceinline__ float pow2i(int e) {
  e = e < -126 ? -126 : (e > 127 ? 127 : e);
  return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23);
}
// floor(log2 x) of a positive finite float (subnormals count as 2^-127)
__device__ __forceinline__ int ilog2f(float x) {
  return (int)((__builtin_bit_cast(uint32_t, x) >> 23) & 255u) - 127;
}

// Sum of a power of two of terms as a binary tree of neighbours.  A row block's readout is summed
// this way inside a workgroup and over the workgroups of a state, so that y has the same bits
// however a state is split.
template <int M>
__device__ __forceinline__ f4_t pairwise_sum(const f4_t (&x)[M]) {
  if constexpr (M == 1) {
    return x[0];
  } else {
    f4_t y[M / 2];
#pragma unroll
    for (int i = 0; i < M / 2; ++i) y[i] = x[2 * i] + x[2 * i + 1];
    return pairwise_sum(y);
  }
}

template <int K_, int V_, int RB_>
struct Tile {
  static constexpr int K = K_, V = V_, RB = RB_;
  static constexpr int CT = V / 16;            // column tiles = waves per row block
  static constexpr int WAVES = RB * CT;
  static constexpr int THREADS = WAVES * 64;
  static constexpr int P = K / (16 * RB);      // workgroups per (b, n) state
  static constexpr int ROWS = RB * 16;         // state rows per workgroup
  static constexpr bool X32 = (V >= 32);       // 16x16x32 MFMA for the V-contraction
  static constexpr int KS = X32 ? V / 32 : 1;  // MFMAs per state contraction
  static constexpr int LDH = V + 8;            // halfs per row of a row-major fp16 exchange buffer
  static constexpr int LDH2 = 2 * V + 8;       // ... of a (hi, lo) pair exchange buffer
  static_assert(K % (16 * RB) == 0 && V % 16 == 0 && WAVES <= 16, "bad tile");
};

// Operand fragment of the V-contraction (8 halfs for the k=32 MFMA, 4 for k=16).
template <bool X32> struct Frag { typedef h8_t type; };
template <> struct Frag<false> { typedef h4_t type; };

// Fragment read through the transposing LDS load of gfx950 (ds_read_b64_tr_b16).  Within each
// group of 16 lanes the 16 x 8 bytes that the lanes address are taken as 64 consecutive
// fp16 values and lane d receives values d, 16 + d, 32 + d, 48 + d of them.  With the tile
// stored as 8-byte items (column j, rows 4 i .. 4 i + 3) -- which is what a lane of the
// accumulator layout holds -- at byte offset 32 j + 8 i, lane d addressing item
// (column c0 + d / 4, rows 4 (d % 4) ..) receives row d, columns c0 .. c0 + 3: the A operand of
// the 16-row MFMAs, with no scattered 2-byte writes and no padded rows.
__device__ __forceinline__ h4_t lds_ld_tr(const lchar *p, int off) {
  typedef short s4_t __attribute__((ext_vector_type(4)));
  const s4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4_t *)(p + off));
  return __builtin_bit_cast(h4_t, v);
}
// Where the four items of a column sit inside the column's 32 bytes, and where a group of
// four columns sits inside its 256-byte pair, is free (every lane of the transposing load
// supplies its own address).  Item (column j, rows 4 i ..) goes to
// a = 32 j + 8 ((i + j / 4) mod 4) and then to a xor (128 if bit 8 of a is set): the items a
// lane group reads are still 128 contiguous bytes, but the four lane groups and the two
// halves of a k = 32 fragment start on different banks.  In the plain order (32 j + 8 i) a
// third of the LDS-active cycles of the backward are bank conflicts; placed like this, 1 %.
// That is worth 6.5 % of the backward on the 128-wide tile (rotation alone 3.5 %); on the
// 64-wide tiles, where the LDS is not what the step waits for, the time does not change.
__device__ __forceinline__ int xch_item_off(int j, int i) {
  const int a = 32 * j + 8 * ((i + (j >> 2)) & 3);
  return a ^ ((a >> 1) & 128);
}
// Per-lane base offsets of a fragment read: lane (d, g) = (lane % 16, lane / 16) reads, for
// the first half of its FE columns c0 = FE g .., item (column c0 + d / 4, rows 4 (d % 4) ..); the
// second half (k = 32 fragments only) is the next group of 4 columns.
template <bool X32>
__device__ __forceinline__ int xch_frag_off(int d, int g, int half) {
  constexpr int FE = X32 ? 8 : 4;
  const int c0 = FE * g + 4 * half;
  return xch_item_off(c0 + (d >> 2), d & 3);
}
template <bool X32>
__device__ __forceinline__ typename Frag<X32>::type lds_ld_frag_tr(const lchar *p0, const lchar *p1, int off) {
  if constexpr (X32) {
    const h4_t lo = lds_ld_tr(p0, off), hi = lds_ld_tr(p1, off);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  } else {
    return lds_ld_tr(p0, off);
  }
}

// blockIdx -> (unit, part).  Workgroups are dealt round-robin to the 8 XCDs, so
// all P parts of a (b, n) state get ids that are equal mod 8: they then share
// one XCD's L2 for v_t, f_t and W.  Returns false for padding blocks.
template <int P>
__device__ __forceinline__ bool map_block(int units, int &unit, int &part) {
  const int x = blockIdx.x;
  const int xcd = x & 7, r = x >> 3;
  part = r % P;
  unit = xcd + 8 * (r / P);
  return unit < units;
}
inline int grid_blocks(int units, int P) { return 8 * P * ((units + 7) / 8); }


// (K, V, RB) tilings that are instantiated
#define M2RNN_TILE_CASES(X)                                                                      \
  X(64, 64, 2) X(64, 64, 1) X(128, 128, 1) X(32, 32, 2) X(32, 32, 1) X(16, 16, 1) X(64, 16, 1)

// (K, V, RB) splits of the forward on 8-row blocks, per shape in increasing RB, and the forms that a launch
// can take on them: waves that share a row's columns (C), waves with whole rows (R; few square states)
#define M2RNN_HALF_CASES(X)  /* K, V, RB, C, R */                                                \
  X(64, 64, 1, 1, 1) X(64, 64, 2, 1, 1) X(64, 64, 4, 1, 0) X(128, 128, 1, 1, 0) X(128, 128, 2, 1, 0) \
  X(32, 32, 1, 0, 1) X(32, 32, 2, 1, 1) X(32, 32, 4, 1, 1) X(16, 16, 1, 1, 0) X(16, 16, 2, 1, 0) \
  X(64, 16, 1, 1, 0) X(64, 16, 2, 1, 0) X(64, 16, 4, 1, 0) X(64, 16, 8, 1, 0) X(32, 16, 1, 1, 0) \
  X(32, 16, 2, 1, 0) X(32, 16, 4, 1, 0) X(64, 32, 1, 1, 0) X(64, 32, 2, 1, 0) X(64, 32, 4, 1, 0) \
  X(64, 32, 8, 1, 0)

// (K, V) shapes of the register-resident (one wave per row block) kernels
#define M2RNN_ROWWAVE_CASES(X)                                                                  \
  X(16, 16) X(32, 16) X(64, 16) X(128, 16) X(16, 32) X(32, 32) X(64, 32) X(128, 32) X(16, 64)   \
  X(32, 64) X(64, 64) X(128, 64)

}  // namespace m2rnn
