// fp32 scan kernels for V <= 64 on the fp32 matrix instructions: every operand, product and sum
// is fp32 (the 1e-5 parity class), the state stays in registers from step to step, and no wave
// waits for another one inside a chunk of steps.
//
// Which instruction, and why.  Row i of H W needs only row i of H, so what a wave must have at
// hand for its rows is the whole of each row, in every lane that holds one of the row's columns.
// v_mfma_f32_4x4x1 computes 16 independent 4 x 4 blocks and can broadcast one block's A operand
// to a group of blocks (cbsz / abid): with A = 4 rows x 1 column of the state, broadcast, and
// B = that row of W spread over the V columns, V such instructions are the product of 4 rows
// with W, and the operand never leaves the registers.  One wave holds 4 rows x 64 columns,
// 8 x 32 or 16 x 16: RW = 256 / V rows.  The rate (64 multiply-adds per clock and SIMD) is that of the
// 16x16x4 form, and twice that of the vector ALU; the 16x16x4 form would spread a row over
// V / 16 waves, with an exchange through LDS and a barrier in every step.
// Layouts.  Accumulator ("D"): lane 4 b + n holds column 4 (b mod V/4) + n, register m row m of
// the lane's group of 4 rows.  A operand: lane 4 b + m holds row m, register j column 4 b + j.
// The two differ by a 4 x 4 transposition inside each group of four lanes (quad_transpose).
// Split (V = 32): both halves of a wave hold the SAME four rows and contract 16 of the 32 columns
// each, half of the matrix instructions; the halves' sums meet by a lane swap that leaves two
// of the four rows to each, half of the vector instructions.  Twice as many waves take part, which
// pays as long as SIMDs are free (split_pays).  A half contracts the columns of two of the four chains
// (columns 4 i, 4 i + 1 or 4 i + 2, 4 i + 3), so that every sum has the order of the whole rows: states,
// checkpoints, y and carried gradients have the same bits in both forms, whatever room a call has.
//
// Measured against the vector-ALU kernels that these replace (one workgroup per state, state and
// W in LDS, three barriers per step): B = 4, N = 8, K = V = 32, T = 512 forward 1.13 -> 0.245 ms,
// backward 4.34 -> 0.59 ms, and with split rows 0.169 and 0.424.  What bounds it there: waves alone on
// their SIMD, each a chain of some 800 cycles per step (forward; 1100 with four rows per lane: 86 vector
// instructions at 5.5 cycles for 133, 131 cycles of matrix instructions for 262).
#include "m2rnn_io.hpp"
#include "m2rnn_kernels.hpp"

#include <type_traits>
#include <utility>

namespace m2rnn {
namespace {

constexpr int TB = 16;  // steps per staged block (forward), per on-chip stash (backward)
typedef float f2_t __attribute__((ext_vector_type(2)));

template <int K_, int V_, int S_>
struct QuadOf {
  static constexpr int K = K_, V = V_, S = S_;         // S: lanes per column of a row group
  static constexpr int E = 4 / S;                      // rows per lane
  static constexpr int CB = V / 4 / S;                 // 4-column blocks that a lane's contraction runs over
  static constexpr int GR = 64 / (V * S);              // row groups per wave
  static constexpr int RW = 4 * GR;                    // rows per wave
  static constexpr int CBSZ = CB == 16 ? 4 : (CB == 8 ? 3 : 2);
  static constexpr int NWU = K / RW;                   // waves per state
  static constexpr int NW = NWU < 4 ? NWU : 4;         // waves per workgroup
  static constexpr int P = NWU / NW;                   // workgroups per state
  static constexpr int ROWS = NW * RW;
  static constexpr int THREADS = NW * 64;
  static constexpr int NQ = TB * ROWS / THREADS;       // staged values per thread: q, k ...
  static constexpr int NV = (TB * V + THREADS - 1) / THREADS;  // ... v, dy
  typedef float rows_t __attribute__((ext_vector_type(E)));  // a lane's elements
  static_assert(NWU >= 1 && NWU % NW == 0 && (TB * ROWS) % THREADS == 0, "quad tile");
  static_assert(S == 1 || (S == 2 && V == 32 && K <= 32), "split");
};
template <int K_, int V_>
struct Quad : QuadOf<K_, V_, 1> {};
// The shapes that have split rows: those whose whole rows are one workgroup per state.  (64 x 32 and 128 x 32,
// two and four of them, would gain as much, 16 states, T = 512 forward 232.5 -> 169.4 and 235.1 -> 174.0 us,
// backward 589 -> 425 and 604 -> 433, with four and eight parts and twice the room; they are not built.)
constexpr bool has_split(int K, int V) { return V == 32 && K <= 32; }
template <int K_, int V_>
struct Split : QuadOf<K_, V_, 2> {};

// tanh.  Below 1 an odd polynomial x + x^3 p(x^2) (a minimax fit of (tanh x - x) / x^3 with every
// coefficient a float, error 4.7e-9 relative to tanh); from 1 on 1 - 2 / (1 + e^(2 |x|)), whose
// subtrahend is below a quarter.  Branch-free, 17 issue slots.  Error, max / rms ulp, here and of the library's
// tanhf: below 0.55 0.77 / 0.30 (0.78 / 0.30), 0.55 to 1 0.88 / 0.32 (1.41 / 0.47), 1 to
// 1.5 1.33 / 0.37 (1.00 / 0.33), 1.5 to 2 0.93 / 0.31 (0.66 / 0.29), beyond 0.66 / 0.29 (0.57 / 0.29).
// (With the argument in two parts and a Newton step the second form is as near as tanhf from 1 on too; the
// state's error does not change, and a state that saturates pays: B 4, N 8, T 512, W of gain one, forward 246 ->
// 292 us, although only waves that need it took it.)
// Infinities give +-1; a NaN goes through the polynomial and stays one.
__device__ __forceinline__ constexpr float tanh_c(int i) {
  constexpr float c[7] = {-0.33333295583724976f, 0.13332346081733704f,  -0.05387984961271286f, 0.02148670330643654f,
                          -0.007946079596877098f, 0.0023012934252619743f, -0.0003584200458135456f};
  return c[i];
}
__device__ __forceinline__ float tanh_f32(float x) {
  const float x2 = x * x;
  float p = tanh_c(6);
#pragma unroll
  for (int i = 5; i >= 0; --i) p = fmaf(x2, p, tanh_c(i));
  const float near = fmaf(x * x2, p, x);
  const float e = __builtin_amdgcn_exp2f(2.885390081777927f * __builtin_fabsf(x));
  const float far = __builtin_copysignf(fmaf(-2.f, __builtin_amdgcn_rcpf(1.f + e), 1.f), x);
  return __builtin_fabsf(x) >= 1.f ? far : near;
}
// The same of all of a lane's elements at once, operation by operation: a lone wave issues an instruction
// every 5.5 cycles, but one that needs the result of the one before it after 8.6.
template <typename X>
__device__ __forceinline__ X tanh_f32(X x) {
  constexpr int E = sizeof(X) / 4;
  X e, p, near, far;
  const X x2 = x * x, x3 = x * x2;
#pragma unroll
  for (int m = 0; m < E; ++m) {
    e[m] = __builtin_amdgcn_exp2f(2.885390081777927f * __builtin_fabsf(x[m]));
    p[m] = tanh_c(6);
  }
#pragma unroll
  for (int i = 5; i >= 0; --i)
#pragma unroll
    for (int m = 0; m < E; ++m) p[m] = fmaf(x2[m], p[m], tanh_c(i));
#pragma unroll
  for (int m = 0; m < E; ++m) {
    near[m] = fmaf(x3[m], p[m], x[m]);
    far[m] = __builtin_copysignf(fmaf(-2.f, __builtin_amdgcn_rcpf(1.f + e[m]), 1.f), x[m]);
    p[m] = __builtin_fabsf(x[m]) >= 1.f ? far[m] : near[m];
  }
  return p;
}

template <int CTRL>
__device__ __forceinline__ float quad_perm(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// y[j] in lane m of a quad = x[m] of lane j: registers and lanes swapped one index bit at a time.
// (Every lane runs the permutations, the selects come after: a permutation inside the select's
// arms would run with part of the lanes switched off, and read nothing from those.)
__device__ __forceinline__ f4_t quad_transpose(f4_t x, bool odd, bool high) {
  const float p0 = quad_perm<0xB1>(x[0]), p1 = quad_perm<0xB1>(x[1]);  // lane xor 1
  const float p2 = quad_perm<0xB1>(x[2]), p3 = quad_perm<0xB1>(x[3]);
  const float a0 = odd ? p1 : x[0], a1 = odd ? x[1] : p0, a2 = odd ? p3 : x[2], a3 = odd ? x[3] : p2;
  const float q0 = quad_perm<0x4E>(a0), q1 = quad_perm<0x4E>(a1);      // lane xor 2
  const float q2 = quad_perm<0x4E>(a2), q3 = quad_perm<0x4E>(a3);
  return f4_t{high ? q2 : a0, high ? q3 : a1, high ? a2 : q0, high ? a3 : q1};
}

// The same out of split rows (registers: rows 2 half, 2 half + 1 of a column): half h gets all four rows
// of the columns that the lanes 16 h .. + 15 of either half hold, in both of its groups of 16 lanes.
__device__ __forceinline__ f4_t quad_transpose(f2_t x, bool odd, bool high) {
  const float p0 = quad_perm<0xB1>(x[0]), p1 = quad_perm<0xB1>(x[1]);
  const float e[2] = {odd ? p1 : x[0], odd ? x[1] : p0};
  float a[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    // groups of 16 lanes 0 1 2 3 -> 0 0 2 2 and 1 1 3 3 -> 0 0 1 1 (rows 0, 1) and 2 2 3 3 (rows 2, 3)
    const uint32_t u = __builtin_bit_cast(uint32_t, e[i]);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const auto t = __builtin_amdgcn_permlane32_swap(r[0], r[1], false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    a[i] = __builtin_bit_cast(float, t0);
    a[2 + i] = __builtin_bit_cast(float, t1);
  }
  const float q0 = quad_perm<0x4E>(a[0]), q1 = quad_perm<0x4E>(a[1]);
  const float q2 = quad_perm<0x4E>(a[2]), q3 = quad_perm<0x4E>(a[3]);
  return f4_t{high ? q2 : a[0], high ? q3 : a[1], high ? a[2] : q0, high ? a[3] : q1};
}

// acc[k mod 4] += (column k of A) x (row k of B) for all k = 4 B0 + j of the blocks B0...: four
// independent chains, because the result of a 4x4x1 is not ready for the next instruction's
// accumulator
template <int CBSZ, int V, int... B0>
__device__ __forceinline__ f4_t contract_blocks(const f4_t &a, const float (&w)[V],
                                                std::integer_sequence<int, B0...>) {
  f4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0, acc2 = acc0, acc3 = acc0;
  (
      [&] {
        acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0], w[4 * B0 + 0], acc0, CBSZ, B0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[1], w[4 * B0 + 1], acc1, CBSZ, B0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[2], w[4 * B0 + 2], acc2, CBSZ, B0, 0);
        acc3 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[3], w[4 * B0 + 3], acc3, CBSZ, B0, 0);
      }(),
      ...);
  return (acc0 + acc1) + (acc2 + acc3);
}
// ... the two of the four chains that a half of a split row group takes
template <int CBSZ, int V, int... B0>
__device__ __forceinline__ f4_t contract_blocks2(const f4_t &a, const float (&w)[V],
                                                 std::integer_sequence<int, B0...>) {
  f4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
  (
      [&] {
        acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0], w[4 * B0 + 0], acc0, CBSZ, B0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[1], w[4 * B0 + 1], acc1, CBSZ, B0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[2], w[4 * B0 + 2], acc0, CBSZ, B0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(a[3], w[4 * B0 + 3], acc1, CBSZ, B0, 0);
      }(),
      ...);
  return acc0 + acc1;
}
// a lane's rows of (rows of A) x W
template <typename Q>
__device__ __forceinline__ typename Q::rows_t contract(const f4_t &a, const float (&w)[4 * Q::CB]) {
  if constexpr (Q::S == 1) {
    return contract_blocks<Q::CBSZ, Q::V>(a, w, std::make_integer_sequence<int, Q::CB>{});
  } else {
    const f4_t x = contract_blocks2<Q::CBSZ, 4 * Q::CB>(a, w, std::make_integer_sequence<int, Q::CB>{});
    // both halves' sums, added as the chains of the whole rows are: rows 0, 1 to the lower half, rows 2, 3 to the upper
    typename Q::rows_t y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float lo = x[i], hi = x[2 + i];
      const auto t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi),
                                                      false, false);
      const uint32_t t0 = t[0], t1 = t[1];
      y[i] = __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1);
    }
    return y;
  }
}
// Pre-activation of a step, H W + k v^T: the outer product joins last, by an FMA on the finished sum.
// (As the start of one of the four chains it is rounded once more, and so is every sum behind it:
// state error against 64 bits, 512 steps, 1.2e-7 for 0.9e-7 at V = 32, 1.4e-7 for 0.9e-7 at 64.)
template <typename Q>
__device__ __forceinline__ typename Q::rows_t preactivation(const f4_t &ha, const float (&w)[4 * Q::CB],
                                                            const typename Q::rows_t &kr, float vj) {
  typename Q::rows_t sp = contract<Q>(ha, w);
#pragma unroll
  for (int m = 0; m < Q::E; ++m) sp[m] = fmaf(kr[m], vj, sp[m]);
  return sp;
}

// Waits for a loaded value here: the first use sits in a loop, where the wait would be repeated
// in every step, and would wait there for the prefetch as well.
template <typename X>
__device__ __forceinline__ void arrived(X &x) { asm volatile("" : "+v"(x)); }

// a lane's elements of a column
template <typename Q>
__device__ __forceinline__ typename Q::rows_t load_rows(const float *p) {
  typename Q::rows_t x;
#pragma unroll
  for (int m = 0; m < Q::E; ++m) x[m] = p[m * Q::V];
  return x;
}

// Per-lane position inside the workgroup's rows
template <typename Q>
struct LanePos {
  int wave, lane, col, row;  // row: first of the lane's E rows inside the workgroup
  int arow, acol, first;     // row of the lane's A operand, and the column from which on it stores it; first column of its contraction
  bool odd, high, second;    // second: of two groups of lanes that hold the same A operand
  __device__ __forceinline__ LanePos() {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane / (Q::V * Q::S), part = lane / Q::V % Q::S;
    first = Q::S == 1 ? 0 : 2 * part;
    col = Q::S == 1 ? lane % Q::V : column(lane & 15) + (lane >> 3 & 2);
    row = wave * Q::RW + 4 * group + Q::E * part;
    arow = wave * Q::RW + 4 * group + (lane & 3);
    second = Q::S > 1 && (lane & 16);
    acol = Q::S == 1 ? 4 * ((lane >> 2) % Q::CB) : 8 * (lane >> 2 & 3) + (lane >> 2 & 4) + first;
    odd = lane & 1;
    high = lane & 2;
  }
  // column of slot c of the contraction, from `first` on (of a half's contraction: the two chains that it takes)
  static __device__ __forceinline__ constexpr int column(int c) { return Q::S == 1 ? c : 4 * (c >> 1) + (c & 1); }
  // the lane's share of the A operand to its place in LDS (of split rows, each group of lanes stores half)
  __device__ __forceinline__ void store_operand(float *at, const f4_t &a) const {
    if constexpr (Q::S == 1) *(f4_t *)at = a;
    else *(f2_t *)at = f2_t{second ? a[2] : a[0], second ? a[3] : a[1]};
  }
};

// ------------------------------------------------------------------ forward
// One barrier per 16 steps.  q, k, v, f of the next 16 steps travel while the current ones are
// computed.  A lane adds q_i H[i][j] over its 4 rows; the rest of the sum over rows goes through
// LDS once per 16 steps, and over the workgroups of a state through parts_sum_kernel.
template <typename Q>
struct FwdLds {
  alignas(16) float q[2][TB][Q::ROWS], k[2][TB][Q::ROWS], v[2][TB][Q::V], f[2][TB];
  float y[2][TB][Q::NW][64];
};

// SEQ: one workgroup runs the P parts of a state one after the other and adds up y in place, in
// the order of parts_sum_kernel (same bits): for callers whose scratch cannot hold the partial sums.
template <typename Q, bool DO_Y, bool SEQ>
__device__ __forceinline__ void quad_fwd_part(const FwdArgs &a, float *__restrict__ ypart, FwdLds<Q> &sm,
                                              int unit, int part) {
  constexpr int V = Q::V, K = Q::K, ROWS = Q::ROWS, THREADS = Q::THREADS, NQ = Q::NQ, NV = Q::NV;
  const int T = a.T, N = a.N, b = unit / N, n = unit - b * N, g = n / (N / a.Nqk);
  const int tid = threadIdx.x, row_base = part * ROWS;
  const LanePos<Q> p;
  const float *qg = (const float *)a.q + ((size_t)b * T * a.Nqk + g) * K + row_base;
  const float *kg = (const float *)a.k + ((size_t)b * T * a.Nqk + g) * K + row_base;
  const float *vg = (const float *)a.v + ((size_t)b * T * N + n) * V;
  const float *fg = a.f + (size_t)b * T * N + n;
  const size_t qk_step = (size_t)a.Nqk * K, v_step = (size_t)N * V;

  constexpr int E = Q::E;
  typedef typename Q::rows_t rows_t;
  float w[4 * Q::CB];
#pragma unroll
  for (int c = 0; c < 4 * Q::CB; ++c) w[c] = ((const float *)a.W)[((size_t)n * V + p.first + p.column(c)) * V + p.col];
  const size_t st_off = ((size_t)unit * K + row_base + p.row) * V + p.col;
  rows_t h = {};
  if (a.H0) h = load_rows<Q>(a.H0 + st_off);
  arrived(h);

  float rq[NQ], rk[NQ], rv[NV], rf = 0.f;
  // (steps behind the end fetch the last step again and are never used)
  auto load = [&](int t0) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS, t = min(t0 + idx / ROWS, T - 1);
      rq[m] = qg[t * qk_step + idx % ROWS];
      rk[m] = kg[t * qk_step + idx % ROWS];
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS, t = min(t0 + idx / V, T - 1);
      rv[m] = vg[t * v_step + idx % V];
    }
    rf = fg[(size_t)min(t0 + (tid & (TB - 1)), T - 1) * N];
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS;
      (&sm.q[buf][0][0])[idx] = rq[m];
      (&sm.k[buf][0][0])[idx] = rk[m];
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS;
      if (TB * V % THREADS == 0 || idx < TB * V) (&sm.v[buf][0][0])[idx] = rv[m];
    }
    if (tid < TB) sm.f[buf][tid] = a.gate_alpha ? gate_psi(rf, a.gate_alpha[n], a.gate_beta[n]) : rf;
  };
  // y rows of one block out of the per-wave sums in LDS
  auto flush = [&](int t0, int len, int buf) {
    for (int idx = tid; idx < len * V; idx += THREADS) {
      const int s = idx / V, j = idx % V;
      const float *ys = &sm.y[buf][s][0][0] + j;
      float acc = 0.f, acc1 = 0.f;
      // Row groups in order; 32 rows of a shape with a split form as its two parts, 16 rows as two halves (with one chain
      // the error of y against 64 bits was 0.5 % above that of four rows in one chain of FMAs per group).
      constexpr int groups = Q::NW * Q::GR, half = has_split(K, V) && ROWS == K ? groups / 2 : groups;
#pragma unroll
      for (int i = 0; i < groups; ++i) (i < half ? acc : acc1) += Q::S == 1 ? ys[i * V] : ys[2 * i * V] + ys[(2 * i + 1) * V];
      if constexpr (half < groups) acc += acc1;
      const size_t off = (size_t)(t0 + s) * v_step + j;
      if constexpr (Q::P == 1 || SEQ) {
        float *dst = (float *)a.y + ((size_t)b * T * N + n) * V + off;
        if (SEQ && part > 0) acc = *dst + acc;
        // (v from memory: its place in LDS may be overwritten already)
        if (a.w_r && part == Q::P - 1) acc = fmaf(((const float *)a.w_r)[n * V + j], vg[off], acc);
        *dst = acc;
      } else {
        ypart[(size_t)part * a.B * T * v_step + ((size_t)b * T * N + n) * V + off] = acc;
      }
    }
  };

  const int nblk = (T + TB - 1) / TB, nck = (T + a.C - 1) / a.C;
  // V = 16: one row group's step by step order, and the loop without checkpoints apart from the one with
  // them.  us, 512 steps, 4 states, as of the wider ones -> so: 16 x 16 212 -> 204, 32 x 16 217 -> 197,
  // 64 x 16 200 -> 195; but 16 x 32 in split rows 165 -> 171 (300 states in whole rows 380 -> 386).
  constexpr bool NARROW = V == 16;
  int next_ck = a.ckpt || NARROW ? 0 : -1;
  float *ckpt = a.ckpt ? a.ckpt + (size_t)unit * nck * K * V + (size_t)(row_base + p.row) * V + p.col : nullptr;
  if (nblk > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  for (int blk = 0; blk < nblk; ++blk) {
    const int t0 = blk * TB, len = min(TB, T - t0), buf = blk & 1;
    if (blk + 1 < nblk) load(t0 + TB);
    // Of 64 columns and of split rows, a step's vectors are fetched during the one before.  (Whole rows of
    // 32: 32 x 32, 64 states, 512 steps 236 us so, 240 with the fetch ahead; 128 x 32 240 and 249.)
    constexpr bool AHEAD = V > 32 || Q::S > 1;
    rows_t kr1, qr1;
    float vj1, f1;
    auto fetch = [&](int s) __attribute__((always_inline)) {
      kr1 = *(const rows_t *)&sm.k[buf][s][p.row];
      vj1 = sm.v[buf][s][p.col];
      f1 = sm.f[buf][s];
      if constexpr (DO_Y && AHEAD) qr1 = *(const rows_t *)&sm.q[buf][s][p.row];
    };
    if constexpr (AHEAD) fetch(0);
#pragma nounroll
    for (int s = 0; s < len; ++s) {
      if ((!NARROW || ckpt) && t0 + s == next_ck) {  // state before step t0 + s
#pragma unroll
        for (int m = 0; m < E; ++m) ckpt[m * V] = h[m];
        ckpt += (size_t)K * V;
        next_ck += a.C;
      }
      if constexpr (!AHEAD) fetch(s);
      const rows_t kr = kr1;
      rows_t qr = qr1;
      const float vj = vj1, f = f1, gm = 1.f - f;
      if constexpr (AHEAD) fetch(min(s + 1, TB - 1));  // (behind the end: a step that is not used)
      const f4_t ha = quad_transpose(h, p.odd, p.high);
      rows_t z = preactivation<Q>(ha, w, kr, vj);
      if constexpr (!NARROW) z = tanh_f32(z);
#pragma unroll
      for (int m = 0; m < E; ++m) h[m] = fmaf(f, h[m], gm * (NARROW ? tanh_f32((float)z[m]) : z[m]));
      if constexpr (DO_Y) {
        if constexpr (!AHEAD) qr = *(const rows_t *)&sm.q[buf][s][p.row];
        float y = qr[0] * h[0];
        if constexpr (E == 4 && has_split(K, V)) {  // (as two lanes of a split row group do it)
          y = fmaf(qr[1], h[1], y) + fmaf(qr[3], h[3], qr[2] * h[2]);
        } else {
#pragma unroll
          for (int m = 1; m < E; ++m) y = fmaf(qr[m], h[m], y);
        }
        // lanes that share rows are consecutive: [rows][column]
        sm.y[buf][s][p.wave][p.lane - p.lane % V + p.col] = y;
      }
    }
    if (blk + 1 < nblk) store(buf ^ 1);
    // one barrier per block: it closes this block's y sums and the next block's vectors; the
    // buffers of this block are written again only behind the next barrier
    __syncthreads();
    if constexpr (DO_Y) flush(t0, len, buf);
  }
  if (a.HT)
#pragma unroll
    for (int m = 0; m < E; ++m) a.HT[st_off + m * V] = h[m];
}

template <typename Q, bool DO_Y, bool SEQ>
__global__ void __launch_bounds__(Q::THREADS, 2) quad_fwd_kernel(FwdArgs a, float *__restrict__ ypart) {
  __shared__ FwdLds<Q> sm;
  if constexpr (SEQ) {
    for (int part = 0; part < Q::P; ++part) {
      quad_fwd_part<Q, DO_Y, true>(a, ypart, sm, blockIdx.x, part);
      __syncthreads();
    }
  } else {
    quad_fwd_part<Q, DO_Y, false>(a, ypart, sm, blockIdx.x / Q::P, blockIdx.x % Q::P);
  }
}

// ------------------------------------------------------------------ backward
// Per stash of up to 16 steps, last to first:
//   recompute  the states from the checkpoint, H before each step and Z of each step to LDS
//   sweep      in reverse: G = q dy^T + carry, dS = (1 - f) G (1 - Z^2) into Z's place,
//              carry = f G + dS W^T; df from a 16x16x4 product with ones, each step's sum kept by
//              one lane of 16 (ones in column s alone and a running sum would let a NaN or an
//              infinity of one step into the df of all others of the stash: 0 x NaN is NaN)
//   finish     everything that contracts over more than a wave holds, for all 16 steps at once,
//              out of LDS: dW += sum_s H^T dS (16x16x4 products over steps and rows), dq = H dy,
//              dk = dS v, dv = dS^T k
// Recompute and sweep are private to a wave (no barrier); two barriers per stash around `finish`.
// H and dS lie row-major with the 16-column blocks of a row placed by (row xor block), so that the
// 4 rows that a matrix operand reads at once fall on different banks.
template <typename Q>
struct BwdLds {
  static constexpr int V = Q::V, ROWS = Q::ROWS;
  alignas(16) float H[TB + 1][ROWS * V];
  alignas(16) float D[TB][ROWS * V];
  alignas(16) float q[TB][ROWS], k[TB][ROWS], v[TB][V], dy[TB][V], f[TB];
  float df[Q::NW * 4][TB];
};
template <int V>
__device__ __forceinline__ int sw(int row, int col) {  // element offset inside [ROWS][V]
  const int x = V == 64 ? (row & 3) : (V == 32 ? ((row >> 1) & 1) : 0);
  return row * V + (col ^ (16 * x));
}

struct QuadBwdWs {
  float *sub;     // [units][P][nsub (+ 1)][THREADS * 4]: states in front of the later stashes of a chunk
                  // (C > 16), and, the parts in turn, each part's carried gradient
  float *dvp, *dfp;  // [P][B,T,N,V], [P][B,T,N]  (P > 1, the parts side by side)
  float *dWp;     // [B N P][V][V], the parts in turn [B N][V][V]
  float *dqh, *dkh;  // [B,T,N,K] (Nqk != N)
  int nsub;
};

// SEQ: one workgroup runs the P parts of a state one after the other inside every stash, their dv and
// df added up in registers in the order of parts_sum_kernel (same bits; dW is added in another
// order): for callers whose workspace cannot hold the partial sums.
template <typename IO, typename Q, bool SEQ>
__global__ void __launch_bounds__(Q::THREADS, Q::V < 64 ? 2 : 1) quad_bwd_kernel(BwdArgs a, QuadBwdWs ws) {
  constexpr int V = Q::V, K = Q::K, ROWS = Q::ROWS, THREADS = Q::THREADS, NQ = Q::NQ, NV = Q::NV,
                NW = Q::NW;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  BwdLds<Q> &sm = *(BwdLds<Q> *)lds;
  constexpr int TURNS = SEQ ? Q::P : 1;
  const int unit = SEQ ? blockIdx.x : blockIdx.x / Q::P;
  int part = SEQ ? 0 : blockIdx.x % Q::P, row_base = part * ROWS;
  const int T = a.T, N = a.N, C = a.C, b = unit / N, n = unit - b * N, g = n / (N / a.Nqk);
  const int tid = threadIdx.x;
  const LanePos<Q> p;
  const size_t qk0 = ((size_t)b * T * a.Nqk + g) * K + (SEQ ? 0 : row_base), v0 = ((size_t)b * T * N + n) * V,
               f0 = (size_t)b * T * N + n;
  const size_t qk_step = (size_t)a.Nqk * K, v_step = (size_t)N * V;
  const IO *qg = (const IO *)a.q + qk0, *kg = (const IO *)a.k + qk0, *vg = (const IO *)a.v + v0,
           *dyg = (const IO *)a.dy + v0;
  const float *fg = a.f + f0;

  constexpr int E = Q::E;
  typedef typename Q::rows_t rows_t;
  float w[4 * Q::CB], wt[4 * Q::CB];
  const IO *wp = (const IO *)a.W + (size_t)n * V * V;
#pragma unroll
  for (int c = 0; c < 4 * Q::CB; ++c) {
    w[c] = to_f32<IO>(wp[p.first * V + p.col + p.column(c) * V]);
    wt[c] = to_f32<IO>(wp[p.col * V + p.first + p.column(c)]);
  }
  auto st_off = [&]() __attribute__((always_inline)) { return ((size_t)unit * K + row_base + p.row) * V + p.col; };
  // a part's slots in the workspace: a place that only the same lane reads again
  const int slots = SEQ ? ws.nsub + 1 : ws.nsub;
  auto slot = [&](int i) __attribute__((always_inline)) { return (rows_t *)ws.sub + (((size_t)unit * Q::P + part) * slots + i) * THREADS + tid; };
  auto turn = [&](int i) __attribute__((always_inline)) {
    if constexpr (SEQ) {
      part = i;
      row_base = i * ROWS;
    }
  };
  rows_t carry = {};
  for (int i = 0; i < TURNS; ++i) {
    turn(i);
    if (a.dHT) carry = load_rows<Q>(a.dHT + st_off());
    arrived(carry);
    if constexpr (SEQ) *slot(ws.nsub) = carry;
  }

  // dW tiles of 16 x 16: with at least one per wave, wave w owns the NTW tiles w NTW ..; with
  // fewer tiles than waves, SPLIT waves add their shares of the rows to the same tile
  constexpr int CT = V / 16, NT = CT * CT, NTW = NT >= NW ? NT / NW : 1, SPLIT = NT >= NW ? 1 : NW / NT;
  f4_t dW[NTW];
#pragma unroll
  for (int i = 0; i < NTW; ++i) dW[i] = f4_t{0.f, 0.f, 0.f, 0.f};

  float rq[NQ], rk[NQ], rv[NV], rdy[NV], rf = 0.f;
  auto load = [&](int t0, int len) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS, t = t0 + min(idx / ROWS, len - 1);
      rq[m] = to_f32<IO>(qg[t * qk_step + idx % ROWS + (SEQ ? row_base : 0)]);
      rk[m] = to_f32<IO>(kg[t * qk_step + idx % ROWS + (SEQ ? row_base : 0)]);
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS, t = t0 + min(idx / V, len - 1);
      rv[m] = to_f32<IO>(vg[t * v_step + idx % V]);
      rdy[m] = to_f32<IO>(dyg[t * v_step + idx % V]);
    }
    rf = fg[(size_t)(t0 + min(tid & (TB - 1), len - 1)) * N];
  };
  auto store = [&]() {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      (&sm.q[0][0])[tid + m * THREADS] = rq[m];
      (&sm.k[0][0])[tid + m * THREADS] = rk[m];
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS;
      if (TB * V % THREADS == 0 || idx < TB * V) {
        (&sm.v[0][0])[idx] = rv[m];
        (&sm.dy[0][0])[idx] = rdy[m];
      }
    }
    if (tid < TB) sm.f[tid] = a.gate_alpha ? gate_psi(rf, a.gate_alpha[n], a.gate_beta[n]) : rf;
  };
  // one recomputed step of the recurrence; the state's A operand is returned for the stash
  // (Of split rows, a step's vectors are fetched during the one before.  With four rows per lane the
  // sweep is 1 % slower so: 64 x 64, 64 states, T = 512 983 -> 993 us.)
  constexpr bool AHEAD = Q::S > 1;
  rows_t kr1;
  float vj1, f1;
  auto fetch = [&](int s) __attribute__((always_inline)) {
    kr1 = *(const rows_t *)&sm.k[s][p.row];
    vj1 = sm.v[s][p.col];
    f1 = sm.f[s];
  };
  auto step = [&](rows_t &h, int s, f4_t &ha) __attribute__((always_inline)) {
    if constexpr (!AHEAD) fetch(s);
    const rows_t kr = kr1;
    const float vj = vj1, f = f1, gm = 1.f - f;
    if constexpr (AHEAD) fetch(min(s + 1, TB - 1));
    ha = quad_transpose(h, p.odd, p.high);
    rows_t z = preactivation<Q>(ha, w, kr, vj);
    if constexpr (AHEAD) {
      z = tanh_f32(z);
#pragma unroll
      for (int m = 0; m < E; ++m) h[m] = fmaf(f, h[m], gm * z[m]);
    } else {  // (element by element: 1 % here, the other way round in the forward)
#pragma unroll
      for (int m = 0; m < E; ++m) {
        z[m] = tanh_f32((float)z[m]);
        h[m] = fmaf(f, h[m], gm * z[m]);
      }
    }
    return z;
  };

  const int nck = (T + C - 1) / C;
  const int a_off = sw<V>(p.arow, p.acol);
  // Z of a step lies where its dS will: a wave's share of the rows, in the order of its lanes
  rows_t *const zst = (rows_t *)&sm.D[0][0];
  if (!SEQ && nck > 0) {  // vectors of the last stash
    const int t0 = (nck - 1) * C, len = T - t0, sub = (len - 1) / TB;
    load(t0 + sub * TB, len - sub * TB);
  }
  for (int ck = nck - 1; ck >= 0; --ck) {
    const int ck0 = ck * C, clen = min(C, T - ck0), nsub = (clen + TB - 1) / TB;
    auto checkpoint = [&]() __attribute__((always_inline)) {
      rows_t h = load_rows<Q>(a.ckpt + ((size_t)unit * nck + ck) * K * V + (size_t)(row_base + p.row) * V + p.col);
      arrived(h);
      return h;
    };
    rows_t hck = {};
    if constexpr (!SEQ) hck = checkpoint();
    // checkpoints further apart than a stash: a first pass leaves the state in front of each
    // later stash in the workspace
    if (nsub > 1) {
      for (int i = 0; i < TURNS; ++i) {
        turn(i);
        if constexpr (SEQ) hck = checkpoint();
        rows_t h = hck;
        f4_t ha;
        for (int sub = 0; sub + 1 < nsub; ++sub) {
          load(ck0 + sub * TB, TB);
          __syncthreads();
          store();
          __syncthreads();
          if constexpr (AHEAD) fetch(0);
#pragma nounroll
          for (int s = 0; s < TB; ++s) step(h, s, ha);
          *slot(sub) = h;
        }
      }
      if constexpr (!SEQ) load(ck0 + (nsub - 1) * TB, clen - (nsub - 1) * TB);
      __syncthreads();
    }
    for (int sub = nsub - 1; sub >= 0; --sub) {
      const int t0 = ck0 + sub * TB, len = min(TB, clen - sub * TB);
      float dvsum[NV], dfsum = 0.f;  // (the parts in turn)
      for (int i = 0; i < TURNS; ++i) {
        turn(i);
        if constexpr (SEQ) {
          load(t0, len);
          carry = *slot(ws.nsub);
          if (sub == 0) hck = checkpoint();
        }
        store();
        rows_t h = sub > 0 ? *slot(sub - 1) : hck;
        f4_t ha;
        arrived(h);
        __syncthreads();
        // the next stash's vectors travel during this one
        if constexpr (!SEQ) {
          if (sub > 0) load(t0 - TB, TB);
          else if (ck > 0 && C <= TB) load(ck0 - C, C);
        }
        // ---- recompute
        if constexpr (AHEAD) fetch(0);
#pragma nounroll
        for (int s = 0; s < len; ++s) {
          const rows_t z = step(h, s, ha);
          p.store_operand(&sm.H[s][a_off], ha);
          zst[s * (ROWS * V / E) + tid] = z;  // (only this lane reads it again)
        }
        ha = quad_transpose(h, p.odd, p.high);
        p.store_operand(&sm.H[len][a_off], ha);
        // ---- sweep
        float dfacc = 0.f;
        rows_t q1, z1, h1;
        float dy1;
        auto fetch_sweep = [&](int s) __attribute__((always_inline)) {
          q1 = *(const rows_t *)&sm.q[s][p.row];
          dy1 = sm.dy[s][p.col];
          f1 = sm.f[s];
          z1 = zst[s * (ROWS * V / E) + tid];
#pragma unroll
          for (int m = 0; m < E; ++m) h1[m] = sm.H[s][sw<V>(p.row + m, p.col)];
        };
        if constexpr (AHEAD) fetch_sweep(len - 1);
#pragma nounroll
        for (int s = len - 1; s >= 0; --s) {
          if constexpr (!AHEAD) fetch_sweep(s);
          const rows_t qr = q1, z = z1, hp = h1;
          const float dyj = dy1, f = f1, gm = 1.f - f;
          if constexpr (AHEAD) fetch_sweep(max(s - 1, 0));
          rows_t G, dS;
          float dfl = 0.f;
#pragma unroll
          for (int m = 0; m < E; ++m) {
            G[m] = fmaf(qr[m], dyj, carry[m]);
            dfl = fmaf(G[m], hp[m] - z[m], dfl);
            dS[m] = gm * G[m] * fmaf(-z[m], z[m], 1.f);
          }
          const f4_t da = quad_transpose(dS, p.odd, p.high);
          p.store_operand(&sm.D[s][a_off], da);
          const f4_t df4 = __builtin_amdgcn_mfma_f32_16x16x4f32(dfl, 1.f, f4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          const rows_t d = contract<Q>(da, wt);
#pragma unroll
          for (int m = 0; m < E; ++m) carry[m] = fmaf(f, G[m], d[m]);
          // every column of df4 is the same: lane (j, i) holds the sums of 4 of the 16 rows i' = 4 i + r
          dfacc = (p.lane & 15) == s ? (df4[0] + df4[1]) + (df4[2] + df4[3]) : dfacc;
          if (a.clip > 0.f)
#pragma unroll
            for (int m = 0; m < E; ++m) carry[m] = __builtin_amdgcn_fmed3f(carry[m], -a.clip, a.clip);
        }
        sm.df[p.wave * 4 + (p.lane >> 4)][p.lane & 15] = dfacc;  // lane (s, i): its rows' sum of step s
        __syncthreads();
        // ---- finish: dW, 4 rows of one step per product
#pragma unroll
        for (int i = 0; i < NTW; ++i) {
          const int tile = SPLIT > 1 ? p.wave / SPLIT : p.wave * NTW + i, ci = tile / CT, cj = tile % CT;
          const int kr = p.lane >> 4, c = p.lane & 15;
          // (summed per stash first: one running sum over all steps would lose two bits)
          f4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
          constexpr int NR = ROWS / SPLIT;
          const int r0 = p.wave % SPLIT * NR;
          for (int s = 0; s < len; ++s) {
#pragma unroll
            for (int r = 0; r < NR; r += 8) {
              const int ra = r0 + r + kr, rb = ra + 4;
              acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(sm.H[s][sw<V>(ra, 16 * ci + c)],
                                                          sm.D[s][sw<V>(ra, 16 * cj + c)], acc0, 0, 0, 0);
              if (r + 4 < NR)
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sm.H[s][sw<V>(rb, 16 * ci + c)],
                                                            sm.D[s][sw<V>(rb, 16 * cj + c)], acc1, 0, 0, 0);
            }
          }
          dW[i] += acc0 + acc1;
        }
        // ---- finish: dq_s[i] = H_s dy_s, dk_s[i] = dS_s v_s, one (step, row) per thread
        for (int idx = tid; idx < len * ROWS; idx += THREADS) {
          const int s = idx / ROWS, i = idx % ROWS;
          f4_t q4 = {0.f, 0.f, 0.f, 0.f}, k4 = q4;
#pragma unroll 4
          for (int c4 = 0; c4 < V / 4; ++c4) {
            const int c = 4 * (c4 ^ ((i >> 2) & 3));  // (rows that share a swizzle start on other banks)
            q4 += *(const f4_t *)&sm.H[s + 1][sw<V>(i, c)] * *(const f4_t *)&sm.dy[s][c];
            k4 += *(const f4_t *)&sm.D[s][sw<V>(i, c)] * *(const f4_t *)&sm.v[s][c];
          }
          const float dq = (q4[0] + q4[1]) + (q4[2] + q4[3]), dk = (k4[0] + k4[1]) + (k4[2] + k4[3]);
          if (ws.dqh) {
            const size_t o = (((size_t)b * T + t0 + s) * N + n) * K + row_base + i;
            ws.dqh[o] = dq;
            ws.dkh[o] = dk;
          } else {
            const size_t o = qk0 + (size_t)(t0 + s) * qk_step + i + (SEQ ? row_base : 0);
            ((IO *)a.dq)[o] = from_f32<IO>(dq);
            ((IO *)a.dk)[o] = from_f32<IO>(dk);
          }
        }
        // ---- finish: dv_s[j] = sum over the workgroup's rows of dS[i][j] k_i, one (step, column)
        const bool last_part = Q::P == 1 || (SEQ && part == Q::P - 1);
        auto finish_dv = [&](int idx, float &sum) __attribute__((always_inline)) {
          const int s = idx / V, j = idx % V;
          float acc = 0.f;
#pragma unroll 8
          for (int r = 0; r < ROWS; ++r) acc = fmaf(sm.D[s][sw<V>(r, j)], sm.k[s][r], acc);
          const size_t o = v0 + (size_t)(t0 + s) * v_step + j;
          if constexpr (SEQ) acc = sum = part ? sum + acc : acc;
          if (last_part) {
            if (a.w_r) acc = fmaf(to_f32<IO>(((const IO *)a.w_r)[n * V + j]), sm.dy[s][j], acc);
            ((IO *)a.dv)[o] = from_f32<IO>(acc);
          } else if constexpr (!SEQ) {
            ws.dvp[(size_t)part * a.B * T * v_step + o] = acc;
          }
        };
        if constexpr (SEQ) {
#pragma unroll
          for (int m = 0; m < NV; ++m)
            if (tid + m * THREADS < len * V) finish_dv(tid + m * THREADS, dvsum[m]);
        } else {
          for (int idx = tid; idx < len * V; idx += THREADS) finish_dv(idx, dvsum[0]);
        }
        if (tid < len) {
          float acc = 0.f;
          if constexpr (Q::S == 1) {
#pragma unroll
            for (int r = 0; r < NW * 4; ++r) acc += sm.df[r][tid];
          } else {  // (twice as many terms: four chains of them)
            f4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < NW * 4; ++r) x[r % 4] += sm.df[r][tid];
            acc = (x[0] + x[1]) + (x[2] + x[3]);
          }
          const size_t o = f0 + (size_t)(t0 + tid) * N;
          if constexpr (SEQ) acc = dfsum = part ? dfsum + acc : acc;
          if (last_part) a.df[o] = acc;
          else if constexpr (!SEQ) ws.dfp[(size_t)part * a.B * T * N + o] = acc;
        }
        if constexpr (SEQ) *slot(ws.nsub) = carry;
        __syncthreads();
      }
    }
  }
  if (a.dH0)
    for (int i = 0; i < TURNS; ++i) {
      turn(i);
      if constexpr (SEQ) carry = *slot(ws.nsub);
#pragma unroll
      for (int m = 0; m < E; ++m) a.dH0[st_off() + m * V] = carry[m];
    }
  // dW of the workgroup: D layout of the 16x16 product, rows 4 (lane / 16) + r, column lane % 16
  float *dst = ws.dWp + (size_t)blockIdx.x * V * V;
  if constexpr (SPLIT > 1) {
    f4_t *red = (f4_t *)sm.H;
    __syncthreads();
    red[tid] = dW[0];
    __syncthreads();
    if (p.wave % SPLIT == 0) {
      const int tile = p.wave / SPLIT, ci = tile / CT, cj = tile % CT;
      f4_t s = red[tid];
#pragma unroll
      for (int i = 1; i < SPLIT; ++i) s += red[i * 64 + tid];
#pragma unroll
      for (int r = 0; r < 4; ++r) dst[(16 * ci + 4 * (p.lane >> 4) + r) * V + 16 * cj + (p.lane & 15)] = s[r];
    }
  } else {
#pragma unroll
    for (int i = 0; i < NTW; ++i) {
      const int tile = p.wave * NTW + i, ci = tile / CT, cj = tile % CT;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        dst[(16 * ci + 4 * (p.lane >> 4) + r) * V + 16 * cj + (p.lane & 15)] = dW[i][r];
    }
  }
}

// out = sum over P parts in increasing order [+ w_r (.) x, the residual's term]
template <typename IO>
__global__ void parts_sum_kernel(const float *__restrict__ part, IO *__restrict__ out, size_t total, int P,
                                 const IO *__restrict__ w_r, const IO *__restrict__ x, int NV) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    float s = part[e];
    for (int p = 1; p < P; ++p) s += part[(size_t)p * total + e];
    if (w_r) s = fmaf(to_f32<IO>(w_r[e % NV]), to_f32<IO>(x[e]), s);
    out[e] = from_f32<IO>(s);
  }
}
template <typename IO>
hipError_t parts_sum(const float *part, IO *out, size_t total, int P, const IO *w_r, const IO *x, int NV,
                     hipStream_t s) {
  if (total == 0) return hipSuccess;
  const size_t blocks = (total + 255) / 256;
  hipLaunchKernelGGL(parts_sum_kernel<IO>, dim3((unsigned)(blocks > 8192 ? 8192 : blocks)), dim3(256), 0, s, part,
                     out, total, P, w_r, x, NV);
  return hipGetLastError();
}

// dW[n] = sum over the batch and the workgroups of a state: a workgroup adds 64 elements of one head,
// its W waves the rows (b, p) w, w + W, ... with four loads in flight, and the waves' sums in increasing
// order.  W grows with the rows (quad_dw_waves): one chain over all of them took most of a launch of
// many short sequences.  Backward at T = 1, 2048 states, one chain -> now: 128 x 64 7301 -> 859 us,
// 64 x 64 2555 -> 414, 16 x 16 643 -> 47.
__global__ void __launch_bounds__(1024)
    quad_dw_sum_kernel(const float *__restrict__ dWp, float *__restrict__ dW, int N, int P, int VV, int R) {
  __shared__ float red[16][64];
  const int W = blockDim.x >> 6, w = threadIdx.x >> 6, cl = threadIdx.x & 63;
  const int n = blockIdx.x / (VV / 64), e = (blockIdx.x % (VV / 64)) * 64 + cl;
  auto row = [&](int r) { return dWp[(((size_t)(r / P) * N + n) * P + r % P) * VV + e]; };
  float s = 0.f;
  int r = w;
  for (; r + 3 * W < R; r += 4 * W) {
    const float x0 = row(r), x1 = row(r + W), x2 = row(r + 2 * W), x3 = row(r + 3 * W);
    s = (((s + x0) + x1) + x2) + x3;
  }
  for (; r < R; r += W) s += row(r);
  red[w][cl] = s;
  __syncthreads();
  if (w == 0) {
    for (int i = 1; i < W; ++i) s += red[i][cl];
    dW[(size_t)n * VV + e] = s;
  }
}
int quad_dw_waves(int rows) { return rows <= 16 ? 1 : rows <= 64 ? 4 : 16; }

template <typename Q>
size_t fwd_parts_bytes(int B, int T, int N) {
  return Q::P > 1 ? align256((size_t)Q::P * B * N * T * Q::V * 4) : 0;
}

template <typename Q>
hipError_t launch_fwd(const FwdArgs &a, hipStream_t s) {
  const int units = a.B * a.N;
  if (units == 0) return hipSuccess;
  float *ypart = (float *)a.ws;
  constexpr bool turns = Q::P > 1 && Q::S == 1;  // (split parts are taken only with room for their sums)
  const bool seq = turns && a.write_y && a.ws_bytes < fwd_parts_bytes<Q>(a.B, a.T, a.N);
  const dim3 grid(seq ? units : units * Q::P), block(Q::THREADS);
  if (!a.write_y)
    hipLaunchKernelGGL((quad_fwd_kernel<Q, false, false>), grid, block, 0, s, a, ypart);
  else if (!seq)
    hipLaunchKernelGGL((quad_fwd_kernel<Q, true, false>), grid, block, 0, s, a, ypart);
  else if constexpr (turns)
    hipLaunchKernelGGL((quad_fwd_kernel<Q, true, true>), grid, block, 0, s, a, ypart);
  hipError_t e = hipGetLastError();
  if (seq) return e;
  if (e == hipSuccess && Q::P > 1 && a.write_y)
    e = parts_sum<float>(ypart, (float *)a.y, (size_t)a.B * a.T * a.N * a.V, Q::P, (const float *)a.w_r,
                         (const float *)a.v, a.N * a.V, s);
  return e;
}

struct QuadLayout {
  size_t sub, dvp, dfp, dWp, heads, total;
  int nsub;
};
// seq: the parts of a state in turn
QuadLayout quad_layout(int B, int T, int N, int Nqk, int K, int V, int C, int P, int threads, bool seq) {
  QuadLayout l;
  const size_t units = (size_t)B * N;
  const bool side = P > 1 && !seq;
  l.nsub = (C - 1) / TB;
  l.sub = align256(units * P * (l.nsub + (seq ? 1 : 0)) * threads * 16);
  l.dvp = side ? align256((size_t)P * units * T * V * 4) : 0;
  l.dfp = side ? align256((size_t)P * units * T * 4) : 0;
  l.dWp = align256(units * (seq ? 1 : P) * V * V * 4);
  l.heads = Nqk != N ? align256(units * T * K * 4) : 0;
  l.total = l.sub + l.dvp + l.dfp + l.dWp + 2 * l.heads;
  return l;
}

template <typename IO, typename Q, bool SEQ>
hipError_t launch_bwd_as(const BwdArgs &a, const QuadLayout &l, hipStream_t s) {
  constexpr bool side = Q::P > 1 && !SEQ;
  const int units = a.B * a.N;
  char *p = a.ws;
  QuadBwdWs ws;
  ws.nsub = l.nsub;
  ws.sub = (float *)p; p += l.sub;
  ws.dvp = (float *)p; p += l.dvp;
  ws.dfp = (float *)p; p += l.dfp;
  ws.dWp = (float *)p; p += l.dWp;
  ws.dqh = l.heads ? (float *)p : nullptr; p += l.heads;
  ws.dkh = l.heads ? (float *)p : nullptr;
  hipError_t e;
  if (units > 0) {
    auto kernel = quad_bwd_kernel<IO, Q, SEQ>;
    if ((e = set_max_lds_once(kernel, (int)sizeof(BwdLds<Q>))) != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(SEQ ? units : units * Q::P), dim3(Q::THREADS), sizeof(BwdLds<Q>), s, a, ws);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t steps = (size_t)units * a.T;
    if (side) {
      e = parts_sum<IO>(ws.dvp, (IO *)a.dv, steps * a.V, Q::P, (const IO *)a.w_r, (const IO *)a.dy, a.N * a.V, s);
      if (e == hipSuccess)
        e = parts_sum<float>(ws.dfp, a.df, steps, Q::P, nullptr, nullptr, 1, s);
      if (e != hipSuccess) return e;
    }
    if (l.heads) {
      if ((e = generic_head_group_sum(a, ws.dqh, a.dq, s)) != hipSuccess) return e;
      if ((e = generic_head_group_sum(a, ws.dkh, a.dk, s)) != hipSuccess) return e;
    }
  }
  const int VV = a.V * a.V, P = SEQ ? 1 : Q::P, rows = a.B * P;
  hipLaunchKernelGGL(quad_dw_sum_kernel, dim3((unsigned)(a.N * (VV / 64))), dim3(64 * quad_dw_waves(rows)), 0, s,
                     ws.dWp, a.dW, a.N, P, VV, rows);
  return hipGetLastError();
}
template <typename IO, typename Q>
hipError_t launch_bwd(const BwdArgs &a, hipStream_t s) {
  auto layout = [&](bool seq) { return quad_layout(a.B, a.T, a.N, a.Nqk, a.K, a.V, a.C, Q::P, Q::THREADS * Q::E / 4, seq); };
  const QuadLayout side = layout(false), turns = layout(true);
  if (a.ws_bytes >= side.total) return launch_bwd_as<IO, Q, false>(a, side, s);
  if constexpr (Q::P > 1 && Q::S == 1)
    if (a.ws_bytes >= turns.total) return launch_bwd_as<IO, Q, true>(a, turns, s);
  return hipErrorInvalidValue;
}

#define M2RNN_QUAD_CASES(X) \
  X(16, 16) X(32, 16) X(64, 16) X(128, 16) X(16, 32) X(32, 32) X(64, 32) X(128, 32) X(16, 64) X(32, 64) X(64, 64) X(128, 64)

}  // namespace

bool quad_supported(int, int V) { return V <= 64; }

namespace {
// the split kernel where there is one
template <int K, int V>
using QuadSplit = std::conditional_t<has_split(K, V), Split<K, V>, Quad<K, V>>;
// As long as every wave has a SIMD (1024) for itself.  us, T = 512, forward / backward, 8 rows per wave -> split:
// 32 x 32 8 states 230 / 583 -> 167 / 409, 128 states 233 / 601 -> 180 / 437, but 192 states 249 / 606 -> 267 / 626;
// 16 x 32 256 states 240 / 618 -> 172 / 424.
bool split_pays(int K, int V, int units) { return has_split(K, V) && (long long)units * K <= 4096; }
// ... and the steps that repay what the split costs besides.  A 32-row state is two workgroups then, whose y
// (dv, df) are summed by a launch (two) more.  us, whole / split, forward and backward, 32 x 32, 32 states:
// T = 1 3.3 / 5.0 and 8.5 / 12.4, 8 6.5 / 7.4 and 15.2 / 16.8, 12 8.4 / 8.6 and 20.0 / 19.7, 16 10.2 / 9.9 and
// 23.8 / 22.5.  16 x 32, 32 states: T = 1 3.2 / 3.3 and 8.1 / 8.4, 2 3.7 / 3.5 and 9.1 / 9.0.
// And only while the two parts' sums stay small: the query is what a caller allocates unasked, and grows
// with the steps (whole rows take none of it, and 1.4 times the time).
constexpr size_t kMostParts = (size_t)64 << 20;
bool steps_repay(int K, int V, int units, int T) {
  return K == 32 ? T >= 16 && (size_t)units * T * V * 8 <= kMostParts : T >= 2;
}

template <typename Q>
size_t workspace_of(int B, int T, int N, int Nqk, int C, int bwd) {
  if (!bwd) return fwd_parts_bytes<Q>(B, T, N);
  return quad_layout(B, T, N, Nqk, Q::K, Q::V, C, Q::P, Q::THREADS * Q::E / 4, false).total;
}
}  // namespace

size_t quad_workspace_bytes(int B, int T, int N, int Nqk, int K, int V, int C, int bwd, bool may_split) {
  const bool split = may_split && split_pays(K, V, B * N) && steps_repay(K, V, B * N, T);
#define X(K_, V_)                                                                                       \
  if (K == K_ && V == V_)                                                                               \
    return split ? workspace_of<QuadSplit<K_, V_>>(B, T, N, Nqk, C, bwd)                                \
                 : workspace_of<Quad<K_, V_>>(B, T, N, Nqk, C, bwd);
  M2RNN_QUAD_CASES(X)
#undef X
  return 0;
}

hipError_t quad_fwd(const FwdArgs &a, hipStream_t s) {
  const size_t room = a.ws_bytes;
  // (a pass without y has nothing to sum and needs no room)
  const bool split = split_pays(a.K, a.V, a.B * a.N) &&
                     (!a.write_y || (steps_repay(a.K, a.V, a.B * a.N, a.T) &&
                                     room >= quad_workspace_bytes(a.B, a.T, a.N, a.Nqk, a.K, a.V, a.C, 0, true)));
#define X(K_, V_)                                                                                       \
  if (a.K == K_ && a.V == V_)                                                                           \
    return split ? launch_fwd<QuadSplit<K_, V_>>(a, s) : launch_fwd<Quad<K_, V_>>(a, s);
  M2RNN_QUAD_CASES(X)
#undef X
  return hipErrorInvalidValue;
}

// bf16 io: the shapes without a matrix-core backward
#define M2RNN_QUAD_BF16_CASES(X) X(16, 32) X(64, 32) X(128, 32) X(16, 64) X(32, 64) X(128, 64)

hipError_t quad_bwd(const BwdArgs &a, hipStream_t s) {
  const size_t room = a.ws_bytes;
  const bool split = split_pays(a.K, a.V, a.B * a.N) && steps_repay(a.K, a.V, a.B * a.N, a.T) &&
                     room >= quad_workspace_bytes(a.B, a.T, a.N, a.Nqk, a.K, a.V, a.C, 1, true);
  if (a.io == 0) {
#define X(K_, V_)                                                                                   \
  if (a.K == K_ && a.V == V_)                                                                       \
    return split ? launch_bwd<float, QuadSplit<K_, V_>>(a, s) : launch_bwd<float, Quad<K_, V_>>(a, s);
    M2RNN_QUAD_CASES(X)
#undef X
  } else {
#define X(K_, V_)                                                                                   \
  if (a.K == K_ && a.V == V_)                                                                       \
    return split ? launch_bwd<__hip_bfloat16, QuadSplit<K_, V_>>(a, s)                              \
                 : launch_bwd<__hip_bfloat16, Quad<K_, V_>>(a, s);
    M2RNN_QUAD_BF16_CASES(X)
#undef X
  }
  return hipErrorInvalidValue;
}

}  // namespace m2rnn
