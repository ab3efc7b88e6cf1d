// The forward on blocks of eight state rows (m2rnn_half_fwd.hip) for launches of few 32 x 32 or 64 x 64 states,
// whose waves have a SIMD each: no wave waits for another one within 16 steps.
//
// What bounds it, and why this split: a wave alone on its SIMD issues an instruction every 5.5 cycles,
// and a step is its chain; spread over V / 16 waves, a row block adds an LDS round trip and a barrier
// to it.  Here a wave owns 128 elements of the state, 2 rows x 64 columns or 4 x 32, and the operand never
// leaves its registers.  Row i of H W needs all of row i of H and nothing else of it.
// v_mfma_f32_4x4x4_16b_f16 computes 16 independent 4 x 4 blocks over four columns and can broadcast one
// block's A operand to a group of blocks (cbsz / abid): with A = the hi and lo parts of two rows
// (H' = hi + lo to ~21 bits, as in all forward kernels) x four columns of the state, broadcast, and
// B = those four rows of W spread over the V columns, V / 4 such instructions are the product of
// two rows, both parts, with W.  They take 8 cycles for an eighth of the products of a 16x16x32 one's 16,
// which is why the exchange is the better way as soon as waves share a SIMD, and at V = 16, where a
// row block is one wave in either form (pair_serves).
// Layouts.  Accumulator: lane (block, n) holds column 4 (block mod V/4) + n, registers {hi0, hi1, lo0, lo1}
// of its two rows.  A operand: lane (block, m) holds part m of four columns.  The two differ by a 4 x 4
// transposition inside each quad of lanes (`operand`), done half in fp32 in front of the split, so that it
// costs four selects.
#include "m2rnn_kernels.hpp"
#include "m2rnn_mfma_common.hpp"

#include <utility>

namespace m2rnn {
namespace {

constexpr int TB = 16;  // steps per staged block

template <int K_, int V_, int RB_>
struct Pair {
  static constexpr int K = K_, V = V_, RB = RB_;
  static constexpr int GR = 64 / V;                  // row pairs per wave
  static constexpr int ROWS = 8 * RB;                // rows per workgroup
  static constexpr int PAIRS = ROWS / 2;
  static constexpr int THREADS = PAIRS / GR * 64;
  static constexpr int P = K / ROWS;
  static constexpr int KB = V / 4;                   // 4-column blocks of a row
  static constexpr int CBSZ = KB == 16 ? 4 : (KB == 8 ? 3 : 2);
  static constexpr int YW = RB == 1 ? 4 : (RB == 2 ? 2 : 1);  // columns per thread of the readout's sum
  static_assert(K % ROWS == 0 && THREADS <= 1024 && THREADS * YW >= TB * V, "bad split");
};

template <typename PT>
struct PairSmem {
  alignas(16) f4_t kq[2][TB][PT::PAIRS];             // c k, c k, q, q of a row pair
  alignas(16) float v[2][TB][PT::V];
  alignas(16) float f[2][TB][2];                     // f, c(1-f)
  alignas(16) float y[2][TB][PT::PAIRS][PT::V];      // q_i H'[i][j] summed over a row pair
};

template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float quad_perm(float x) {
  return __builtin_bit_cast(float, quad_perm<CTRL>(__builtin_bit_cast(uint32_t, x)));
}
// The A operand out of a lane's two rows of one column.  Even lanes take row 0 of their own and the next
// lane's column, odd lanes row 1 of the previous one's and their own; after the split the lower two lanes
// of a quad take the hi parts of its four columns, the upper two the lo parts.
__device__ __forceinline__ h4_t operand(const float (&h)[2], bool odd, bool high) {
  const float p0 = quad_perm<0xB1>(h[0]), p1 = quad_perm<0xB1>(h[1]);
  const u2_t s = split2_hi_lo(odd ? p1 : h[0], odd ? h[1] : p0);
  const uint32_t q0 = quad_perm<0x4E>(s.x), q1 = quad_perm<0x4E>(s.y);
  return __builtin_bit_cast(h4_t, u2_t{high ? q1 : s.x, high ? s.y : q0});
}
// H W of the wave's rows, hi and lo parts apart: two chains, because the result of a 4x4x4 is not ready
// for the next instruction's accumulator
template <int CBSZ, int KB, int... B0>
__device__ __forceinline__ f4_t contract(h4_t a, const h4_t (&w)[KB], std::integer_sequence<int, B0...>) {
  f4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
  (
      [&] {
        c0 = __builtin_amdgcn_mfma_f32_4x4x4f16(a, w[2 * B0], c0, CBSZ, 2 * B0, 0);
        c1 = __builtin_amdgcn_mfma_f32_4x4x4f16(a, w[2 * B0 + 1], c1, CBSZ, 2 * B0 + 1, 0);
      }(),
      ...);
  return c0 + c1;
}

// M rows of a readout block as a binary tree of neighbours (the order in which y_parts_sum_kernel goes on
// over the parts of a state: y has the same bits however a state is split)
template <int M, int W>
__device__ __forceinline__ void tree_sum(const float *p, int stride, float (&out)[W]) {
  if constexpr (M == 1) {
    typedef float vec_t __attribute__((ext_vector_type(W)));
    if constexpr (W == 1) {
      out[0] = *p;
    } else {
      const vec_t x = *(const vec_t *)p;
#pragma unroll
      for (int i = 0; i < W; ++i) out[i] = x[i];
    }
  } else {
    float lo[W], hi[W];
    tree_sum<M / 2, W>(p, stride, lo);
    tree_sum<M / 2, W>(p + (M / 2) * stride, stride, hi);
#pragma unroll
    for (int i = 0; i < W; ++i) out[i] = lo[i] + hi[i];
  }
}

template <typename PT, bool DO_Y>
__global__ void __launch_bounds__(PT::THREADS, 2) half_fwd_kernel(FwdArgs a, float *__restrict__ ypart_ws) {
  constexpr int K = PT::K, V = PT::V, THREADS = PT::THREADS, PAIRS = PT::PAIRS, KB = PT::KB, YW = PT::YW;
  constexpr int NQ = (TB * PAIRS + THREADS - 1) / THREADS;    // staged row pairs per thread
  constexpr int NV = (TB * V / 2 + THREADS - 1) / THREADS;    // ... column pairs

  int unit, part;
  if (!map_block<PT::P>(a.B * a.N, unit, part)) return;
  const int T = a.T, N = a.N;
  const int b = unit / N, n = unit - b * N;
  const int g = n / (N / a.Nqk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane % V, pair = wave * PT::GR + lane / V;
  const bool odd = lane & 1, high = lane & 2;
  const int row_base = part * PT::ROWS;

  extern __shared__ __attribute__((aligned(16))) char lds[];
  PairSmem<PT> &sm = *(PairSmem<PT> *)lds;

  const uint32_t *__restrict__ qg = (const uint32_t *)((const bf16_raw *)a.q + ((size_t)b * T * a.Nqk + g) * K + row_base);
  const uint32_t *__restrict__ kg = (const uint32_t *)((const bf16_raw *)a.k + ((size_t)b * T * a.Nqk + g) * K + row_base);
  const size_t v0 = ((size_t)b * T * N + n) * V, v_step = (size_t)N * V, qk_step = (size_t)a.Nqk * K / 2;
  const uint32_t *__restrict__ vg = (const uint32_t *)((const bf16_raw *)a.v + v0);
  const float *__restrict__ fg = a.f + (size_t)b * T * N + n;

  // ---- state: rows 2 pair, + 1 of column col, scaled by c
  const size_t st_off = ((size_t)unit * K + row_base + 2 * pair) * V + col;
  float h[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    h[r] = a.H0 ? a.H0[st_off + r * V] : 0.f;
    if (T == 0 && a.HT) a.HT[st_off + r * V] = h[r];
    h[r] *= kC;
  }
  if (T == 0) return;

  // ---- W (B operand): slot e of block m is W[4 m + e][col]
  h4_t w[KB];
  {
    const bf16_raw *Wn = (const bf16_raw *)a.W + (size_t)n * V * V + col;
#pragma unroll
    for (int m = 0; m < KB; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) w[m][e] = (_Float16)bf16_to_f32(Wn[(size_t)(4 * m + e) * V]);
  }

  // ---- staging of q, k, v, f (TB steps per block); every thread loads from a valid (clamped)
  //      address, steps past the end of the sequence are staged but never used
  uint32_t rq[NQ], rk[NQ], rv[NV];
  float rf = 1.f;
  const float g_alpha = a.gate_alpha ? a.gate_alpha[n] : 0.f, g_beta = a.gate_alpha ? a.gate_beta[n] : 0.f;
  auto stage_load = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS, t = min(t0 + idx / PAIRS, T - 1);
      rq[m] = qg[t * qk_step + idx % PAIRS];
      rk[m] = kg[t * qk_step + idx % PAIRS];
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS, t = min(t0 + idx / (V / 2), T - 1);
      rv[m] = vg[t * (v_step / 2) + idx % (V / 2)];
    }
    rf = fg[(size_t)min(t0 + (tid & (TB - 1)), T - 1) * N];
  };
  auto stage_store = [&](int buf) __attribute__((always_inline)) {
    // keep the conversions here: hoisted to the loads they would wait for the loads at once
#pragma unroll
    for (int m = 0; m < NQ; ++m) asm volatile("" : "+v"(rq[m]), "+v"(rk[m]));
#pragma unroll
    for (int m = 0; m < NV; ++m) asm volatile("" : "+v"(rv[m]));
    asm volatile("" : "+v"(rf));
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS;
      if (TB * PAIRS % THREADS == 0 || idx < TB * PAIRS)
        (&sm.kq[buf][0][0])[idx] = f4_t{kC * bf16_to_f32((bf16_raw)rk[m]), kC * bf16_to_f32((bf16_raw)(rk[m] >> 16)),
                                        bf16_to_f32((bf16_raw)rq[m]), bf16_to_f32((bf16_raw)(rq[m] >> 16))};
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS;
      if (TB * V / 2 % THREADS == 0 || idx < TB * V / 2)
        ((float2 *)&sm.v[buf][0][0])[idx] =
            make_float2(bf16_to_f32((bf16_raw)rv[m]), bf16_to_f32((bf16_raw)(rv[m] >> 16)));
    }
    // the gate function by the last wave; its parameters are loaded once: a load here would wait
    // for the y and checkpoint stores in flight
    if (tid >= THREADS - 64 && lane < TB) {
      if (a.gate_alpha) rf = gate_psi(rf, g_alpha, g_beta);
      sm.f[buf][lane][0] = rf;
      sm.f[buf][lane][1] = kC * (1.f - rf);
    }
  };

  // ---- readout: thread -> (step, YW columns)
  const int ys = tid * YW / V, yc = tid * YW % V;
  float yv[YW], wr[YW];
#pragma unroll
  for (int i = 0; i < YW; ++i)
    wr[i] = PT::P == 1 && DO_Y && a.w_r ? bf16_to_f32(((const bf16_raw *)a.w_r)[n * V + yc + i]) : 0.f;
  auto y_store = [&](int buf, int t0, int len) __attribute__((always_inline)) {
    if (ys >= len) return;
    float s[YW];
    tree_sum<PAIRS, YW>(&sm.y[buf][ys][0][yc], V, s);
    const size_t off = v0 + (size_t)(t0 + ys) * v_step + yc;
    if constexpr (PT::P == 1) {
#pragma unroll
      for (int i = 0; i < YW; ++i) {
        s[i] *= kInvC;
        if (a.w_r) s[i] = fmaf(wr[i], yv[i], s[i]);  // residual w_r (.) v_t of the y equation
        ((bf16_raw *)a.y)[off + i] = __builtin_bit_cast(bf16_raw, (__bf16)s[i]);
      }
    } else {
      float *dst = ypart_ws + (size_t)part * a.B * T * v_step + off;
#pragma unroll
      for (int i = 0; i < YW; ++i) dst[i] = s[i];
    }
  };

  stage_load(0);
  stage_store(0);
  lds_barrier();

  const int nblk = (T + TB - 1) / TB;
  const int nck = (T + a.C - 1) / a.C;
  int next_ck = a.ckpt ? 0 : -1;
  float *__restrict__ ckpt =
      a.ckpt ? a.ckpt + (size_t)unit * nck * K * V + (size_t)(row_base + 2 * pair) * V + col : nullptr;

  struct StepRegs {
    f4_t kq;
    float v, f, gp;
  };
  auto step_L = [&](StepRegs &x, int s, int sb) __attribute__((always_inline)) {
    x.kq = sm.kq[sb][s][pair];
    const float2 ff = *(const float2 *)&sm.f[sb][s][0];
    x.f = ff.x;
    x.gp = ff.y;
    x.v = sm.v[sb][s][col];
  };
  h4_t ha = operand(h, odd, high);

  for (int blk = 0; blk < nblk; ++blk) {
    const int t0 = blk * TB;
    const int len = (T - t0) < TB ? (T - t0) : TB;
    const int sb = blk & 1;
    // Unconditional (the last block fetches itself again): behind a condition the compiler
    // merges old and new registers with copies that wait for the loads at once.
    stage_load(blk + 1 < nblk ? t0 + TB : t0);
    StepRegs nx;
    step_L(nx, 0, sb);
    auto step = [&](int s, bool last) __attribute__((always_inline)) {
      const StepRegs x = nx;
      if (t0 + s == next_ck) {  // state before step t0 + s
        ckpt[0] = h[0] * kInvC;
        ckpt[V] = h[1] * kInvC;
        ckpt += (size_t)K * V;
        next_ck += a.C;
      }
      if (s == TB / 2) stage_store(sb ^ 1);  // the next block's vectors have landed
      if (!last) step_L(nx, s + 1, sb);
      f4_t acc = contract<PT::CBSZ, KB>(ha, w, std::make_integer_sequence<int, KB / 2>{});
      settle(acc);
      h[0] = gate_tanh_step(x.f, x.gp, h[0], fmaf(x.kq[0], x.v, acc[0] + acc[2]));
      h[1] = gate_tanh_step(x.f, x.gp, h[1], fmaf(x.kq[1], x.v, acc[1] + acc[3]));
      ha = operand(h, odd, high);
      if constexpr (DO_Y) sm.y[sb][s][pair][col] = fmaf(x.kq[3], h[1], x.kq[2] * h[0]);
    };
    if (len == TB) {
#pragma unroll
      for (int s = 0; s < TB; ++s) step(s, s == TB - 1);
    } else {
#pragma nounroll
      for (int s = 0; s < len; ++s) step(s, s == len - 1);
#pragma unroll
      for (int m = 0; m < NQ; ++m) asm volatile("" : : "v"(rq[m]), "v"(rk[m]));
#pragma unroll
      for (int m = 0; m < NV; ++m) asm volatile("" : : "v"(rv[m]));
      asm volatile("" : : "v"(rf));
    }
    if constexpr (PT::P == 1 && DO_Y) {  // (behind the barrier the next block's v may take its place)
#pragma unroll
      for (int i = 0; i < YW; ++i) yv[i] = ys < TB ? sm.v[sb][ys][yc + i] : 0.f;
    }
    // One barrier per block: it closes this block's sums and the next block's vectors; this block's
    // buffers are written again only behind the next one.
    lds_barrier();
    if constexpr (DO_Y) y_store(sb, t0, len);
  }
  if (a.HT) {
    a.HT[st_off] = h[0] * kInvC;
    a.HT[st_off + V] = h[1] * kInvC;
  }
}

template <typename PT>
hipError_t launch(const FwdArgs &a, hipStream_t s) {
  const int units = a.B * a.N;
  if (units == 0) return hipSuccess;
  const dim3 grid(grid_blocks(units, PT::P)), block(PT::THREADS);
  constexpr int bytes = (int)sizeof(PairSmem<PT>), no_y = (int)offsetof(PairSmem<PT>, y);
  static_assert(bytes <= kLdsLimit, "LDS");
  hipError_t e;
  if (a.write_y) {
    if (bytes > 65536 && (e = set_max_lds_once(half_fwd_kernel<PT, true>, bytes)) != hipSuccess) return e;
    hipLaunchKernelGGL((half_fwd_kernel<PT, true>), grid, block, bytes, s, a, (float *)a.ws);
  } else if constexpr (PT::RB * PT::V <= 64) {  // (the others are taken for want of room, and no y needs none)
    hipLaunchKernelGGL((half_fwd_kernel<PT, false>), grid, block, no_y, s, a, (float *)a.ws);
  } else {
    return hipErrorInvalidValue;
  }
  e = hipGetLastError();
  if (e != hipSuccess || PT::P == 1 || !a.write_y || a.T == 0) return e;
  return y_parts_sum(a, PT::P, s);
}

}  // namespace

hipError_t pair_fwd(const FwdArgs &a, int rb, hipStream_t s) {
#define X(K_, V_, RB_, C_, R_) \
  if constexpr (R_) if (a.K == K_ && a.V == V_ && rb == RB_) return launch<Pair<K_, V_, RB_>>(a, s);
  M2RNN_HALF_CASES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace m2rnn
