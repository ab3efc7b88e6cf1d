// Matrix-core forward scan (Algorithm 1 of the paper; recurrence equations) on blocks of EIGHT
// state rows: the forward of the tiled path.
//
// A workgroup owns RB blocks of 8 rows of one (b, n) state and all V columns; a block is
// spread over V/16 waves of 16 columns.  The 16 rows of an MFMA's A operand are the 8 rows
// twice: operand row 4 g + {0, 1} is the hi part of rows 2 g, 2 g + 1 and operand row
// 4 g + {2, 3} the lo part (H' = hi + lo to ~21 bits, as in all forward kernels).  One
// 16x16x32 instruction therefore contracts 32 columns of both parts with an unrepeated W
// fragment, and a lane (column j = lane % 16, g = lane / 16) of the result holds the two
// partial sums of two state elements, rows 2 g and 2 g + 1 of column j.
//
// What bounds it, and why 8 rows: the scan is serial in T, and a launch with few states is
// bound by the latency of one step (LDS round trip, the contraction, the vector work of the
// one or two waves of a SIMD, the barrier).  Against 16-row blocks the vector work per wave
// and step is less than half (two elements per lane instead of four, no transposing product in
// the readout), the contraction is half as long a chain, and twice as many CUs take part.
//
// Per step:
//   L  the block's fragments through the transposing LDS load, the step's vectors
//   R  S' = c (H W), hi and lo rows
//   E  s' = S'_hi + S'_lo + (c k_i) v_j, gate_tanh_step, split; the lane's two rows are ONE
//      8-byte item {hi0, hi1, lo0, lo1} of the exchange layout; barrier (V > 16)
//   Y  readout y_t = H_t^T q_t: the item is, as it stands, the B operand of a 16x16x16 MFMA
//      over the rows (hi and lo both count), A = q_t in every row; row t mod 16 of the product
//      is kept, one register of 16 lanes per step, so that 16 steps of y collect in four registers.
//      (Kept by a select: with zeros in the other rows of A and a running sum, 0 x NaN would
//      carry a NaN of the state into the y of earlier steps.)
// Launches of few 32 x 32 or 64 x 64 states run on waves with whole rows instead (m2rnn_pair_fwd.hip).
// q, k, v, f for 16 steps at a time are staged through LDS, the next block's global loads in
// flight behind the current block.
#include "m2rnn_kernels.hpp"
#include "m2rnn_mfma_common.hpp"

#include <limits.h>

namespace m2rnn {
namespace {

constexpr int TB = 16;  // steps per staging / readout block (= MFMA N)

template <int K_, int V_, int RB_>
struct Half {
  static constexpr int K = K_, V = V_, RB = RB_;
  static constexpr int CT = V / 16;
  static constexpr int THREADS = RB * CT * 64;
  static constexpr int P = K / (8 * RB);
  static constexpr int ROWS = 8 * RB;
  static constexpr bool X32 = V >= 32;
  static constexpr int KS = X32 ? V / 32 : 1;
  static_assert(K % (8 * RB) == 0 && THREADS <= 1024, "bad split");
};

template <typename HT>
struct HalfSmem {
  alignas(16) char Hx[2][HT::RB][HT::V * 32];      // exchange items
  alignas(16) float kS[2][TB][HT::ROWS];           // c * k
  alignas(16) _Float16 qS[2][TB][HT::ROWS];
  alignas(16) float vS[2][TB][HT::V];
  alignas(16) float fS[2][TB][2];                  // f, c(1-f)
  alignas(16) f4_t yB[2][HT::RB][HT::CT][64];      // readout accumulators of a 16-step block
};

template <typename HF, bool DO_Y>
__global__ void __launch_bounds__(HF::THREADS, 2) half_fwd_kernel(FwdArgs a, float *__restrict__ ypart_ws) {
  constexpr int K = HF::K, V = HF::V, RB = HF::RB, CT = HF::CT, ROWS = HF::ROWS, KS = HF::KS;
  constexpr int THREADS = HF::THREADS;
  constexpr bool X32 = HF::X32;
  constexpr int NQ = (TB * ROWS + THREADS - 1) / THREADS;
  constexpr int NV = (TB * V + THREADS - 1) / THREADS;
  typedef typename Frag<X32>::type frag_t;
  constexpr int FE = X32 ? 8 : 4;

  int unit, part;
  if (!map_block<HF::P>(a.B * a.N, unit, part)) return;
  const int T = a.T, N = a.N;
  const int b = unit / N, n = unit - b * N;
  const int g = n / (N / a.Nqk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rb = wave / CT, ct = wave - rb * CT;
  const int jl = lane & 15, ig = lane >> 4;
  const int col0 = ct * 16, rowb = rb * 8;
  const int row_base = part * ROWS;

  __shared__ HalfSmem<HF> sm;

  const bf16_raw *__restrict__ qg = (const bf16_raw *)a.q;
  const bf16_raw *__restrict__ kg = (const bf16_raw *)a.k;
  const bf16_raw *__restrict__ vg = (const bf16_raw *)a.v;
  const float *__restrict__ fg = a.f;

  // ---- state: rows rowb + 2 ig, + 1 of column col0 + jl, scaled by c
  const size_t st_off = (size_t)unit * K * V + (size_t)(row_base + rowb + 2 * ig) * V + col0 + jl;
  float h[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    h[r] = a.H0 ? a.H0[st_off + r * V] : 0.f;
    if (T == 0 && a.HT) a.HT[st_off + r * V] = h[r];
    h[r] *= kC;
  }
  if (T == 0) return;

  // ---- W fragments (B operand): slot e of fragment m is W[(X32 ? 32 : 16) m + FE ig + e][col0 + jl]
  frag_t wf[KS];
  {
    const bf16_raw *Wn = (const bf16_raw *)a.W + (size_t)n * V * V + col0 + jl;
#pragma unroll
    for (int m = 0; m < KS; ++m)
#pragma unroll
      for (int e = 0; e < FE; ++e)
        wf[m][e] = (_Float16)bf16_to_f32(Wn[(size_t)(4 * FE * m + FE * ig + e) * V]);
  }

  // ---- exchange: item (column, ig) written by its lane, fragments read by every wave of the block
  lchar *const hx = (lchar *)&sm.Hx[0][0][0];
  constexpr int HXBUF = RB * V * 32;     // bytes of one exchange buffer
  constexpr int FRAG = 4 * FE * 32;      // ... of one fragment's columns
  lchar *const hx_w = hx + rb * V * 32 + xch_item_off(col0 + jl, ig);
  const lchar *const hx_r0 = hx + rb * V * 32 + xch_frag_off<X32>(jl, ig, 0);
  const lchar *const hx_r1 = hx + rb * V * 32 + xch_frag_off<X32>(jl, ig, 1);

  // ---- staging of q, k, v, f (TB steps per block); every thread loads from a valid (clamped)
  //      address, steps past the end of the sequence are staged but never used
  bf16_raw rq[NQ], rk[NQ], rv[NV];
  float rf = 1.f;
  const float g_alpha = a.gate_alpha ? a.gate_alpha[n] : 0.f, g_beta = a.gate_alpha ? a.gate_beta[n] : 0.f;
  auto stage_load = [&](int t0) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS;
      const int s = idx / ROWS, i = idx - s * ROWS;
      const int t = (t0 + s) < T ? (t0 + s) : (T - 1);
      const size_t off = (((size_t)b * T + t) * a.Nqk + g) * K + row_base + i;
      rq[m] = qg[off];
      rk[m] = kg[off];
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS;
      const int s = idx / V, j = idx - s * V;
      const int t = (t0 + s) < T ? (t0 + s) : (T - 1);
      rv[m] = vg[(((size_t)b * T + t) * N + n) * V + j];
    }
    const int t = (t0 + (tid & (TB - 1))) < T ? (t0 + (tid & (TB - 1))) : (T - 1);
    rf = fg[((size_t)b * T + t) * N + n];
  };
  auto stage_store = [&](int buf) {
    // keep the conversions here: hoisted to the loads they would wait for the loads at once
#pragma unroll
    for (int m = 0; m < NQ; ++m) asm volatile("" : "+v"(rq[m]), "+v"(rk[m]));
#pragma unroll
    for (int m = 0; m < NV; ++m) asm volatile("" : "+v"(rv[m]));
    asm volatile("" : "+v"(rf));
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int idx = tid + m * THREADS;
      if (idx < TB * ROWS) {
        (&sm.kS[buf][0][0])[idx] = kC * bf16_to_f32(rk[m]);
        (&sm.qS[buf][0][0])[idx] = (_Float16)bf16_to_f32(rq[m]);
      }
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int idx = tid + m * THREADS;
      if (idx < TB * V) (&sm.vS[buf][0][0])[idx] = bf16_to_f32(rv[m]);
    }
    // the gate function by the last wave (the first one also stores y); its parameters are
    // loaded once: a load here would wait for the y and checkpoint stores in flight
    if (tid >= THREADS - 64 && lane < TB) {
      if (a.gate_alpha) rf = gate_psi(rf, g_alpha, g_beta);
      sm.fS[buf][lane][0] = rf;
      sm.fS[buf][lane][1] = kC * (1.f - rf);
    }
  };
  // A block of one wave exchanges with itself only: its LDS accesses complete in order.
  auto step_barrier = [&]() __attribute__((always_inline)) {
    if constexpr (CT > 1) lds_barrier();
    else asm volatile("" ::: "memory");
  };

  stage_load(0);
  stage_store(0);
  lds_st<u2_t>(hx_w, 0, split2_hi_lo(h[0], h[1]));
  lds_barrier();

  const int nblk = (T + TB - 1) / TB;
  const int nck = (T + a.C - 1) / a.C;
  int next_ck = 0, ck_idx = 0;
  bf16_raw *__restrict__ yg = (bf16_raw *)a.y;
  const f4_t zero4 = {0.f, 0.f, 0.f, 0.f};

  struct StepRegs {
    frag_t hf[KS];
    float k0, k1, v, f, gp;
    uint32_t q;
  };
  auto ckpt_store = [&](int t) __attribute__((always_inline)) {
    if (a.ckpt && t == next_ck) {  // state before step t
      float *dst = a.ckpt + ((size_t)unit * nck + ck_idx) * K * V +
                   (size_t)(row_base + rowb + 2 * ig) * V + col0 + jl;
      dst[0] = h[0] * kInvC;
      dst[V] = h[1] * kInvC;
      next_ck += a.C;
      ++ck_idx;
    }
  };
  // L: fragments from exchange buffer `buf` first (they are needed first), then the vectors
  auto step_L = [&](StepRegs &x, int s, int sb, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < KS; ++m) x.hf[m] = lds_ld_frag_tr<X32>(hx_r0, hx_r1, buf * HXBUF + m * FRAG);
    const float2 kk = *(const float2 *)&sm.kS[sb][s][rowb + 2 * ig];
    const float2 ff = *(const float2 *)&sm.fS[sb][s][0];
    x.k0 = kk.x;
    x.k1 = kk.y;
    x.f = ff.x;
    x.gp = ff.y;
    x.v = sm.vS[sb][s][col0 + jl];
    if constexpr (DO_Y) x.q = *(const uint32_t *)&sm.qS[sb][s][rowb + 2 * ig];
  };
  // lane (ig, jl) of a block's readout holds steps 4 ig + r of column col0 + jl
  const size_t row = (size_t)N * V, y_lane = ((size_t)b * T + 4 * ig) * row + (size_t)n * V + col0 + jl;
  auto y_store = [&](f4_t ys, int t0, int len) __attribute__((always_inline)) {
    const size_t yoff = y_lane + t0 * row;
    if constexpr (HF::P == 1) {
      ys *= kInvC;
      if (a.w_r) {  // residual w_r (.) v_t of the y equation
        const float wr = bf16_to_f32(((const bf16_raw *)a.w_r)[n * V + col0 + jl]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * ig + r < len) ys[r] = fmaf(wr, bf16_to_f32(vg[yoff + r * row]), ys[r]);
      }
      bf16_raw *dst = yg + yoff;
      if (len == TB) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[r * row] = __builtin_bit_cast(bf16_raw, (__bf16)ys[r]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * ig + r < len) dst[r * row] = __builtin_bit_cast(bf16_raw, (__bf16)ys[r]);
      }
    } else {
      float *dst = ypart_ws + (size_t)part * a.B * T * row + yoff;
      if (len == TB) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[r * row] = ys[r];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * ig + r < len) dst[r * row] = ys[r];
      }
    }
  };

  for (int blk = 0; blk < nblk; ++blk) {
    const int t0 = blk * TB;
    const int len = (T - t0) < TB ? (T - t0) : TB;
    const int sb = blk & 1;
    // Unconditional (the last block fetches itself again): behind a condition the compiler
    // merges old and new registers with copies that wait for the loads at once.
    stage_load(blk + 1 < nblk ? t0 + TB : t0);
    f4_t yacc = zero4;  // [step t0 + 4 ig + r][column col0 + jl]: c * y partial
    StepRegs nx;
    step_L(nx, 0, sb, 0);
    auto step = [&](int s, bool last) __attribute__((always_inline)) {
      StepRegs x = nx;
      ckpt_store(t0 + s);
      if (s == TB / 2) stage_store(sb ^ 1);  // the next block's vectors have landed
      f4_t acc = zero4;
#pragma unroll
      for (int m = 0; m < KS; ++m) {
        if constexpr (X32) acc = mfma_k32(x.hf[m], wf[m], acc);
        else acc = mfma_k16(x.hf[m], wf[m], acc);
      }
      settle(acc);
      h[0] = gate_tanh_step(x.f, x.gp, h[0], fmaf(x.k0, x.v, acc[0] + acc[2]));
      h[1] = gate_tanh_step(x.f, x.gp, h[1], fmaf(x.k1, x.v, acc[1] + acc[3]));
      const u2_t it = split2_hi_lo(h[0], h[1]);
      lds_st<u2_t>(hx_w, ((s & 1) ^ 1) * HXBUF, it);  // (a full block has 16 steps: parity of s)
      step_barrier();
      if (!last) step_L(nx, s + 1, sb, (s + 1) & 1);
      if constexpr (DO_Y) {
        const f4_t yd = mfma_k16(__builtin_bit_cast(h4_t, u2_t{x.q, x.q}), __builtin_bit_cast(h4_t, it), zero4);
#pragma unroll
        for (int r = 0; r < 4; ++r) yacc[r] = 4 * ig + r == s ? yd[r] : yacc[r];
      }
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
    settle(yacc);
    if constexpr (DO_Y) {
      // block flush: the row blocks are added through LDS (yB alternates: with one wave per
      // row block the barrier below is the only one of a block)
      if constexpr (RB > 1) {
        if (rb > 0) sm.yB[sb][rb][ct][lane] = yacc;
      }
      if constexpr (RB > 1 || CT == 1) lds_barrier();
      if (rb == 0) {
        if constexpr (RB > 1) {
          f4_t part[RB];
          part[0] = yacc;
#pragma unroll
          for (int r2 = 1; r2 < RB; ++r2) part[r2] = sm.yB[sb][r2][ct][lane];
          yacc = pairwise_sum(part);
        }
        y_store(yacc, t0, len);
      }
    } else if constexpr (CT == 1) {
      lds_barrier();  // the next block's staged vectors
    }
  }
  if (a.HT) {
    a.HT[st_off] = h[0] * kInvC;
    a.HT[st_off + V] = h[1] * kInvC;
  }
}

template <typename HF>
hipError_t launch(const FwdArgs &a, hipStream_t s) {
  const int units = a.B * a.N;
  if (units == 0) return hipSuccess;
  float *ypart = (float *)a.ws;
  const dim3 grid(grid_blocks(units, HF::P)), block(HF::THREADS);
  if (a.write_y) hipLaunchKernelGGL((half_fwd_kernel<HF, true>), grid, block, 0, s, a, ypart);
  else if constexpr (HF::K < 128 || HF::RB == 1)  // (that split is taken for want of room, and no y needs none)
    hipLaunchKernelGGL((half_fwd_kernel<HF, false>), grid, block, 0, s, a, ypart);
  else return hipErrorInvalidValue;
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || HF::P == 1 || !a.write_y || a.T == 0) return e;
  return y_parts_sum(a, HF::P, s);
}

}  // namespace

// Row blocks per workgroup: the split with the fewest waves on the fullest SIMD (workgroups are
// dealt evenly over 256 CUs; a step takes as long as the waves of the fullest SIMD need for it).
// Among equals the smallest workgroup that still gives every workgroup a CU (the row blocks of a
// workgroup wait for each other), else the largest (fewer partial sums of y).  Only splits whose
// partial sums fit `avail` bytes; 0 if there is none.  Parts of a state cost a second launch
// for the sum of their y, some 2.5 us, and save 0.01 us a step, 0.05 more for every wave that the fullest
// SIMD has less: where one workgroup can hold a state, they are taken from the T on that repays the launch.
// One part / parts, us: 64 x 32, 8 states, T = 4 8.2 / 11.2, 17 10.3 / 11.1, 24 13.4 / 11.1; 32 x 32, 8 states,
// T = 32 11.3 / 11.2, 48 15.3 / 14.1, 200 53.9 / 43.6 (launches in a graph, on waves with whole rows: 16 states
// T = 16 6.9 / 7.5, 24 9.4 / 9.4, 44 14.1 / 12.9, 128 states 24 9.7 / 10.2, 44 14.1 / 13.8); 16 x 16, 8 states, T = 128 22.7 / 22.6, 256 46 / 40.1.
// Measured (us, forward, no checkpoints
// unless stated, RB = 1 / 2 / 4 / 8):
//   64 x 64, T 8192: 32 states 1735 / 2134 (waves with whole rows; sharing columns 1772 / 2122 / 2938);  T 4096: 64 states 1105 / 1097 / 1491, 96 states
//   1388 / 1518 / 1510;  T 2048 with checkpoints: 128 states 862 / 787 / 772
//   32 x 32, with checkpoints: 16 states, T 333 60.8 / 61.3 / 75 (whole rows; 69 / 74 / 85);  128, T 2048
//   sharing columns 458 / 431 / 499, whole rows RB = 2 365;
//   512, T 1024 408 / 355 / 336
//   64 x 16, T 777: 84 states 131 / 146 / 119 / 137;  336 252 / 233 / 184 / 216;  504 273 / 246 / 229 / 217
namespace {
// waves on the fullest SIMD
long long half_load(int K, int V, int units, int rb) {
  const long long groups = (long long)units * (K / (8 * rb));
  return ((groups + 255) / 256 * rb * (V / 16) + 3) / 4;
}
}  // namespace
int half_pick_rb(int K, int V, int units, size_t part_bytes, size_t avail, int T) {
  int best = 0, whole = 0;  // whole: one workgroup per state
  long long best_load = 0;
  bool best_fits = false;
  auto consider = [&](int rb) {  // (in increasing rb)
    const int P = K / (8 * rb);
    if (P > 1 && (size_t)P * part_bytes > avail) return;
    const long long groups = (long long)units * P, load = half_load(K, V, units, rb);
    if (!best || load < best_load || (load == best_load && !best_fits))
      best = rb, best_load = load, best_fits = groups <= 256;
    if (P == 1) whole = rb;
  };
#define X(K_, V_, RB_, C_, R_) \
  if (K == K_ && V == V_) consider(RB_);
  M2RNN_HALF_CASES(X)
#undef X
  if (!whole || whole == best) return best;
  return T * (4 * (half_load(K, V, units, whole) - best_load) + 1) < 224 ? whole : best;
}

// Which launches: below two 16-row blocks per SIMD (1024 SIMDs) of all shapes that have a split;
// beyond, one wave per 16 rows and all columns (m2rnn_rowwave_fwd.hip) needs no exchange and is
// faster.  128 x 128 only while twice as many workgroups have a CU each: T = 2048 with checkpoints,
// 16-row tile -> RB = 1: 8 states 933 -> 655 us, 16 states 947 -> 686, but 32 states 982 -> 1381
// (RB = 2: 1037; the exchange traffic of sixteen waves meets in one LDS).
// Shapes with V = 32 have a 16-row kernel whose waves the same number of states fills evenly (one or two
// on every SIMD for each 256 of them); 8-row waves are half of one, and from five on a SIMD, where latency
// no longer counts, the fullest SIMD's odd wave decides.  us, 16-row kernel -> this one:
//   64 x 32, row-wave, T = 512: 200 states 219 -> 180, 257 302 -> 231, 384 310 -> 271 (load 6), 400 306 -> 296
//   (7; T = 48 31.5 -> 35.8), 450 308 -> 356 (8); without a workspace (one part per state) 200 217 -> 180, but
//   257 to 384 305 -> 350; 300 states, T = 48 31.3 -> 30.5, 24 18.5 -> 21.2, 8 9.3 -> 15.6.
//   32 x 32, tile: T = 512: 512 states 193 -> 169 (4), 513 241 -> 231 (5), 700 247 -> 269 (6), 900 327 -> 329;
//   600 states, T = 100 52.7 -> 55.4, 32 19.3 -> 22.1.
//   32 x 16, row-wave, T = 512: 200 140 -> 86, 511 182 -> 98, 1023 179 -> 145, without a workspace the same.
// (The choice does not look at the workspace: a call's bits do not depend on its room.)
bool half_serves(int K, int V, int units, int T) {
  const int rb = half_pick_rb(K, V, units, 0, 0, INT_MAX);
  if (!rb) return false;
  if (K == 128) return (long long)units * (K / 8) <= 256;
  if ((long long)units * (K / 16) >= 2048) return false;
  const long long load = half_load(K, V, units, rb);
  return V != 32 || load <= 4 || (K == 64 && load <= 6 && T >= 32);
}

namespace {
// Which launches of this path run on one wave per 128 elements (m2rnn_pair_fwd.hip): square states, as few as
// leave every wave a SIMD on the finest split.  us, T = 2048, waves that share columns -> waves with whole rows: 64 x 64
// 4 states 420 -> 399, 16 431 -> 410, 32 443 -> 424, but 128 (four waves a SIMD, with checkpoints, T = 4096) 1550 -> 2120;
// 32 x 32 16 states 402 -> 334; 64 x 16 16 states 287 -> 300.  On the coarser splits that short sequences take they are
// the faster ones too: 32 x 32, one workgroup per state (two waves a SIMD), 16 states, T = 8 6.4 -> 5.8 us, 44 15.6 -> 14.0.
// (By the shape and the states alone, not by the split that the room allows: y's bits do not depend on the room.
// So not 64 x 32: 405 -> 339 on the finest split, but without a workspace one workgroup holds the state, four waves
// a SIMD, and 16 states take 661 -> 750 us, T = 16 9.2 -> 10.3.)
bool pair_serves(int K, int V, int units) {
  return K == V && (V == 32 || V == 64) && half_load(K, V, units, 1) <= 1;
}
}  // namespace
hipError_t half_fwd(const FwdArgs &a, hipStream_t s) {
  // (a pass that only writes checkpoints has no partial sums)
  const size_t part = a.write_y ? (size_t)a.B * a.T * a.N * a.V * 4 : 0;
  const int rb = half_pick_rb(a.K, a.V, a.B * a.N, part, a.ws_bytes, a.write_y ? a.T : INT_MAX);
  if (rb && pair_serves(a.K, a.V, a.B * a.N)) return pair_fwd(a, rb, s);
#define X(K_, V_, RB_, C_, R_) \
  if constexpr (C_) if (a.K == K_ && a.V == V_ && rb == RB_) return launch<Half<K_, V_, RB_>>(a, s);
  M2RNN_HALF_CASES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace m2rnn
