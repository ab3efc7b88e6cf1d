// Gradients of the scan's options that are sums over all (b, t): dw_r of the residual of the y
// equation, dalpha and dbeta of the gate function (whose chain rule also finishes df in place).
//
// Both are one pass over [B*T, columns] arrays and a column sum, so memory bounds them: what
// matters is that enough loads are in flight.  A workgroup takes up to 256 columns and deals the
// rows to walkers (as many as its threads allow), a walker keeps four rows in flight, the
// walkers are added in LDS and the workgroups by rows_sum_kernel.  Every order is fixed.
// B T = 32000, N = 16, V = 64, bf16: dw_r 299 -> 29 us (131 MB of dy and v), gate 164 -> 12 us;
// one column per thread and a serial second stage over 1024 rows took the longer times.
#include "m2rnn_io.hpp"
#include "m2rnn_kernels.hpp"
#include "m2rnn_mfma_common.hpp"

namespace m2rnn {
namespace {

constexpr int kThreads = 256;
constexpr int kAhead = 4;  // rows of a walker whose loads are issued together
constexpr int kDwrStages = 1024, kGateStages = 256;  // most partial rows (the scratch is sized for them)
constexpr int kBlocks = 1024;  // workgroups that fill the chip (four on each CU)

// part[s][c] = sum over the rows of workgroup row s of dy[r][c] v[r][c]; cw = column vectors of
// eight per workgroup (NV is a multiple of 16, the tensors are 16-byte aligned)
template <typename IO>
__global__ void __launch_bounds__(kThreads)
    dwr_stage1_kernel(const IO *__restrict__ dy, const IO *__restrict__ v, float *__restrict__ part, size_t BT,
                      int NV, int cw) {
  __shared__ __attribute__((aligned(16))) float red[kThreads][8];
  const int walkers = kThreads / cw, wl = threadIdx.x / cw, cl = threadIdx.x - wl * cw;
  const int c = (blockIdx.x * cw + cl) * 8;
  const size_t step = (size_t)gridDim.y * walkers;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (wl < walkers && c < NV) {
    size_t r = (size_t)blockIdx.y * walkers + wl;
    auto add = [&](const typename Vec8<IO>::Raw &rx, const typename Vec8<IO>::Raw &ry) {
      float x[8], y[8];
      Vec8<IO>::widen(rx, x);
      Vec8<IO>::widen(ry, y);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fmaf(x[i], y[i], acc[i]);
    };
    for (; r + (kAhead - 1) * step < BT; r += kAhead * step) {
      typename Vec8<IO>::Raw x[kAhead], y[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        x[u] = Vec8<IO>::load_raw(dy, (r + u * step) * NV + c);
        y[u] = Vec8<IO>::load_raw(v, (r + u * step) * NV + c);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) add(x[u], y[u]);
    }
    for (; r < BT; r += step) add(Vec8<IO>::load_raw(dy, r * NV + c), Vec8<IO>::load_raw(v, r * NV + c));
  }
  *(f4_t *)&red[threadIdx.x][0] = f4_t{acc[0], acc[1], acc[2], acc[3]};
  *(f4_t *)&red[threadIdx.x][4] = f4_t{acc[4], acc[5], acc[6], acc[7]};
  __syncthreads();
  const int col = blockIdx.x * cw * 8 + threadIdx.x;
  if ((int)threadIdx.x < cw * 8 && col < NV) {
    float s = 0.f;
    for (int w = 0; w < walkers; ++w) s += red[w * cw + threadIdx.x / 8][threadIdx.x % 8];
    part[(size_t)blockIdx.y * NV + col] = s;
  }
}

// Chain rule through the gate function.  df holds dL/d(gate value) g; with u = x + beta,
// psi = exp(-alpha softplus(u)):  dL/dx = dL/dbeta-term = -g alpha psi sigmoid(u),
// dL/dalpha-term = -g psi softplus(u).  part[s][0 or 1][n]: dalpha, dbeta of workgroup row s;
// cw = heads per workgroup.
__global__ void __launch_bounds__(kThreads)
    gate_bwd_stage1_kernel(float *__restrict__ df, const float *__restrict__ x, const float *__restrict__ alpha,
                           const float *__restrict__ beta, float *__restrict__ part, size_t BT, int N, int cw) {
  __shared__ float red[2][kThreads];
  const int walkers = kThreads / cw, wl = threadIdx.x / cw, cl = threadIdx.x - wl * cw;
  const int n = blockIdx.x * cw + cl;
  const size_t step = (size_t)gridDim.y * walkers;
  float sa = 0.f, sb = 0.f;
  if (wl < walkers && n < N) {
    const float al = alpha[n], be = beta[n];
    auto one = [&](float xv, float g) {
      const float u = xv + be;
      const float sp = fmaxf(u, 0.f) + log1pf(expf(-fabsf(u)));
      const float psi = expf(-al * sp);
      const float dx = -g * al * psi / (1.f + expf(-u));
      sa = fmaf(-g * psi, sp, sa);
      sb += dx;
      return dx;
    };
    size_t r = (size_t)blockIdx.y * walkers + wl;
    for (; r + (kAhead - 1) * step < BT; r += kAhead * step) {
      float xv[kAhead], g[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        xv[u] = x[(r + u * step) * N + n];
        g[u] = df[(r + u * step) * N + n];
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) df[(r + u * step) * N + n] = one(xv[u], g[u]);
    }
    for (; r < BT; r += step) df[r * N + n] = one(x[r * N + n], df[r * N + n]);
  }
  red[0][threadIdx.x] = sa;
  red[1][threadIdx.x] = sb;
  __syncthreads();
  if (wl < 2 && n < N) {  // (walkers >= 4)
    float s = 0.f;
    for (int w = 0; w < walkers; ++w) s += red[wl][w * cw + cl];
    part[((size_t)blockIdx.y * 2 + wl) * N + n] = s;
  }
}

// Column sums of part [S][E]; columns from `split` on go to out1.
__global__ void __launch_bounds__(1024)
    rows_sum_kernel(const float *__restrict__ part, int S, int E, float *__restrict__ out0, int split,
                    float *__restrict__ out1) {
  const int c = blockIdx.x * 32 + (threadIdx.x & 31);
  const float t = column_sum(part, E, c, 0, S);
  if (threadIdx.x < 32 && c < E) {
    if (c < split) out0[c] = t;
    else out1[c - split] = t;
  }
}

hipError_t rows_sum(const float *part, int S, int E, float *out0, int split, float *out1, hipStream_t s) {
  hipLaunchKernelGGL(rows_sum_kernel, dim3((E + 31) / 32), dim3(1024), 0, s, part, S, E, out0, split, out1);
  return hipGetLastError();
}

// Workgroup rows: enough for kAhead rows per walker, no more than fill the chip with `gx`
// workgroups side by side (further ones only add partial rows).
int stage_rows(size_t BT, int walkers, int gx, int most) {
  const size_t per = (size_t)kAhead * walkers, want = (BT + per - 1) / per;
  const int cap = kBlocks / gx < 1 ? 1 : kBlocks / gx < most ? kBlocks / gx : most;
  return want < (size_t)cap ? (int)want : cap;
}

template <typename IO>
hipError_t dwr(const BwdArgs &a, hipStream_t s) {
  const int NV = a.N * a.V, cv = NV / 8, cw = cv < 32 ? cv : 32, gx = (cv + cw - 1) / cw;
  const size_t BT = (size_t)a.B * a.T;
  const int S = stage_rows(BT, kThreads / cw, gx, kDwrStages);
  if (S > 0) {
    hipLaunchKernelGGL(dwr_stage1_kernel<IO>, dim3(gx, S), dim3(kThreads), 0, s, (const IO *)a.dy,
                       (const IO *)a.v, a.dwr_ws, BT, NV, cw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return rows_sum(a.dwr_ws, S, NV, a.dw_r, NV, nullptr, s);
}

}  // namespace

size_t gate_scratch_bytes(int N) { return align256((size_t)kGateStages * 2 * N * sizeof(float)); }

hipError_t gate_backward(const BwdArgs &a, hipStream_t s) {
  const int cw = a.N < 64 ? a.N : 64, gx = (a.N + cw - 1) / cw;
  const size_t BT = (size_t)a.B * a.T;
  const int S = stage_rows(BT, kThreads / cw, gx, kGateStages);
  if (S > 0) {
    hipLaunchKernelGGL(gate_bwd_stage1_kernel, dim3(gx, S), dim3(kThreads), 0, s, a.df, a.f, a.gate_alpha,
                       a.gate_beta, a.gate_ws, BT, a.N, cw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return rows_sum(a.gate_ws, S, 2 * a.N, a.dgate_alpha, a.N, a.dgate_beta, s);
}

size_t residual_dw_r_scratch_bytes(int N, int V) {
  return align256((size_t)kDwrStages * N * V * sizeof(float));
}

hipError_t residual_dw_r(const BwdArgs &a, hipStream_t s) {
  return a.io == 0 ? dwr<float>(a, s) : dwr<__hip_bfloat16>(a, s);
}

}  // namespace m2rnn
