// The scan's two neighbours in the M2RNN block (layer equations of the "M2RNN Block"
// section), as bandwidth-bound kernels that touch every tensor once:
//   * prologue of q, k, v:  out = SiLU(conv1d(x)), depthwise causal convolution of kernel
//     size 4 along time (zero left padding; tap j meets step t - 3 + j), and its backward;
//   * epilogue of y:  out = RMSNorm(y (.) SiLU(a)) over all D = N V features of a token
//     (forward and backward as printed in the "RMSNormTP Module" appendix, eps under the
//     root), and its backward.
// Why they are kernels of their own and not folded into the scan kernels: the norm spans all
// heads of a token while a scan workgroup holds one head, and the scan is bound by its vector
// ALUs with HBM at a few percent of peak, where a convolution re-evaluated by every workgroup
// that stages the same q, k, v rows would add exactly the instructions that bind it.  Here
// each tensor makes one trip through HBM: x -> out, and (y, a) -> out.
// Sums over tokens (dw, dbias) are two-stage and ordered: bit-reproducible, no atomics.
#include "m2rnn_io.hpp"
#include "m2rnn_kernels.hpp"
#include "m2rnn_mfma_common.hpp"

#include <algorithm>

namespace m2rnn {
namespace {

// 1 / (1 + e^-u) on the hardware's exp2 and reciprocal (1 ulp each; e^-u = inf gives 0)
__device__ __forceinline__ float sigmoidf_(float u) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * u));
}

// ------------------------------------------------------------------ conv1d(4) + SiLU
constexpr int kTaps = 4;
constexpr int kThreads = 256;

// taps [4 channels][4] (16 consecutive elements of w [C,4]) and bias of channels c0 .. c0 + 3
template <typename IO>
__device__ __forceinline__ void load_taps(const void *w, const void *bias, int c0, float (&wt)[4][kTaps],
                                          float (&bs)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) Vec4<IO>::widen(Vec4<IO>::load_raw(w, ((size_t)c0 + i) * kTaps), wt[i]);
  if (bias) Vec4<IO>::widen(Vec4<IO>::load_raw(bias, c0), bs);
  else
#pragma unroll
    for (int i = 0; i < 4; ++i) bs[i] = 0.f;
}

// How a launch is dealt out.  A work item is four channels x `seg` steps of one batch row; a
// workgroup is `cw` channel vectors (at most 64, gx workgroups side by side) x kThreads / cw walkers,
// and walker w of rg workgroup rows takes the rows w, w + walkers, ... of the B * nseg segments.
//
// Four channels, not eight: taps, windows and sums are half the registers, 4 waves per SIMD in the
// backward instead of 2, whose arithmetic and loads then overlap.  cw is a multiple of eight where
// it can be: with 31 instead of 32 vectors side by side the forward of 1472 channels took 48 us, not
// 37.  Long segments read fewer halo rows twice, short ones fill the chip with a short tensor: the
// longest segment is taken that still gives kConvItems items (262144, every thread resident:
// 8 x 4000 x 520 in 48 us backward, 39 with this).  Forward / backward, bf16, before and now:
//   8 x 4096 x 1472   42 / 101 -> 36 / 77 us        2 x 150 x 1016   20 / 37 -> 5 / 11 us
struct ConvPlan {
  int seg, nseg, cw, gx, walkers, rg;
};
constexpr long long kConvItems = 160 * 1024;

inline ConvPlan conv_plan(int B, int T, int C, int most_rows) {
  ConvPlan p;
  const int CV = C / 4;
  p.gx = (CV + 63) / 64;
  p.cw = ((CV + p.gx - 1) / p.gx + 7) & ~7;
  if (p.cw > CV) p.cw = CV;
  p.walkers = kThreads / p.cw;
  p.seg = 64;
  while (p.seg > 8 && (long long)B * ((T + p.seg - 1) / p.seg) * CV < kConvItems) p.seg /= 2;
  p.nseg = (T + p.seg - 1) / p.seg;
  const long long want = ((long long)B * p.nseg + p.walkers - 1) / p.walkers;
  p.rg = (int)(want < 1 ? 1 : want < most_rows ? want : most_rows);
  return p;
}

template <typename IO>
__global__ void __launch_bounds__(kThreads)
    conv_silu_fwd_kernel(const void *__restrict__ x, const void *__restrict__ w,
                         const void *__restrict__ bias, void *__restrict__ out, int B, int T, int C, ConvPlan p) {
  constexpr int BLK = 8;  // steps whose loads are issued together
  const int wl = threadIdx.x / p.cw, cl = threadIdx.x - wl * p.cw;
  const int bx = blockIdx.x % p.gx, rgi = blockIdx.x / p.gx;
  const int cv = bx * p.cw + cl, rows = B * p.nseg;
  if (wl >= p.walkers || cv >= C / 4) return;
  const int c0 = cv * 4;
  float wt[4][kTaps], bs[4];
  load_taps<IO>(w, bias, c0, wt, bs);
  for (long long r = (long long)rgi * p.walkers + wl; r < rows; r += (long long)p.rg * p.walkers) {
    const int seg = (int)r % p.nseg, b = (int)r / p.nseg;
    const int t0 = seg * p.seg, t1 = t0 + p.seg < T ? t0 + p.seg : T;
    const size_t base = (size_t)b * T * C + c0;
    float win[kTaps - 1][4];  // steps t-3, t-2, t-1
#pragma unroll
    for (int j = 0; j < kTaps - 1; ++j) {
      const int ts = t0 - (kTaps - 1) + j;
      if (ts >= 0) Vec4<IO>::widen(Vec4<IO>::load_raw(x, base + (size_t)ts * C), win[j]);
      else
#pragma unroll
        for (int i = 0; i < 4; ++i) win[j][i] = 0.f;
    }
    for (int tb = t0; tb < t1; tb += BLK) {
      typename Vec4<IO>::Raw raw[BLK];
#pragma unroll
      for (int u = 0; u < BLK; ++u)  // (clamped: every load is unconditional)
        raw[u] = Vec4<IO>::load_raw(x, base + (size_t)(tb + u < t1 ? tb + u : t1 - 1) * C);
#pragma unroll
      for (int u = 0; u < BLK; ++u) {
        if (tb + u < t1) {
          float cur[4], o[4];
          Vec4<IO>::widen(raw[u], cur);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = bs[i] + wt[i][0] * win[0][i] + wt[i][1] * win[1][i] + wt[i][2] * win[2][i] +
                            wt[i][3] * cur[i];
            o[i] = a * sigmoidf_(a);
            win[0][i] = win[1][i];
            win[1][i] = win[2][i];
            win[2][i] = cur[i];
          }
          Vec4<IO>::store(out, base + (size_t)(tb + u) * C, o);
        }
      }
    }
  }
}

// Backward.  A work item recomputes the pre-activation of its own steps and of the three
// after them (their gradients reach back into its steps), forms da = dout SiLU'(a), and
// finishes dx of step t-3 as soon as da of step t is known.  dw and dbias of its OWN steps are
// summed per walker over the items it walks (increasing time inside a batch row, increasing
// batch row), the walkers of a workgroup through LDS (increasing), and written to
// part[workgroup row][C][5]; the ordered sum behind adds those.
template <typename IO>
__global__ void __launch_bounds__(kThreads, 4)
    conv_silu_bwd_kernel(const void *__restrict__ x, const void *__restrict__ w,
                         const void *__restrict__ bias, const void *__restrict__ dout,
                         void *__restrict__ dx, float *__restrict__ part, int B, int T, int C, ConvPlan p) {
  constexpr int BLK = sizeof(IO) == 4 ? 4 : 8;  // steps whose loads are issued together
  constexpr int PER = 4 * (kTaps + 1);          // sums per channel vector: [4 channels][4 taps, bias]
  __shared__ float red[kThreads][PER + 1];
  const int wl = threadIdx.x / p.cw, cl = threadIdx.x - wl * p.cw;
  const int bx = blockIdx.x % p.gx, rgi = blockIdx.x / p.gx;
  const int cv = bx * p.cw + cl, rows = B * p.nseg;
  const bool walker = wl < p.walkers && cv < C / 4;
  const int c0 = (cv < C / 4 ? cv : C / 4 - 1) * 4;
  float wt[4][kTaps], bs[4], dwacc[4][kTaps], dbacc[4];
  load_taps<IO>(w, bias, c0, wt, bs);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < kTaps; ++j) dwacc[i][j] = 0.f;
    dbacc[i] = 0.f;
  }
  for (long long r = walker ? (long long)rgi * p.walkers + wl : rows; r < rows; r += (long long)p.rg * p.walkers) {
    const int seg = (int)r % p.nseg, b = (int)r / p.nseg;
    const int t0 = seg * p.seg, t1 = t0 + p.seg < T ? t0 + p.seg : T;
    const size_t base = (size_t)b * T * C + c0;
    float win[kTaps - 1][4], dawin[kTaps - 1][4];  // x and da of steps t-3, t-2, t-1
#pragma unroll
    for (int j = 0; j < kTaps - 1; ++j) {
      const int ts = t0 - (kTaps - 1) + j;
      if (ts >= 0) Vec4<IO>::widen(Vec4<IO>::load_raw(x, base + (size_t)ts * C), win[j]);
      else
#pragma unroll
        for (int i = 0; i < 4; ++i) win[j][i] = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) dawin[j][i] = 0.f;  // da of earlier steps does not reach mine
    }
    const int tend = t1 + (kTaps - 1), tlast = (tend < T ? tend : T) - 1;
    for (int tb = t0; tb < tend; tb += BLK) {
      typename Vec4<IO>::Raw rx[BLK], rd[BLK];
#pragma unroll
      for (int u = 0; u < BLK; ++u) {  // (clamped: every load is unconditional)
        const size_t e = base + (size_t)(tb + u < tlast ? tb + u : tlast) * C;
        rx[u] = Vec4<IO>::load_raw(x, e);
        rd[u] = Vec4<IO>::load_raw(dout, e);
      }
#pragma unroll
      for (int u = 0; u < BLK; ++u) {
        const int t = tb + u;
        if (t >= tend) break;
        float cur[4], da[4];
        if (t < T) {
          float dd[4];
          Vec4<IO>::widen(rx[u], cur);
          Vec4<IO>::widen(rd[u], dd);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = bs[i] + wt[i][0] * win[0][i] + wt[i][1] * win[1][i] + wt[i][2] * win[2][i] +
                            wt[i][3] * cur[i];
            const float sg = sigmoidf_(a);
            da[i] = dd[i] * (sg * (1.f + a * (1.f - sg)));
          }
          if (t < t1) {  // my own step: its share of dw, dbias
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              dwacc[i][0] = fmaf(da[i], win[0][i], dwacc[i][0]);
              dwacc[i][1] = fmaf(da[i], win[1][i], dwacc[i][1]);
              dwacc[i][2] = fmaf(da[i], win[2][i], dwacc[i][2]);
              dwacc[i][3] = fmaf(da[i], cur[i], dwacc[i][3]);
              dbacc[i] += da[i];
            }
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) { cur[i] = 0.f; da[i] = 0.f; }
        }
        const int td = t - (kTaps - 1);  // dx of this step is complete now
        if (td >= t0) {
          float o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            o[i] = wt[i][3] * dawin[0][i] + wt[i][2] * dawin[1][i] + wt[i][1] * dawin[2][i] + wt[i][0] * da[i];
          Vec4<IO>::store(dx, base + (size_t)td * C, o);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          win[0][i] = win[1][i]; win[1][i] = win[2][i]; win[2][i] = cur[i];
          dawin[0][i] = dawin[1][i]; dawin[1][i] = dawin[2][i]; dawin[2][i] = da[i];
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < kTaps; ++j) red[threadIdx.x][i * (kTaps + 1) + j] = dwacc[i][j];
    red[threadIdx.x][i * (kTaps + 1) + kTaps] = dbacc[i];
  }
  __syncthreads();
  float *dst = part + ((size_t)rgi * C + (size_t)bx * p.cw * 4) * (kTaps + 1);
  for (int o = threadIdx.x; o < p.cw * PER; o += kThreads) {
    const int c = o / PER, j = o - c * PER;
    if (bx * p.cw + c < C / 4) {
      float acc = red[c][j];
      for (int q = 1; q < p.walkers; ++q) acc += red[q * p.cw + c][j];
      dst[o] = acc;
    }
  }
}

// Ordered sum of R partial rows of E floats.  A workgroup adds up to 32 columns with 32 walkers
// (rows wl, wl + 32, ..., four loads in flight) and the walkers in LDS.  Up to kDirectRows rows
// that is all; more are first added in groups of about kDirectRows / 4 (blockIdx.y) into rows
// of `lvl` (kSumGroups rows behind the partials).  What bounds it is the chain of dependent
// loads: 128 rows of 7360 took two launches, some 13 us, with one column per thread; 4.7 us now.
constexpr int kSumGroups = 32;
constexpr int kDirectRows = 512;

// column e of a plain [D] result, and of the convolution's [C][4 taps, bias]
struct PlainOut {
  float *out;
  __device__ __forceinline__ void put(int e, float s) const { out[e] = s; }
};
struct ConvOut {
  float *dw, *dbias;
  __device__ __forceinline__ void put(int e, float s) const {
    const int c = e / (kTaps + 1), j = e - c * (kTaps + 1);
    if (j < kTaps) dw[c * kTaps + j] = s;
    else if (dbias) dbias[c] = s;
  }
};
template <typename Out>
__global__ void __launch_bounds__(1024)
    ordered_sum_kernel(const float *__restrict__ part, float *__restrict__ lvl, Out out, int E, int R) {
  const int e = blockIdx.x * 32 + (threadIdx.x & 31), per = (R + gridDim.y - 1) / gridDim.y;
  const int r0 = blockIdx.y * per, r1 = r0 + per < R ? r0 + per : R;
  const float t = column_sum(part, E, e, r0, r1);
  if (threadIdx.x < 32 && e < E) {
    if (gridDim.y > 1) lvl[(size_t)blockIdx.y * E + e] = t;
    else out.put(e, t);
  }
}
template <typename Out>
hipError_t ordered_sum(const float *part, float *lvl, const Out &out, int E, int R, hipStream_t s) {
  const int bx = (E + 31) / 32;
  if (R > kDirectRows) {
    const int want = (R + kDirectRows / 4 - 1) / (kDirectRows / 4), G = want < kSumGroups ? want : kSumGroups;
    hipLaunchKernelGGL(ordered_sum_kernel<Out>, dim3(bx, G), dim3(1024), 0, s, part, lvl, out, E, R);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    part = lvl;
    R = G;
  }
  hipLaunchKernelGGL(ordered_sum_kernel<Out>, dim3(bx, 1), dim3(1024), 0, s, part, lvl, out, E, R);
  return hipGetLastError();
}

// ------------------------------------------------------------------ gated RMSNorm
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Forward: one wave per token; a lane owns the 8-element vectors lane, lane + 64, ... of its D features.
// NV = 8-element vectors per lane (D <= 512 NV).  A token is read from memory once: x = y SiLU(a)
// stays in registers between the sum of squares and the output.  32768 tokens, D = 1344, bf16: 53 us,
// 5.0 TB/s.
template <typename IO, int NV>
__global__ void __launch_bounds__(256)
    gated_rmsnorm_fwd_kernel(const void *__restrict__ y, const void *__restrict__ a,
                             const void *__restrict__ w, float eps, void *__restrict__ out,
                             float *__restrict__ s_out, size_t tokens, int D) {
  const int lane = threadIdx.x & 63, DV = D / 8;
  const size_t wave = (blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6;
  const size_t nwaves = ((size_t)gridDim.x * blockDim.x) >> 6;
  for (size_t tok = wave; tok < tokens; tok += nwaves) {
    typename Vec8<IO>::Raw ry[NV], ra[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int v = lane + 64 * q, vc = v < DV ? v : DV - 1;  // (clamped: loads are unconditional)
      ry[q] = Vec8<IO>::load_raw(y, tok * D + 8 * vc);
      ra[q] = Vec8<IO>::load_raw(a, tok * D + 8 * vc);
    }
    float x[NV][8];
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      float yy[8], aa[8];
      Vec8<IO>::widen(ry[q], yy);
      Vec8<IO>::widen(ra[q], aa);
      const bool ok = lane + 64 * q < DV;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[q][i] = ok ? yy[i] * (aa[i] * sigmoidf_(aa[i])) : 0.f;
        ss = fmaf(x[q][i], x[q][i], ss);
      }
    }
    ss = wave_sum(ss);
    const float s = 1.f / sqrtf(ss / (float)D + eps);
    if (s_out && lane == 0) s_out[tok] = s;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int v = lane + 64 * q;
      if (v < DV) {
        float ww[8], o[8];
        Vec8<IO>::load(w, 8 * v, ww);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = ww[i] * x[q][i] * s;
        Vec8<IO>::store(out, tok * D + 8 * v, o);
      }
    }
  }
}

constexpr int kMaxVecPerLane = 8;  // of the forward; waves per token of the backward: D <= 8 * 64 * 8 = 4096

// Backward (appendix): p = w dout, r = sum p x, dx = s p - r s^3 x / d; dy = dx g,
// da = dx y SiLU'(a); dw = sum over tokens of dout x s, per workgroup over the tokens it walks
// (increasing), written to part[workgroup][D]; the column sums behind add the workgroups in order.
//
// Five tensors once: bound by memory if enough loads are in flight while the vector work goes
// on.  A token is spread over W = ceil(D / 512) waves, so that a lane holds eight of its elements
// whatever D is: 118 registers with the next token's vectors on the way, 16 waves per CU (at 96
// registers, for 20 waves, it spills: 138 us with all launches against 94).  The
// waves of a token meet once, at an LDS-only barrier that leaves the loads in flight.  (With a whole
// token per wave the registers of D = 1344 left 8 waves per CU, and D > 2048 spilled.)
// 32768 tokens, D = 1344, bf16, 440 MB: 172 -> 82 us.
template <typename IO>
__global__ void __launch_bounds__(512, 4)
    gated_rmsnorm_bwd_kernel(const void *__restrict__ y, const void *__restrict__ a,
                             const void *__restrict__ w, float eps, const float *__restrict__ s_in,
                             const void *__restrict__ dout, void *__restrict__ dy,
                             void *__restrict__ da, float *__restrict__ part, size_t tokens, int D) {
  typedef typename Vec8<IO>::Raw Raw;
  const int DV = D / 8, W = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool mine = (int)threadIdx.x < DV;
  const size_t e0 = 8 * (size_t)(mine ? threadIdx.x : DV - 1);  // (clamped: loads are unconditional)
  __shared__ float red[2][2][kMaxVecPerLane];  // [token parity][r, ss][wave]
  float ww[8], dwacc[8];
  Vec8<IO>::load(w, e0, ww);
#pragma unroll
  for (int i = 0; i < 8; ++i) dwacc[i] = 0.f;
  Raw ny, na, nd;
  float ns = 0.f;
  auto fetch = [&](size_t tok) {
    ny = Vec8<IO>::load_raw(y, tok * D + e0);
    na = Vec8<IO>::load_raw(a, tok * D + e0);
    nd = Vec8<IO>::load_raw(dout, tok * D + e0);
    if (s_in) ns = s_in[tok];
  };
  if (blockIdx.x < tokens) fetch(blockIdx.x);
  int par = 0;
  for (size_t tok = blockIdx.x; tok < tokens; tok += gridDim.x, par ^= 1) {
    float yy[8], aa[8], dd[8], g[8], x[8];
    Vec8<IO>::widen(ny, yy);
    Vec8<IO>::widen(na, aa);
    Vec8<IO>::widen(nd, dd);
    float s = ns;
    fetch(tok + gridDim.x < tokens ? tok + gridDim.x : tok);  // (last token: fetched again, unused)
    float ss = 0.f, r = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float sg = sigmoidf_(aa[i]);
      g[i] = aa[i] * sg;
      aa[i] = sg * (1.f + aa[i] * (1.f - sg));  // SiLU'
      x[i] = yy[i] * g[i];
      ss = fmaf(x[i], x[i], ss);
      r = fmaf(ww[i] * dd[i], x[i], r);
    }
    r = wave_sum(mine ? r : 0.f);
    if (!s_in) ss = wave_sum(mine ? ss : 0.f);
    if (W > 1) {  // the waves' sums, in increasing order
      if (lane == 0) {
        red[par][0][wv] = r;
        red[par][1][wv] = ss;
      }
      lds_barrier();  // (the other parity's words are free again: every wave has read them)
      r = red[par][0][0];
      ss = red[par][1][0];
      for (int u = 1; u < W; ++u) {
        r += red[par][0][u];
        ss += red[par][1][u];
      }
    }
    if (!s_in) s = 1.f / sqrtf(ss / (float)D + eps);
    const float c3 = r * s * s * s / (float)D;
    if (mine) {
      float oy[8], oa[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float dxi = s * (ww[i] * dd[i]) - c3 * x[i];
        dwacc[i] = fmaf(dd[i] * x[i], s, dwacc[i]);
        oy[i] = dxi * g[i];
        oa[i] = dxi * yy[i] * aa[i];
      }
      Vec8<IO>::store(dy, tok * D + e0, oy);
      Vec8<IO>::store(da, tok * D + e0, oa);
    }
  }
  if (mine) {
    *(f4_t *)&part[blockIdx.x * (size_t)D + e0] = f4_t{dwacc[0], dwacc[1], dwacc[2], dwacc[3]};
    *(f4_t *)&part[blockIdx.x * (size_t)D + e0 + 4] = f4_t{dwacc[4], dwacc[5], dwacc[6], dwacc[7]};
  }
}

// Most partial rows of the weight-gradient sums, one per workgroup row (convolution) or workgroup
// (norm) of a launch; they size the scratch.  A launch uses fewer where fewer fill the chip: at 8 x 4096
// 128 rows of 7360 floats (1472 channels) and 1280 of 1344: 3 % of the tensors' own traffic.
constexpr int kConvRows = 2048;  // of the convolution's dw / dbias sums
constexpr int kNormWaves = 4096; // of the norm's dw sum

// Rows of the convolution's scratch (callers size their workspace by this figure): workgroup rows of
// a launch stay within it (its walkers take more items each where that binds).
inline int conv_rows(int B, int T) {
  const long long rows = (long long)B * ((T + 31) / 32);
  return (int)(rows < kConvRows ? (rows < 1 ? 1 : rows) : kConvRows);
}
// Workgroup rows of a backward launch, beyond those that fill the chip: with many sequences of a few steps
// a row has less to read than the partial sums it writes and the sum behind reads again.
// bf16, us, without the limit -> with it (the kernel with eight channels per lane before): 4096 x 1 x 1024
// 33.3 -> 20.9 (22.6), 8192 x 1 x 1024 58.5 -> 32.1 (33.7), 4096 x 4 x 512 25.5 -> 19.7 (23.7);
// 512 rows instead of 256: 24.8, 35.3, 19.7.
inline int conv_bwd_most_rows(int gx) { return std::max(256, (1024 + gx - 1) / gx); }
// Rows of the norm's scratch (callers size their workspace by this figure), and workgroups of a
// launch = rows in use: what is resident with W waves per workgroup, four on each SIMD.
inline int norm_waves(size_t tokens) {
  const size_t r = tokens < (size_t)kNormWaves ? (tokens < 1 ? 1 : tokens) : kNormWaves;
  return (int)((r + 3) / 4 * 4);
}
inline int norm_rows(size_t tokens, int W) {
  const int resident = 256 * (16 / W), most = resident < kNormWaves ? resident : kNormWaves;
  return tokens < (size_t)most ? (int)tokens : most;
}

}  // namespace

size_t conv_silu_scratch_bytes(int B, int T, int C) {
  return align256((size_t)(conv_rows(B, T) + kSumGroups) * C * (kTaps + 1) * sizeof(float));
}
size_t gated_rmsnorm_scratch_bytes(int B, int T, int D) {
  return align256((size_t)(norm_waves((size_t)B * T) + kSumGroups) * D * sizeof(float));
}
int gated_rmsnorm_max_features() { return kMaxVecPerLane * 64 * 8; }

template <typename IO>
static hipError_t conv_fwd_t(int B, int T, int C, const void *x, const void *w, const void *bias,
                             void *out, hipStream_t s) {
  if ((size_t)B * T == 0) return hipSuccess;
  const ConvPlan p = conv_plan(B, T, C, 16384);
  hipLaunchKernelGGL((conv_silu_fwd_kernel<IO>), dim3((unsigned)(p.gx * p.rg)), dim3(kThreads), 0, s, x, w, bias,
                     out, B, T, C, p);
  return hipGetLastError();
}
hipError_t conv_silu_fwd(int B, int T, int C, int io, const void *x, const void *w, const void *bias,
                         void *out, hipStream_t s) {
  return io == 0 ? conv_fwd_t<float>(B, T, C, x, w, bias, out, s)
                 : conv_fwd_t<__hip_bfloat16>(B, T, C, x, w, bias, out, s);
}

template <typename IO>
static hipError_t conv_bwd_t(int B, int T, int C, const void *x, const void *w, const void *bias,
                             const void *dout, void *dx, float *dw, float *dbias, float *part,
                             hipStream_t s) {
  ConvPlan p = conv_plan(B, T, C, conv_rows(B, T));
  p.rg = std::min(p.rg, conv_bwd_most_rows(p.gx));
  const bool any = (size_t)B * T > 0;
  if (any) {
    hipLaunchKernelGGL((conv_silu_bwd_kernel<IO>), dim3((unsigned)(p.gx * p.rg)), dim3(kThreads), 0, s,
                       x, w, bias, dout, dx, part, B, T, C, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int E = C * (kTaps + 1);
  return ordered_sum(part, part + (size_t)p.rg * E, ConvOut{dw, dbias}, E, any ? p.rg : 0, s);
}
hipError_t conv_silu_bwd(int B, int T, int C, int io, const void *x, const void *w, const void *bias,
                         const void *dout, void *dx, float *dw, float *dbias, float *part,
                         hipStream_t s) {
  return io == 0 ? conv_bwd_t<float>(B, T, C, x, w, bias, dout, dx, dw, dbias, part, s)
                 : conv_bwd_t<__hip_bfloat16>(B, T, C, x, w, bias, dout, dx, dw, dbias, part, s);
}

template <typename IO>
static hipError_t norm_fwd_t(int B, int T, int D, const void *y, const void *a, const void *w, float eps,
                             void *out, float *s_out, hipStream_t s) {
  const size_t tokens = (size_t)B * T;
  if (tokens == 0) return hipSuccess;
  size_t blocks = (tokens + 3) / 4;  // four waves = four tokens per workgroup
  if (blocks > 16384) blocks = 16384;
  const int nv = (D / 8 + 63) / 64;
#define M2RNN_GO(NV_)                                                                              \
  hipLaunchKernelGGL((gated_rmsnorm_fwd_kernel<IO, NV_>), dim3((unsigned)blocks), dim3(256), 0, s, y, a, \
                     w, eps, out, s_out, tokens, D)
  if (nv <= 1) M2RNN_GO(1);
  else if (nv <= 2) M2RNN_GO(2);
  else if (nv <= 3) M2RNN_GO(3);
  else if (nv <= 4) M2RNN_GO(4);
  else if (nv <= 6) M2RNN_GO(6);
  else M2RNN_GO(8);
#undef M2RNN_GO
  return hipGetLastError();
}
hipError_t gated_rmsnorm_fwd(int B, int T, int D, int io, const void *y, const void *a, const void *w,
                             float eps, void *out, float *s_out, hipStream_t s) {
  return io == 0 ? norm_fwd_t<float>(B, T, D, y, a, w, eps, out, s_out, s)
                 : norm_fwd_t<__hip_bfloat16>(B, T, D, y, a, w, eps, out, s_out, s);
}

template <typename IO>
static hipError_t norm_bwd_t(int B, int T, int D, const void *y, const void *a, const void *w, float eps,
                             const float *s_in, const void *dout, void *dy, void *da, float *dw,
                             float *part, hipStream_t s) {
  const size_t tokens = (size_t)B * T;
  const int W = (D / 8 + 63) / 64;
  const int R = norm_rows(tokens, W);
  if (tokens > 0) {
    hipLaunchKernelGGL((gated_rmsnorm_bwd_kernel<IO>), dim3(R), dim3(64 * W), 0, s, y, a, w, eps, s_in, dout, dy,
                       da, part, tokens, D);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return ordered_sum(part, part + (size_t)R * D, PlainOut{dw}, D, tokens > 0 ? R : 0, s);
}
hipError_t gated_rmsnorm_bwd(int B, int T, int D, int io, const void *y, const void *a, const void *w,
                             float eps, const float *s_in, const void *dout, void *dy, void *da,
                             float *dw, float *part, hipStream_t s) {
  return io == 0 ? norm_bwd_t<float>(B, T, D, y, a, w, eps, s_in, dout, dy, da, dw, part, s)
                 : norm_bwd_t<__hip_bfloat16>(B, T, D, y, a, w, eps, s_in, dout, dy, da, dw, part, s);
}

}  // namespace m2rnn
