// Elements of io tensors (float or bfloat16) as floats, one, four and eight at a time, and the column
// sum that ends the fixed-order sums over rows.
#pragma once
#include <hip/hip_bf16.h>

#include "m2rnn_mfma_common.hpp"

namespace m2rnn {

template <typename IO> __device__ __forceinline__ float to_f32(IO x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<__hip_bfloat16>(__hip_bfloat16 x) {
  return __bfloat162float(x);
}
template <typename IO> __device__ __forceinline__ IO from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ __hip_bfloat16 from_f32<__hip_bfloat16>(float x) {
  return __float2bfloat16(x);  // round to nearest even
}
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t lo16) {
  return __builtin_bit_cast(float, lo16 << 16);
}
// two floats, rounded to nearest even, in one dword (one conversion instruction; done on integers
// the six of each element were a third of the norm's vector work)
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  typedef float f2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
  const f2_t x = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, b2_t));
}

// eight consecutive elements of an io tensor <-> eight floats
template <typename IO> struct Vec8;
template <> struct Vec8<float> {
  struct Raw { f4_t a, b; };
  static __device__ __forceinline__ Raw load_raw(const void *base, size_t e) {
    return Raw{*(const f4_t *)((const float *)base + e), *(const f4_t *)((const float *)base + e + 4)};
  }
  static __device__ __forceinline__ void widen(const Raw &r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[i] = r.a[i]; x[4 + i] = r.b[i]; }
  }
  static __device__ __forceinline__ void load(const void *base, size_t e, float (&x)[8]) {
    widen(load_raw(base, e), x);
  }
  static __device__ __forceinline__ void store(void *base, size_t e, const float (&x)[8]) {
    *(f4_t *)((float *)base + e) = f4_t{x[0], x[1], x[2], x[3]};
    *(f4_t *)((float *)base + e + 4) = f4_t{x[4], x[5], x[6], x[7]};
  }
};
template <> struct Vec8<__hip_bfloat16> {
  typedef u4_t Raw;
  static __device__ __forceinline__ Raw load_raw(const void *base, size_t e) {
    return *(const u4_t *)((const unsigned short *)base + e);
  }
  static __device__ __forceinline__ void widen(const Raw &w, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = bf16_bits_to_f32(w[i] & 0xFFFFu);
      x[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ void load(const void *base, size_t e, float (&x)[8]) {
    widen(load_raw(base, e), x);
  }
  static __device__ __forceinline__ void store(void *base, size_t e, const float (&x)[8]) {
    u4_t w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack2_bf16(x[2 * i], x[2 * i + 1]);
    *(u4_t *)((unsigned short *)base + e) = w;
  }
};
// four consecutive elements of an io tensor <-> four floats
template <typename IO> struct Vec4;
template <> struct Vec4<float> {
  typedef f4_t Raw;
  static __device__ __forceinline__ Raw load_raw(const void *base, size_t e) {
    return *(const f4_t *)((const float *)base + e);
  }
  static __device__ __forceinline__ void widen(const Raw &w, float (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = w[i];
  }
  static __device__ __forceinline__ void store(void *base, size_t e, const float (&x)[4]) {
    *(f4_t *)((float *)base + e) = f4_t{x[0], x[1], x[2], x[3]};
  }
};
template <> struct Vec4<__hip_bfloat16> {
  typedef uint32_t Raw __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ Raw load_raw(const void *base, size_t e) {
    return *(const Raw *)((const unsigned short *)base + e);
  }
  static __device__ __forceinline__ void widen(const Raw &w, float (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      x[2 * i] = bf16_bits_to_f32(w[i] & 0xFFFFu);
      x[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ void store(void *base, size_t e, const float (&x)[4]) {
    *(Raw *)((unsigned short *)base + e) = Raw{pack2_bf16(x[0], x[1]), pack2_bf16(x[2], x[3])};
  }
};

// Sum over the rows r0 <= r < r1 of column e of part [.][E], by a workgroup of 1024 threads for 32
// columns: walker w = thread / 32 takes the rows r0 + w, r0 + w + 32, ... with four loads in flight, and
// the walkers are added in increasing order.  The result is that of the first 32 threads.
__device__ __forceinline__ float column_sum(const float *__restrict__ part, int E, int e, int r0, int r1) {
  __shared__ float red[32][33];
  const int cl = threadIdx.x & 31, wl = threadIdx.x >> 5;
  float s = 0.f;
  if (e < E) {
    int r = r0 + wl;
    for (; r + 96 < r1; r += 128) {
      float x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = part[(size_t)(r + 32 * u) * E + e];
      s += (x[0] + x[1]) + (x[2] + x[3]);
    }
    for (; r < r1; r += 32) s += part[(size_t)r * E + e];
  }
  red[wl][cl] = s;
  __syncthreads();
  float t = 0.f;
  if (wl == 0) {
#pragma unroll
    for (int w = 0; w < 32; ++w) t += red[w][cl];
  }
  return t;
}

}  // namespace m2rnn
