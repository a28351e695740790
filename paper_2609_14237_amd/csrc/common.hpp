// Device helpers shared by the gfx950 kernels: bf16 <-> fp32, MFMA wrappers,
// wave reductions. CDNA4 only: wave64, bf16 MFMA (16x16x32 and 16x16x16).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace ods {

// Raise a kernel's dynamic-LDS limit on the current device, once per device
// (`done` holds one bit per device id below 64; higher ids set it every call).
inline hipError_t ensure_lds_limit(const void *kern, size_t bytes, std::atomic<uint64_t> &done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kPage = 16;

// bf16 bits -> fp32 (exact).
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// fp32 -> bf16 bits, round to nearest even (hardware conversion on gfx950).
__device__ __forceinline__ uint16_t f2bf(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
}

__device__ __forceinline__ f32x4 mfma_16x16x32(const bf16x8 &a, const bf16x8 &b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_16x16x16(const bf16x4 &a, const bf16x4 &b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}

// Sum over a 256-thread block; `red` is >= 4 floats of shared memory.
__device__ __forceinline__ float block_sum_256(float v, float *red) {
  v = wave_sum(v);
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) red[w] = v;
  __syncthreads();
  float t = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return t;
}

// cos and sin of the RoPE angle of dimension pair i (of D / 2) at position p:
// p * theta^(-2 i / D), reduced mod 2 pi in double before the fp32 functions.
__device__ __forceinline__ void rope_angle(int p, int i, int D, float theta, float &cv, float &sv) {
  const double two_pi_hi = 6.283185307179586, two_pi_lo = 2.4492935982947064e-16;
  const double inv = exp2(-(2.0 * i / D) * log2((double)theta));
  const double a = (double)p * inv;
  const double k = rint(a * (1.0 / two_pi_hi));
  const double r = fma(-k, two_pi_lo, fma(-k, two_pi_hi, a));
  sincosf((float)r, &sv, &cv);
}

// 8 bf16 values: their sum of squares, and their product with inv and a gain.
__device__ __forceinline__ float sumsq8(const u32x4 &w) {
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = bf_lo(w[j]), b = bf_hi(w[j]);
    t += a * a + b * b;
  }
  return t;
}
__device__ __forceinline__ u32x4 norm8(const u32x4 &w, const u32x4 &gw, float inv) {
  u32x4 o;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    o[j] = pack2(bf_lo(w[j]) * inv * bf_lo(gw[j]), bf_hi(w[j]) * inv * bf_hi(gw[j]));
  return o;
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + __expf(-z)); }

}  // namespace ods
