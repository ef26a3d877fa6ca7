// Device-side building blocks shared by the gfx950 kernels: vector types, bf16 conversion,
// wave64 reductions and the kernel-launch record used for timing.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.hpp"

namespace attt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// float -> bf16 bits, round to nearest even (inputs here are finite).
// v_cvt_pk_bf16_f32: round to nearest even, NaN stays NaN.
typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
typedef float f32x2_hw __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_hw){lo, hi}, bf16x2_hw));
}

// Raw buffer descriptor over [p, p + bytes): loads at offsets at or past `bytes` return zero.
// Both arguments must be wave-uniform; they are moved to scalar registers explicitly, since a
// uniform value computed on the vector unit would otherwise turn every access through the
// descriptor into a loop over lanes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* p, int bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  void* q = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(q, (short)0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// Job of workgroup `bid` of a launch over several jobs: the last whose b_begin is at most bid. Each lane
// looks at one job (two above 64), so the search is one load and a ballot however many jobs a launch
// has (a scan is a chain of scalar loads, 18 us for 96 jobs). Wave-uniform, and made explicit, so that
// descriptors built from the job's pointers live in scalar registers.
template <class Batch>
__device__ __forceinline__ int find_job(const Batch& b, int bid) {
  const int lane = threadIdx.x & 63;
  int n = __popcll(__ballot(lane < b.count && b.j[lane < b.count ? lane : 0].b_begin <= bid));
  if constexpr (Batch::kCap > 64)
    n += __popcll(__ballot(lane + 64 < b.count && b.j[lane + 64 < b.count ? lane + 64 : 0].b_begin <= bid));
  return __builtin_amdgcn_readfirstlane(n - 1);
}

template <int W>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Merge two (max, sum of exp(x - max)) pairs; an empty pair is (-inf, 0).
__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {
  if (m2 == -INFINITY) return;
  if (m == -INFINITY) { m = m2; s = s2; return; }
  float mn = fmaxf(m, m2);
  s = s * expf(m - mn) + s2 * expf(m2 - mn);
  m = mn;
}

}  // namespace attt
