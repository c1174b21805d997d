// Device helpers of the bf16 attention kernels.
#pragma once

#include "device_util.h"

namespace rs3 {

// One direct-to-LDS load: 16 bytes per lane from g into the wave's 1 KB at
// lds_wave (lane l lands at lds_wave + 16 l).
__device__ __forceinline__ void dma16(const void* g, void* lds_wave) {
  __builtin_amdgcn_global_load_lds(g, lds_wave, 16, 0, 0);
}

// Value of lane l^32 for every lane (v_permlane32_swap: both halves come back
// in registers; op(r[0], r[1]) combines a lane with its partner).
__device__ __forceinline__ float max_with_partner(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_partner(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Workgroup barrier without a memory fence: the fence of __syncthreads()
// would wait for every outstanding load, including the K/V prefetches.
// LDS stages are published by the explicit vmcnt waits before it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_barrier" ::: "memory"); }

// s_waitcnt encoding: wait until at most n vector-memory ops are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Waits until at most `later` stages of PW loads each are still in flight
// (`later` is wave-uniform and at most MAXL).
template <int PW, int MAXL>
__device__ __forceinline__ void wait_stages(int later) {
  if constexpr (MAXL >= 6) if (later >= 6) { wait_vmcnt<6 * PW>(); return; }
  if constexpr (MAXL >= 5) if (later == 5) { wait_vmcnt<5 * PW>(); return; }
  if constexpr (MAXL >= 4) if (later == 4) { wait_vmcnt<4 * PW>(); return; }
  if constexpr (MAXL >= 3) if (later == 3) { wait_vmcnt<3 * PW>(); return; }
  if constexpr (MAXL >= 2) if (later == 2) { wait_vmcnt<2 * PW>(); return; }
  if (later == 1) {
    wait_vmcnt<PW>();
    return;
  }
  wait_vmcnt<0>();
}

// Maximum that propagates NaN (the logits hold none): v_maximum3_f32 needs
// no canonicalising of its inputs, unlike fmaxf.
__device__ __forceinline__ float max3f(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// Sum of the two bf16 values of a packed pair added to acc (v_dot2 with 1,1):
// the row sums then add exactly the rounded probabilities the PV product uses.
__device__ __forceinline__ float add_bf16x2(uint32_t p, float acc) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t one = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, p), one, acc, false);
}

}  // namespace rs3
