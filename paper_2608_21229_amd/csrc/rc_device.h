// Device helpers shared by the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rc {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// Largest magnitude of 8 bf16 values (one 16-byte granule).
__device__ __forceinline__ float amax8(u32x4 g) {
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m = fmaxf(m, fabsf(bf16_bits_to_float(g[i] & 0xffffu)));
    m = fmaxf(m, fabsf(bf16_bits_to_float(g[i] >> 16)));
  }
  return m;
}

}  // namespace rc
