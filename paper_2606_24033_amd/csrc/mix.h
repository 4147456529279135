// Softmax weights times value radii, packed as fp16 operands (prefill.hip,
// decode_impl.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bgtq {

// fp16(p0 lo(w)) | fp16(p1 hi(w)) << 16, w = two fp16: one mixed-precision
// product into each half (v_fma_mixlo_f16, v_fma_mixhi_f16).  In C++ and not in
// inline asm: p0 and p1 come straight from v_exp_f32, and gfx950 wants a wait
// state between a transcendental instruction and a plain VALU one that reads
// its result.  The compiler keeps it only for instructions that it knows; with
// asm here every prefill attention kernel had a product right behind its
// exponential.
__device__ __forceinline__ uint32_t mix_pair(float p0, float p1, uint32_t w) {
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  const half2_t h = __builtin_bit_cast(half2_t, w);
  const half2_t r = {static_cast<_Float16>(__builtin_fmaf(p0, static_cast<float>(h[0]), 0.f)),
                     static_cast<_Float16>(__builtin_fmaf(p1, static_cast<float>(h[1]), 0.f))};
  return __builtin_bit_cast(uint32_t, r);
}

}  // namespace bgtq
