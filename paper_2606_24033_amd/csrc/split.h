// 128 x 128 fp32 matrix times bf16 rows on bf16 MFMAs, exact but for the fp32
// accumulation.
//
// An fp32 matrix entry is the exact sum of three bf16 numbers (8 + 8 + 8 bits
// of its significand, taken by truncation) and a bf16 input is an operand as
// it lies in memory, so the product runs as three v_mfma_f32_16x16x32_bf16
// products whose terms are exact in fp32, at 3/16 of the time of the fp32
// MFMAs.
#pragma once
#include <hip/hip_runtime.h>

#include "layout.h"

namespace bgtq {
namespace split {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));
constexpr int kSub = 16;                    // rows per wave sub-tile (one MFMA column block)
constexpr int kSplitRows = 2 * kSub;        // rows of a wave
constexpr int kMatF4 = kMfmaMatFloats / 4;  // float4 entries of one MFMA-order matrix
constexpr int kMatOps = kMatF4 / 2;         // its 8-element operands: [t][q][lane]

__device__ __forceinline__ float4_t mfma_bf16(uint4_t a, uint4_t b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

// The fp32 matrix from memory into its three bf16 parts in LDS: operand o =
// (t * 4 + q) * 64 + lane holds the lane's input dims 32 (lane / 16) + 8 q ..
// + 7, two float4 of the fp32 order.
template <int W>
__device__ __forceinline__ void stage_split(uint4_t (*dst)[kMatOps], const float4* __restrict__ src, int tid) {
  constexpr int kPer = kMatOps / (W * 64), kRound = kPer < 4 ? kPer : 4;
  static_assert(kMatOps % (W * 64) == 0 && kPer % kRound == 0, "matrix staging");
#pragma unroll 1
  for (int u0 = 0; u0 < kPer; u0 += kRound) {
    float4 lo[kRound], hi[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const int o = tid + (u0 + u) * W * 64, f = ((o >> 6) * 2) * 64 + (o & 63);
      lo[u] = src[f];
      hi[u] = src[f + 64];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const float w[8] = {lo[u].x, lo[u].y, lo[u].z, lo[u].w, hi[u].x, hi[u].y, hi[u].z, hi[u].w};
      uint32_t part[3][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        part[0][e] = __float_as_uint(w[e]) & 0xFFFF0000u;
        const float r1 = w[e] - __uint_as_float(part[0][e]);
        part[1][e] = __float_as_uint(r1) & 0xFFFF0000u;
        part[2][e] = __float_as_uint(r1 - __uint_as_float(part[1][e]));
      }
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        uint4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (part[p][2 * e] >> 16) | (part[p][2 * e + 1] & 0xFFFF0000u);
        dst[p][tid + (u0 + u) * W * 64] = v;
      }
    }
  }
}

// The lane's 32 dims of one bf16 row as four operands.
__device__ __forceinline__ void load_operands(const void* src, size_t elem_off, bool valid, uint4_t (&x)[4]) {
  const uint4_t* p = reinterpret_cast<const uint4_t*>(static_cast<const uint16_t*>(src) + elem_off);
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = valid ? p[q] : uint4_t{0u, 0u, 0u, 0u};
}

// Output tile t of the products of the wave's two sub-tiles (the matrix is the
// A operand).  The two small parts have their own accumulator.
__device__ __forceinline__ void split_product(const uint4_t (*mat)[kMatOps], int t, int lane, const uint4_t (&x)[2][4],
                                              float4_t (&out)[2]) {
  float4_t hi[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, lo[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int o = (t * 4 + q) * 64 + lane;
    const uint4_t w0 = mat[0][o], w1 = mat[1][o], w2 = mat[2][o];
#pragma unroll
    for (int s = 0; s < 2; ++s) lo[s] = mfma_bf16(w2, x[s][q], lo[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) hi[s] = mfma_bf16(w0, x[s][q], hi[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) lo[s] = mfma_bf16(w1, x[s][q], lo[s]);
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) out[s] = hi[s] + lo[s];
}

}  // namespace split
}  // namespace bgtq
