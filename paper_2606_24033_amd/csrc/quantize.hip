// Prefill quantize + pack + append on fp32 MFMAs: the TQ-MSE encode of
// Sec. 2.2 applied to every same-rate group of a key row (end of Sec. 3.2)
// and to the value row, for the long appends of a prefill (Sec. 4, prefill
// paragraph).  Appends of a few rows (decode steps) use k_append_rows; bf16
// rows of the ordinary widths take the bf16 products further down.
//
// Both encodes are dense 128 x 128 products per row on
// v_mfma_f32_16x16x4f32 (16 rows of a wave at a time), with the reduction
// index arranged so that a lane's 32 k-steps read 32 contiguous input dims
// (k-step s of lane l pairs with dim 32 (l / 16) + s): a lane loads its slice
// of a row with 16-byte loads and no gather.
//
// One launch (k_quant_rows) for both: its first workgroups encode keys, the
// others values.
//  keys   : Z = W X^T.  W (the layout's dense key rotation on the natural
//           dims, the gather into stream order folded in) is the A operand,
//           staged in LDS once per workgroup; the key rows are the B
//           operand.  A lane ends with four consecutive stream positions of
//           one row, i.e. one contiguous bit field of the packed row.  The
//           group radii come from the same kind of product, a 0/1 group
//           membership matrix times the squared inputs.
//  values : Z = X Pi_V^T.  The value rows are the A operand, Pi_V the B
//           operand.  A lane ends with one coordinate of four consecutive
//           rows, i.e. one contiguous bit field of a 32-row value tile.
// Codes: number of thresholds <= z (binary search over the fp32 midpoints of
// the fp16 centroids, LDS); rows and tiles are assembled in LDS with atomic
// ORs and written with whole-word stores.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "layout.h"

namespace bgtq {
namespace quant_detail {

typedef float float4_t __attribute__((ext_vector_type(4)));

// Workgroups of W waves: 16 for long appends (the 64 KB matrix staged in LDS
// serves more rows), 4 for calls of up to 64K rows, which then spread over
// more CUs: two such workgroups fit a CU (under 80 KB of LDS each), and a
// value tile is split between two waves.  (A 16-wave value workgroup of 16
// tiles keeps each SIMD's MFMA pipe busy ~30 us on its own, with most CUs
// idle in a short call.)
constexpr int kWavesLong = 16, kWavesShort = 4;
constexpr int kSub = 16;                          // rows per wave sub-tile (one MFMA column block)
constexpr int kMatF4 = kMfmaMatFloats / 4;        // float4 entries of one MFMA-order matrix

template <int W>
struct LdsK {
  float4 wa[kMatF4];                          // the row's W, A operand order
  float4 ma[W == kWavesLong ? 8 * 64 : 1];    // group membership, A operand order ([s4][lane]);
                                              // the short path keeps it in registers
  uint32_t rw[W][kSub][kMaxKWords];           // per wave: packed key rows
  float sc[W][kSub][kMaxGroups];              // per wave: sqrt(d_g) / radius of each row and group
  float thr[kThresholdEntries];
  uint32_t pm[kHeadDim];                      // per stream position: bit offset | b << 10 | group << 14
  float gs[kMaxGroups];                       // sqrt(d_g)
  uint8_t gd[kHeadDim];                       // group ordinal of each input dim
};
template <int W>
struct LdsV {
  float4 rb[kMatF4];                          // Pi_V, B operand order
  uint32_t vt[W][kHeadDim][8];                // per wave: words of one value tile
  float nv[W][32];                            // per wave: the tile's value radii
  float thr[kThresholdEntries];
};
// Short calls: a value tile is shared by two waves (16 rows each), two tiles
// per 4-wave workgroup.
struct LdsVS {
  float4 rb[kMatF4];                          // Pi_V, B operand order
  uint32_t vt[kWavesShort / 2][kHeadDim][8];  // per tile: its words
  float nv[kWavesShort / 2][32];              // per tile: its value radii
  float thr[kThresholdEntries];
};
static_assert(sizeof(LdsK<kWavesLong>) <= 160 * 1024 && sizeof(LdsV<kWavesLong>) <= 160 * 1024, "LDS of one workgroup");
// two short-call workgroups share a CU
static_assert(sizeof(LdsK<kWavesShort>) <= 80 * 1024 && sizeof(LdsVS) <= 80 * 1024, "LDS of a short-call workgroup");

// Copy of the 64 KB MFMA-order matrix into LDS with every global load issued
// before the first store (a loop of load-store pairs waits out one memory
// latency per round: 16 rounds in a 4-wave workgroup).
template <int W>
__device__ __forceinline__ void stage_matrix(float4* dst, const float4* __restrict__ src, int tid) {
  constexpr int kPer = kMatF4 / (W * 64);
  static_assert(kMatF4 % (W * 64) == 0, "matrix staging");
  float4 t[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) t[u] = src[tid + u * W * 64];
#pragma unroll
  for (int u = 0; u < kPer; ++u) dst[tid + u * W * 64] = t[u];
}

__device__ __forceinline__ void wave_sync() {
  // LDS operations of one wave complete in order; only the compiler must
  // keep them in program order
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Number of thresholds t <= z among the 2^b - 1 sorted thresholds at thr.
__device__ __forceinline__ uint32_t scalar_code(const float* thr, int b, float z) {
  int idx = 0;
  for (int step = 1 << (b - 1); step > 0; step >>= 1)
    if (thr[idx + step - 1] <= z) idx += step;
  return static_cast<uint32_t>(idx);
}

// Dims [32 kk, 32 kk + 32) of one input row (zeros when !valid); the row
// starts 16-byte aligned (the host checks the base pointer).
template <bool BF16>
__device__ __forceinline__ void load_slice(const void* src, size_t elem_off, bool valid, float (&x)[32]) {
  if (!valid) {
#pragma unroll
    for (int i = 0; i < 32; ++i) x[i] = 0.f;
    return;
  }
  if constexpr (BF16) {
    const uint4* p = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(src) + elem_off);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 v = p[q];
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[8 * q + 2 * e] = __uint_as_float(w[e] << 16);
        x[8 * q + 2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
      }
    }
  } else {
    const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(src) + elem_off);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 v = p[q];
      x[4 * q] = v.x;
      x[4 * q + 1] = v.y;
      x[4 * q + 2] = v.z;
      x[4 * q + 3] = v.w;
    }
  }
}

__device__ __forceinline__ float4_t mfma(float a, float b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- keys
// Workgroup bx of the key part: rows [bx R, bx R + R) of the call, R =
// W kSub iters.
template <bool BF16, int W>
__device__ __forceinline__ void quant_keys(LdsK<W>& S, int bx, int iters, const Dims& d,
                                           const uint8_t* __restrict__ blob, const void* __restrict__ kin, int n_new,
                                           const int32_t* __restrict__ wpos, const CachePtrs& c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y, lz = blockIdx.z;
  const int layer = d.layer >= 0 ? d.layer : lz / d.batch;
  const int seq = lz % d.batch;
  const int cap = d.capacity;
  const int wp = wpos[seq];
  if (wp < 0 || wp >= cap) return;
  const int n_fit = min(n_new, cap - wp);  // rows that fit (the host rejects overflow)
  constexpr int kThreads = W * 64;
  const int r_wg = bx * W * kSub * iters;
  if (r_wg >= n_fit) return;
  const int n_rows_blob = d.n_layers * d.n_kv;
  const int ri = layer * d.n_kv + head;
  const RowMeta* M = reinterpret_cast<const RowMeta*>(blob + kOffRows) + ri;
  const float4* wsrc = reinterpret_cast<const float4*>(blob + layout_kdense_offset(n_rows_blob)) +
                       static_cast<size_t>(ri) * kMatF4;
  const float* gthr = reinterpret_cast<const float*>(blob + kOffThr);
  const int ng = M->n_groups;

  stage_matrix<W>(S.wa, wsrc, tid);
  for (int i = tid; i < W * kSub * kMaxKWords; i += kThreads) (&S.rw[0][0][0])[i] = 0u;
  for (int i = tid; i < kThresholdEntries; i += kThreads) S.thr[i] = gthr[i];
  if (tid < kHeadDim) {
    const int g = M->grp[tid];
    S.gd[M->dim[tid]] = static_cast<uint8_t>(g);
    S.pm[tid] = static_cast<uint32_t>(M->bitoff[tid]) | (static_cast<uint32_t>(M->width[tid]) << 10) |
                (static_cast<uint32_t>(g) << 14);
  }
  if (tid < kMaxGroups) S.gs[tid] = tid < ng ? sqrtf(static_cast<float>(M->g_dim[tid])) : 0.f;
  __syncthreads();
  float mreg[32];  // short path: this lane's membership entries (unused in the long path)
  if constexpr (W == kWavesLong) {
    for (int i = tid; i < 8 * 64; i += kThreads) {
      const int s4 = i >> 6, l = i & 63, g = l & 15, d0 = 32 * (l >> 4) + 4 * s4;
      S.ma[i] = make_float4(S.gd[d0] == g ? 1.f : 0.f, S.gd[d0 + 1] == g ? 1.f : 0.f, S.gd[d0 + 2] == g ? 1.f : 0.f,
                            S.gd[d0 + 3] == g ? 1.f : 0.f);
    }
    __syncthreads();
  } else {
    const int g = lane & 15, d0 = 32 * (lane >> 4);
#pragma unroll
    for (int j = 0; j < 32; ++j) mreg[j] = S.gd[d0 + j] == g ? 1.f : 0.f;
  }

  const int tk = lane & 15, kk = lane >> 4;
  const int kw = d.k_words, nslot = (ng + 1) & ~1;
  const size_t row = (static_cast<size_t>(layer) * d.batch + seq) * d.n_kv + head;
  for (int it = 0; it < iters; ++it) {
    const int r0 = r_wg + (it * W + wave) * kSub;
    if (r0 >= n_fit) break;  // wave-uniform
    const int r = r0 + tk;
    const bool valid = r < n_fit;
    float x[32];
    load_slice<BF16>(kin, ((static_cast<size_t>(lz) * n_new + r) * d.n_kv + head) * kHeadDim + 32 * kk, valid, x);

    // group radii: R2[g][row] = sum_d [group(d) = g] x[row][d]^2
    float4_t n2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
      float4 m;
      if constexpr (W == kWavesLong) m = S.ma[s4 * 64 + lane];
      else m = make_float4(mreg[4 * s4], mreg[4 * s4 + 1], mreg[4 * s4 + 2], mreg[4 * s4 + 3]);
      n2 = mfma(m.x, x[4 * s4] * x[4 * s4], n2);
      n2 = mfma(m.y, x[4 * s4 + 1] * x[4 * s4 + 1], n2);
      n2 = mfma(m.z, x[4 * s4 + 2] * x[4 * s4 + 2], n2);
      n2 = mfma(m.w, x[4 * s4 + 3] * x[4 * s4 + 3], n2);
    }
    // rotation: Z[p][row] = sum_d W[p][d] x[row][d], 8 tiles of 16 positions
    float4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float4 w = S.wa[(t * 8 + s4) * 64 + lane];
        acc[t] = mfma(w.x, x[4 * s4], acc[t]);
        acc[t] = mfma(w.y, x[4 * s4 + 1], acc[t]);
        acc[t] = mfma(w.z, x[4 * s4 + 2], acc[t]);
        acc[t] = mfma(w.w, x[4 * s4 + 3], acc[t]);
      }
    }
    // this lane holds R2 of row tk for groups 4 kk .. 4 kk + 3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = 4 * kk + i;
      if (g < ng) {
        const float nrm = sqrtf(n2[i]);
        S.sc[wave][tk][g] = nrm > 0.f ? S.gs[g] / nrm : 0.f;
        if (valid)
          c.k_norms[row * kMaxGroups * cap + static_cast<size_t>(wp + r) * nslot + g] =
              __half_as_ushort(__float2half_rn(nrm));
      }
    }
    wave_sync();
    // codes of stream positions 16 t + 4 kk + i of row tk: one bit field
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int p0 = 16 * t + 4 * kk;
      uint32_t field = 0;
      int nb = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t pm = S.pm[p0 + i];
        const int b = (pm >> 10) & 15, g = (pm >> 14) & 7;
        const uint32_t code = scalar_code(S.thr + thr_index(b), b, acc[t][i] * S.sc[wave][tk][g]);
        field |= code << nb;
        nb += b;
      }
      const int bo = S.pm[p0] & 1023, w = bo >> 5, sh = bo & 31;
      if (valid) {
        atomicOr(&S.rw[wave][tk][w], field << sh);
        if (sh + nb > 32) atomicOr(&S.rw[wave][tk][w + 1], field >> (32 - sh));
      }
    }
    wave_sync();
    for (int idx = lane; idx < kSub * kw; idx += 64) {
      const int t2 = idx / kw, w = idx - t2 * kw;
      if (r0 + t2 < n_fit) c.k_codes[(row * cap + wp + r0 + t2) * kw + w] = S.rw[wave][t2][w];
      S.rw[wave][t2][w] = 0u;
    }
    wave_sync();
  }
}

// ---------------------------------------------------------------- values
// Workgroup bx of the value part: value tiles [bx T, bx T + T) of the rows
// the call touches, T = W iters.  A wave owns whole 32-row value tiles;
// the words of a tile partly outside [write_pos, write_pos + n_new) keep the
// bits of the other rows.
template <bool BF16, int W>
__device__ __forceinline__ void quant_values(LdsV<W>& S, int bx, int iters, const Dims& d,
                                             const uint8_t* __restrict__ blob, const void* __restrict__ vin,
                                             int n_new, const int32_t* __restrict__ wpos, const CachePtrs& c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y, lz = blockIdx.z;
  const int layer = d.layer >= 0 ? d.layer : lz / d.batch;
  const int seq = lz % d.batch;
  const int cap = d.capacity, bv = d.v_bits;
  const int wp = wpos[seq];
  if (wp < 0 || wp >= cap) return;
  const int n_fit = min(n_new, cap - wp);
  const int tile0 = wp / kTile, n_tiles = (wp + n_fit - 1) / kTile - tile0 + 1;
  constexpr int kThreads = W * 64;
  const int tw0 = bx * W * iters;
  if (tw0 >= n_tiles) return;
  const int n_rows_blob = d.n_layers * d.n_kv;
  const float4* rsrc = reinterpret_cast<const float4*>(blob + layout_rotv_mfma_offset(n_rows_blob));
  const float* gthr = reinterpret_cast<const float*>(blob + kOffThr);
  stage_matrix<W>(S.rb, rsrc, tid);
  for (int i = tid; i < kThresholdEntries; i += kThreads) S.thr[i] = gthr[i];
  __syncthreads();

  const int tk = lane & 15, kk = lane >> 4;
  const float* thr = S.thr + thr_index(bv);
  const float sq = sqrtf(static_cast<float>(kHeadDim));
  const size_t row = (static_cast<size_t>(layer) * d.batch + seq) * d.n_kv + head;
  for (int it = 0; it < iters; ++it) {
    const int tw = tw0 + it * W + wave;
    if (tw >= n_tiles) break;  // wave-uniform
    const int tile = tile0 + tw, P0 = tile * kTile;
    const int s_lo = max(P0, wp) - P0, s_hi = min(P0 + kTile, wp + n_fit) - P0;  // rows [s_lo, s_hi) are new
    uint32_t* gv = c.v_codes + (row * (cap / kTile) + tile) * kHeadDim * static_cast<size_t>(bv);
    const bool full = s_lo == 0 && s_hi == kTile;
    // tile words: zero, or the old words with the new rows' bits cleared
    for (int idx = lane; idx < kHeadDim * bv; idx += 64) {
      const int j = idx / bv, w = idx - j * bv;
      uint32_t old = 0u;
      if (!full) {
        const int lo_b = max(s_lo * bv - 32 * w, 0), hi_b = min(s_hi * bv - 32 * w, 32);
        const uint32_t mask = hi_b <= lo_b ? 0u : (hi_b - lo_b == 32 ? ~0u : ((1u << (hi_b - lo_b)) - 1u) << lo_b);
        old = gv[idx] & ~mask;
      }
      S.vt[wave][j][w] = old;
    }
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      const int slot = 16 * h + tk;
      const bool valid = slot >= s_lo && slot < s_hi;
      float x[32];
      load_slice<BF16>(vin, ((static_cast<size_t>(lz) * n_new + (P0 + slot - wp)) * d.n_kv + head) * kHeadDim +
                                32 * kk,
                       valid, x);
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 32; ++i) ss = fmaf(x[i], x[i], ss);
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      const float nrm = sqrtf(ss);
      if (kk == 0) {
        S.nv[wave][slot] = nrm;
        if (valid) c.v_norms[row * cap + P0 + slot] = __half_as_ushort(__float2half_rn(nrm));
      }
      // Z[row][j] = sum_d x[row][d] Pi_V[j][d], 8 tiles of 16 coordinates
      float4_t acc[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s4 = 0; s4 < 8; ++s4) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float4 b = S.rb[(t * 8 + s4) * 64 + lane];
          acc[t] = mfma(x[4 * s4], b.x, acc[t]);
          acc[t] = mfma(x[4 * s4 + 1], b.y, acc[t]);
          acc[t] = mfma(x[4 * s4 + 2], b.z, acc[t]);
          acc[t] = mfma(x[4 * s4 + 3], b.w, acc[t]);
        }
      }
      wave_sync();
      // this lane: coordinate j = 16 t + tk of rows 16 h + 4 kk + i
      float scl[4];
      uint32_t keep = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s = 16 * h + 4 * kk + i;
        const float n = S.nv[wave][s];
        scl[i] = n > 0.f ? sq / n : 0.f;
        keep |= (s >= s_lo && s < s_hi ? ((1u << bv) - 1u) : 0u) << (i * bv);
      }
      const int bit = (16 * h + 4 * kk) * bv, w = bit >> 5, sh = bit & 31;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        uint32_t field = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) field |= scalar_code(thr, bv, acc[t][i] * scl[i]) << (i * bv);
        field &= keep;
        const int j = 16 * t + tk;
        atomicOr(&S.vt[wave][j][w], field << sh);
        if (sh + 4 * bv > 32) atomicOr(&S.vt[wave][j][w + 1], field >> (32 - sh));
      }
      wave_sync();
    }
    for (int idx = lane; idx < kHeadDim * bv; idx += 64) gv[idx] = S.vt[wave][idx / bv][idx % bv];
    wave_sync();
  }
}

// Short calls: workgroup bx encodes value tiles 2 bx and 2 bx + 1 of the
// rows the call touches; waves 2 u and 2 u + 1 take rows 0-15 and 16-31 of
// tile 2 bx + u and assemble its words together in LDS.
template <bool BF16>
__device__ __forceinline__ void quant_values_short(LdsVS& S, int bx, const Dims& d, const uint8_t* __restrict__ blob,
                                                   const void* __restrict__ vin, int n_new,
                                                   const int32_t* __restrict__ wpos, const CachePtrs& c) {
  constexpr int W = kWavesShort, kThreads = W * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y, lz = blockIdx.z;
  const int layer = d.layer >= 0 ? d.layer : lz / d.batch;
  const int seq = lz % d.batch;
  const int cap = d.capacity, bv = d.v_bits;
  const int wp = wpos[seq];
  if (wp < 0 || wp >= cap) return;  // (uniform over the workgroup: before any barrier)
  const int n_fit = min(n_new, cap - wp);
  const int tile0 = wp / kTile, n_tiles = (wp + n_fit - 1) / kTile - tile0 + 1;
  const int tw0 = bx * (W / 2);
  if (tw0 >= n_tiles) return;
  const int n_rows_blob = d.n_layers * d.n_kv;
  const float4* rsrc = reinterpret_cast<const float4*>(blob + layout_rotv_mfma_offset(n_rows_blob));
  const float* gthr = reinterpret_cast<const float*>(blob + kOffThr);
  stage_matrix<W>(S.rb, rsrc, tid);
  for (int i = tid; i < kThresholdEntries; i += kThreads) S.thr[i] = gthr[i];

  const int u = wave >> 1, h = wave & 1;  // the wave's tile of the workgroup and its half
  const int tile = tile0 + tw0 + u, P0 = tile * kTile;
  const bool active = tw0 + u < n_tiles;  // the same for both waves of a tile
  const int s_lo = max(P0, wp) - P0, s_hi = min(P0 + kTile, wp + n_fit) - P0;  // rows [s_lo, s_hi) are new
  const size_t row = (static_cast<size_t>(layer) * d.batch + seq) * d.n_kv + head;
  uint32_t* gv = c.v_codes + (row * (cap / kTile) + tile) * kHeadDim * static_cast<size_t>(bv);
  if (active) {
    // tile words: zero, or the old words with the new rows' bits cleared
    const bool full = s_lo == 0 && s_hi == kTile;
    for (int idx = 64 * h + lane; idx < kHeadDim * bv; idx += 128) {
      const int j = idx / bv, w = idx - j * bv;
      uint32_t old = 0u;
      if (!full) {
        const int lo_b = max(s_lo * bv - 32 * w, 0), hi_b = min(s_hi * bv - 32 * w, 32);
        const uint32_t mask = hi_b <= lo_b ? 0u : (hi_b - lo_b == 32 ? ~0u : ((1u << (hi_b - lo_b)) - 1u) << lo_b);
        old = gv[idx] & ~mask;
      }
      S.vt[u][j][w] = old;
    }
  }
  __syncthreads();  // matrix, thresholds and the tile words
  if (active) {
    const int tk = lane & 15, kk = lane >> 4;
    const float* thr = S.thr + thr_index(bv);
    const float sq = sqrtf(static_cast<float>(kHeadDim));
    const int slot = 16 * h + tk;
    const bool valid = slot >= s_lo && slot < s_hi;
    float x[32];
    load_slice<BF16>(vin, ((static_cast<size_t>(lz) * n_new + (P0 + slot - wp)) * d.n_kv + head) * kHeadDim + 32 * kk,
                     valid, x);
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 32; ++i) ss = fmaf(x[i], x[i], ss);
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    const float nrm = sqrtf(ss);
    if (kk == 0) {
      S.nv[u][slot] = nrm;
      if (valid) c.v_norms[row * cap + P0 + slot] = __half_as_ushort(__float2half_rn(nrm));
    }
    // Z[row][j] = sum_d x[row][d] Pi_V[j][d], 8 tiles of 16 coordinates
    float4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float4 b = S.rb[(t * 8 + s4) * 64 + lane];
        acc[t] = mfma(x[4 * s4], b.x, acc[t]);
        acc[t] = mfma(x[4 * s4 + 1], b.y, acc[t]);
        acc[t] = mfma(x[4 * s4 + 2], b.z, acc[t]);
        acc[t] = mfma(x[4 * s4 + 3], b.w, acc[t]);
      }
    }
    wave_sync();  // this half's radii (written by this wave)
    // this lane: coordinate j = 16 t + tk of rows 16 h + 4 kk + i
    float scl[4];
    uint32_t keep = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 16 * h + 4 * kk + i;
      const float n = S.nv[u][r];
      scl[i] = n > 0.f ? sq / n : 0.f;
      keep |= (r >= s_lo && r < s_hi ? ((1u << bv) - 1u) : 0u) << (i * bv);
    }
    const int bit = (16 * h + 4 * kk) * bv, w = bit >> 5, sh = bit & 31;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      uint32_t field = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) field |= scalar_code(thr, bv, acc[t][i] * scl[i]) << (i * bv);
      field &= keep;
      const int j = 16 * t + tk;
      atomicOr(&S.vt[u][j][w], field << sh);
      if (sh + 4 * bv > 32) atomicOr(&S.vt[u][j][w + 1], field >> (32 - sh));
    }
  }
  __syncthreads();  // both halves' bits are in the tile words
  if (active)
    for (int idx = 64 * h + lane; idx < kHeadDim * bv; idx += 128) gv[idx] = S.vt[u][idx / bv][idx % bv];
}

// One launch for both parts; grid (n_kwg + n_vwg, n_kv, batch x layers in
// the call).  16-wave workgroups: [0, n_kwg) encode keys, the rest values.
// 4-wave workgroups (short calls, two per CU): the value workgroups come
// first, so that the key workgroups fill in behind.
template <bool BF16, int W>
__global__ __launch_bounds__(W * 64) void k_quant_rows(Dims d, const uint8_t* __restrict__ blob,
                                                        const void* __restrict__ kin, const void* __restrict__ vin,
                                                        int n_new, const int32_t* __restrict__ wpos, CachePtrs c,
                                                        int n_kwg, int n_vwg, int k_iters, int v_iters) {
  constexpr size_t kVBytes = W == kWavesLong ? sizeof(LdsV<W>) : sizeof(LdsVS);
  constexpr size_t kBytes = sizeof(LdsK<W>) > kVBytes ? sizeof(LdsK<W>) : kVBytes;
  __shared__ __attribute__((aligned(16))) uint8_t smem[kBytes];
  const int bx = static_cast<int>(blockIdx.x);
  const bool keys = W == kWavesLong ? bx < n_kwg : bx >= n_vwg;
  if (keys)
    quant_keys<BF16, W>(*reinterpret_cast<LdsK<W>*>(smem), W == kWavesLong ? bx : bx - n_vwg, k_iters, d, blob, kin,
                        n_new, wpos, c);
  else if constexpr (W == kWavesLong)
    quant_values<BF16, W>(*reinterpret_cast<LdsV<W>*>(smem), bx - n_kwg, v_iters, d, blob, vin, n_new, wpos, c);
  else
    quant_values_short<BF16>(*reinterpret_cast<LdsVS*>(smem), bx, d, blob, vin, n_new, wpos, c);
}

// ---------------------------------------------------------------- bf16 inputs
// bf16 rows of the ordinary widths (key rows of up to kSplitKWords words,
// values of up to kSplitVBits bits).  An fp32 matrix entry is the exact sum of
// three bf16 numbers (8 + 8 + 8 bits of its significand, taken by truncation)
// and a bf16 input is an operand as it lies in memory, so the 128 x 128
// products run as three v_mfma_f32_16x16x32_bf16 products whose terms are
// exact in fp32: the only rounding left is that of the fp32 accumulation.
// The three cost 3/16 of the fp32 matrix time.  The group radii stay on fp32
// MFMAs (their squares don't fit bf16).  131072 rows x 8 heads, K2V2: 809 us
// with fp32 products, 334 us here; 8192 rows x 2 heads, K3V3: 23.7 and
// 21.7 us.  fp32 inputs, and the wider formats (whose packing buffers don't
// fit beside 96 KB of matrix), keep the fp32 products.
//
// A wave takes 32 rows at a time, so that each matrix operand read from LDS
// (96 KB per workgroup, split while it is staged) serves two products, and
// finishes the codes of one 16-wide output tile before it starts the next:
// 16 accumulator registers, so four waves fit a SIMD.  Codes by counting: up
// to three (width <= 2) or seven (width 3) comparisons against thresholds
// held per position, binary search only for tiles that hold wider codes.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));
constexpr int kSplitKWords = 16, kSplitVBits = 4;
constexpr int kSplitRows = 2 * kSub;        // rows of a wave
constexpr int kMatOps = kMatF4 / 2;         // 8-element operands of one matrix: [t][q][lane]

template <int W>
struct LdsKS {
  uint4_t wa[3][kMatOps];                        // W's three parts, A operand order
  float4 ma[8 * 64];                             // group membership, fp32 A operand order
  float4 ta[kHeadDim], tb[kHeadDim];             // first seven thresholds of each position, +inf past its last
  uint32_t rw[W][kSplitRows * kSplitKWords];     // per wave: packed key rows, k_words apart
  float sc[W][kSplitRows][kMaxGroups];           // per wave: sqrt(d_g) / radius
  uint32_t pm[kHeadDim];                         // bit offset | b << 10 | group << 14
  float thr[kThresholdEntries];
  float gs[kMaxGroups];
  int mw[8];                                     // largest width in each tile of 16 positions
  uint8_t gd[kHeadDim];
};
template <int W>
struct LdsVSplit {
  uint4_t rb[3][kMatOps];                        // Pi_V's three parts, B operand order
  uint32_t vt[W][kHeadDim * kSplitVBits];        // per wave: words of one value tile
  float nv[W][kSplitRows];
  float thr[kThresholdEntries];
};
static_assert(sizeof(LdsKS<kWavesLong>) <= 160 * 1024 && sizeof(LdsVSplit<kWavesLong>) <= 160 * 1024, "LDS");

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

__device__ __forceinline__ float bf16_elem(const uint4_t (&x)[4], int i) {  // i known at compile time
  const uint32_t w = x[i >> 3][(i & 7) >> 1];
  return __uint_as_float(i & 1 ? w & 0xFFFF0000u : w << 16);
}

// Output tile t of the products of the wave's two sub-tiles (KEYS: the matrix
// is the A operand).  The two small parts have their own accumulator.
template <bool KEYS>
__device__ __forceinline__ void split_product(const uint4_t (*mat)[kMatOps], int t, int lane, const uint4_t (&x)[2][4],
                                              float4_t (&out)[2]) {
  float4_t hi[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, lo[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int o = (t * 4 + q) * 64 + lane;
    const uint4_t w0 = mat[0][o], w1 = mat[1][o], w2 = mat[2][o];
#pragma unroll
    for (int s = 0; s < 2; ++s) lo[s] = KEYS ? mfma_bf16(w2, x[s][q], lo[s]) : mfma_bf16(x[s][q], w2, lo[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) hi[s] = KEYS ? mfma_bf16(w0, x[s][q], hi[s]) : mfma_bf16(x[s][q], w0, hi[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) lo[s] = KEYS ? mfma_bf16(w1, x[s][q], lo[s]) : mfma_bf16(x[s][q], w1, lo[s]);
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) out[s] = hi[s] + lo[s];
}

template <int W>
__device__ __forceinline__ void quant_keys_split(LdsKS<W>& S, int bx, int iters, const Dims& d,
                                                 const uint8_t* __restrict__ blob, const void* __restrict__ kin,
                                                 int n_new, const int32_t* __restrict__ wpos, const CachePtrs& c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y, lz = blockIdx.z;
  const int layer = d.layer >= 0 ? d.layer : lz / d.batch;
  const int seq = lz % d.batch;
  const int cap = d.capacity;
  const int wp = wpos[seq];
  if (wp < 0 || wp >= cap) return;
  const int n_fit = min(n_new, cap - wp);  // rows that fit (the host rejects overflow)
  constexpr int kThreads = W * 64;
  const int r_wg = bx * W * kSplitRows * iters;
  if (r_wg >= n_fit) return;
  const int n_rows_blob = d.n_layers * d.n_kv;
  const int ri = layer * d.n_kv + head;
  const RowMeta* M = reinterpret_cast<const RowMeta*>(blob + kOffRows) + ri;
  const float* gthr = reinterpret_cast<const float*>(blob + kOffThr);
  const int ng = M->n_groups, kw = d.k_words;

  for (int i = tid; i < W * kSplitRows * kSplitKWords; i += kThreads) (&S.rw[0][0])[i] = 0u;
  for (int i = tid; i < kThresholdEntries; i += kThreads) S.thr[i] = gthr[i];
  if (tid < kHeadDim) {
    const int g = M->grp[tid], b = M->width[tid], n = (1 << b) - 1;
    S.gd[M->dim[tid]] = static_cast<uint8_t>(g);
    S.pm[tid] = static_cast<uint32_t>(M->bitoff[tid]) | (static_cast<uint32_t>(b) << 10) |
                (static_cast<uint32_t>(g) << 14);
    float th[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) th[j] = j < n ? gthr[thr_index(b) + j] : __builtin_huge_valf();
    S.ta[tid] = make_float4(th[0], th[1], th[2], th[3]);
    S.tb[tid] = make_float4(th[4], th[5], th[6], th[7]);
  }
  if (tid < kMaxGroups) {
    S.gs[tid] = tid < ng ? sqrtf(static_cast<float>(M->g_dim[tid])) : 0.f;
    int w = 0;
    for (int j = 0; j < 16; ++j) w = max(w, static_cast<int>(M->width[16 * tid + j]));
    S.mw[tid] = w;
  }
  stage_split<W>(S.wa, reinterpret_cast<const float4*>(blob + layout_kdense_offset(n_rows_blob)) +
                           static_cast<size_t>(ri) * kMatF4,
                 tid);
  __syncthreads();
  for (int i = tid; i < 8 * 64; i += kThreads) {
    const int s4 = i >> 6, l = i & 63, g = l & 15, d0 = 32 * (l >> 4) + 4 * s4;
    S.ma[i] = make_float4(S.gd[d0] == g ? 1.f : 0.f, S.gd[d0 + 1] == g ? 1.f : 0.f, S.gd[d0 + 2] == g ? 1.f : 0.f,
                          S.gd[d0 + 3] == g ? 1.f : 0.f);
  }
  __syncthreads();

  const int tk = lane & 15, kk = lane >> 4;
  const int nslot = (ng + 1) & ~1;
  const size_t row = (static_cast<size_t>(layer) * d.batch + seq) * d.n_kv + head;
  for (int it = 0; it < iters; ++it) {
    const int r0 = r_wg + (it * W + wave) * kSplitRows;
    if (r0 >= n_fit) break;  // wave-uniform
    uint4_t x[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int r = r0 + kSub * s + tk;
      load_operands(kin, ((static_cast<size_t>(lz) * n_new + r) * d.n_kv + head) * kHeadDim + 32 * kk, r < n_fit, x[s]);
    }
    // group radii: R2[g][row] = sum_d [group(d) = g] x[row][d]^2
    float4_t n2[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
      const float4 m = S.ma[s4 * 64 + lane];
      const float me[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const float v = bf16_elem(x[s], 4 * s4 + e);
          n2[s] = mfma(me[e], v * v, n2[s]);
        }
      __builtin_amdgcn_sched_barrier(0);  // (eight steps' squares at once would spill)
    }
    // this lane holds R2 of rows tk, 16 + tk for groups 4 kk .. 4 kk + 3
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int g = 4 * kk + i, r = r0 + kSub * s + tk;
        if (g < ng) {
          const float nrm = sqrtf(n2[s][i]);
          S.sc[wave][kSub * s + tk][g] = nrm > 0.f ? S.gs[g] / nrm : 0.f;
          if (r < n_fit)
            c.k_norms[row * kMaxGroups * cap + static_cast<size_t>(wp + r) * nslot + g] =
                __half_as_ushort(__float2half_rn(nrm));
        }
      }
    wave_sync();
    // Z[p][row] = sum_d W[p][d] x[row][d]; codes of stream positions
    // 16 t + 4 kk + i of a row: one bit field
#pragma unroll 1
    for (int t = 0; t < 8; ++t) {
      const int p0 = 16 * t + 4 * kk;
      float4_t z[2];
      split_product<true>(S.wa, t, lane, x, z);
      uint32_t pm[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) pm[i] = S.pm[p0 + i];
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) z[s][i] *= S.sc[wave][kSub * s + tk][(pm[i] >> 14) & 7];
      const int mw = __builtin_amdgcn_readfirstlane(S.mw[t]);
      uint32_t code[2][4];
      if (mw <= 3) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 th = S.ta[p0 + i];
#pragma unroll
          for (int s = 0; s < 2; ++s)
            code[s][i] = (th.x <= z[s][i] ? 1u : 0u) + (th.y <= z[s][i] ? 1u : 0u) + (th.z <= z[s][i] ? 1u : 0u);
        }
        if (mw == 3) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float t3 = S.ta[p0 + i].w;
            const float4 th = S.tb[p0 + i];
#pragma unroll
            for (int s = 0; s < 2; ++s)
              code[s][i] += (t3 <= z[s][i] ? 1u : 0u) + (th.x <= z[s][i] ? 1u : 0u) + (th.y <= z[s][i] ? 1u : 0u) +
                            (th.z <= z[s][i] ? 1u : 0u);
          }
        }
        // a +inf past a narrow position's last threshold is no threshold
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int s = 0; s < 2; ++s) code[s][i] = min(code[s][i], (1u << ((pm[i] >> 10) & 15)) - 1u);
      } else {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int i = 0; i < 4; ++i) code[s][i] = 0u;
#pragma unroll 1
        for (uint32_t step = 1u << (mw - 1); step > 0; step >>= 1)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int b = (pm[i] >> 10) & 15;
            const bool in = step < (1u << b);  // (thr_index(b) + step - 1 is inside the table for every b)
            const float* th = S.thr + thr_index(b) + step - 1;
#pragma unroll
            for (int s = 0; s < 2; ++s) code[s][i] += in && th[code[s][i]] <= z[s][i] ? step : 0u;
          }
      }
      const int b0 = (pm[0] >> 10) & 15, b1 = b0 + ((pm[1] >> 10) & 15), b2 = b1 + ((pm[2] >> 10) & 15);
      const int nb = b2 + ((pm[3] >> 10) & 15), bo = pm[0] & 1023, w = bo >> 5, sh = bo & 31;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint32_t field = code[s][0] | code[s][1] << b0 | code[s][2] << b1 | code[s][3] << b2;
        uint32_t* dst = &S.rw[wave][(kSub * s + tk) * kw + w];
        atomicOr(dst, field << sh);
        if (sh + nb > 32) atomicOr(dst + 1, field >> (32 - sh));
      }
    }
    wave_sync();
    const int n_w = min(kSplitRows, n_fit - r0) * kw;
    uint32_t* out = c.k_codes + (row * cap + wp + r0) * kw;
    for (int idx = lane; idx < kSplitRows * kw; idx += 64) {
      if (idx < n_w) out[idx] = S.rw[wave][idx];
      S.rw[wave][idx] = 0u;
    }
    wave_sync();
  }
}

// The BV-bit codes of one value tile, ORed into its words.
template <int BV, int W>
__device__ __forceinline__ void value_tiles(LdsVSplit<W>& S, int wave, int lane, const uint4_t (&x)[2][4], int s_lo,
                                            int s_hi) {
  constexpr int kThr = (1 << BV) - 1;
  const int tk = lane & 15, kk = lane >> 4;
  const float sq = sqrtf(static_cast<float>(kHeadDim));
  float scl[2][4], thr[BV <= 3 ? kThr : 1];
  uint32_t keep[2] = {0u, 0u};
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = kSub * h + 4 * kk + i;
      const float n = S.nv[wave][s];
      scl[h][i] = n > 0.f ? sq / n : 0.f;
      keep[h] |= (s >= s_lo && s < s_hi ? ((1u << BV) - 1u) : 0u) << (i * BV);
    }
  if constexpr (BV <= 3) {
#pragma unroll
    for (int j = 0; j < kThr; ++j)
      thr[j] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(S.thr[thr_index(BV) + j])));
  }
#pragma unroll 1
  for (int t = 0; t < 8; ++t) {
    // Z[row][j] = sum_d x[row][d] Pi_V[j][d]; this lane: coordinate j of
    // rows 16 h + 4 kk + i
    float4_t z[2];
    split_product<false>(S.rb, t, lane, x, z);
    const int j = 16 * t + tk;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int bit = (kSub * h + 4 * kk) * BV, w = bit >> 5, sh = bit & 31;
      uint32_t field = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = z[h][i] * scl[h][i];
        uint32_t code = 0;
        if constexpr (BV <= 3) {
#pragma unroll
          for (int e = 0; e < kThr; ++e) code += thr[e] <= v ? 1u : 0u;
        } else {
          code = scalar_code(S.thr + thr_index(BV), BV, v);
        }
        field |= code << (i * BV);
      }
      field &= keep[h];
      atomicOr(&S.vt[wave][j * BV + w], field << sh);
      if (sh + 4 * BV > 32) atomicOr(&S.vt[wave][j * BV + w + 1], field >> (32 - sh));
    }
  }
}

template <int W, int BV>
__device__ __forceinline__ void quant_values_split(LdsVSplit<W>& S, int bx, int iters, const Dims& d,
                                                   const uint8_t* __restrict__ blob, const void* __restrict__ vin,
                                                   int n_new, const int32_t* __restrict__ wpos, const CachePtrs& c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y, lz = blockIdx.z;
  const int layer = d.layer >= 0 ? d.layer : lz / d.batch;
  const int seq = lz % d.batch;
  const int cap = d.capacity;
  constexpr int bv = BV;
  const int wp = wpos[seq];
  if (wp < 0 || wp >= cap) return;
  const int n_fit = min(n_new, cap - wp);
  const int tile0 = wp / kTile, n_tiles = (wp + n_fit - 1) / kTile - tile0 + 1;
  const int tw0 = bx * W * iters;
  if (tw0 >= n_tiles) return;
  const float* gthr = reinterpret_cast<const float*>(blob + kOffThr);
  for (int i = tid; i < kThresholdEntries; i += W * 64) S.thr[i] = gthr[i];
  stage_split<W>(S.rb, reinterpret_cast<const float4*>(blob + layout_rotv_mfma_offset(d.n_layers * d.n_kv)), tid);
  __syncthreads();

  const int tk = lane & 15, kk = lane >> 4;
  const size_t row = (static_cast<size_t>(layer) * d.batch + seq) * d.n_kv + head;
  for (int it = 0; it < iters; ++it) {
    const int tw = tw0 + it * W + wave;
    if (tw >= n_tiles) break;  // wave-uniform
    const int tile = tile0 + tw, P0 = tile * kTile;
    const int s_lo = max(P0, wp) - P0, s_hi = min(P0 + kTile, wp + n_fit) - P0;  // rows [s_lo, s_hi) are new
    uint4_t x[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int slot = kSub * h + tk;
      load_operands(vin, ((static_cast<size_t>(lz) * n_new + (P0 + slot - wp)) * d.n_kv + head) * kHeadDim + 32 * kk,
                    slot >= s_lo && slot < s_hi, x[h]);
    }
    uint32_t* gv = c.v_codes + (row * (cap / kTile) + tile) * kHeadDim * static_cast<size_t>(bv);
    // tile words: zero, or the old words with the new rows' bits cleared
    if (s_lo == 0 && s_hi == kTile) {
      for (int idx = lane; idx < kHeadDim * bv; idx += 64) S.vt[wave][idx] = 0u;
    } else {
      for (int idx = lane; idx < kHeadDim * bv; idx += 64) {
        const int w = idx % bv;
        const int lo_b = max(s_lo * bv - 32 * w, 0), hi_b = min(s_hi * bv - 32 * w, 32);
        const uint32_t mask = hi_b <= lo_b ? 0u : (hi_b - lo_b == 32 ? ~0u : ((1u << (hi_b - lo_b)) - 1u) << lo_b);
        S.vt[wave][idx] = gv[idx] & ~mask;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int slot = kSub * h + tk;
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 32; ++i) ss = fmaf(bf16_elem(x[h], i), bf16_elem(x[h], i), ss);
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      const float nrm = sqrtf(ss);
      if (kk == 0) {
        S.nv[wave][slot] = nrm;
        if (slot >= s_lo && slot < s_hi) c.v_norms[row * cap + P0 + slot] = __half_as_ushort(__float2half_rn(nrm));
      }
    }
    wave_sync();
    value_tiles<BV, W>(S, wave, lane, x, s_lo, s_hi);
    wave_sync();
    for (int idx = lane; idx < kHeadDim * bv; idx += 64) gv[idx] = S.vt[wave][idx];
    wave_sync();
  }
}

// Grid as k_quant_rows; the key workgroups (the longer ones) come first.
template <int W, int BV>
__global__ __launch_bounds__(W * 64) void k_quant_rows_bf16(Dims d, const uint8_t* __restrict__ blob,
                                                             const void* __restrict__ kin,
                                                             const void* __restrict__ vin, int n_new,
                                                             const int32_t* __restrict__ wpos, CachePtrs c, int n_kwg,
                                                             int k_iters, int v_iters) {
  constexpr size_t kBytes = sizeof(LdsKS<W>) > sizeof(LdsVSplit<W>) ? sizeof(LdsKS<W>) : sizeof(LdsVSplit<W>);
  __shared__ __attribute__((aligned(16))) uint8_t smem[kBytes];
  const int bx = static_cast<int>(blockIdx.x);
  if (bx < n_kwg)
    quant_keys_split<W>(*reinterpret_cast<LdsKS<W>*>(smem), bx, k_iters, d, blob, kin, n_new, wpos, c);
  else
    quant_values_split<W, BV>(*reinterpret_cast<LdsVSplit<W>*>(smem), bx - n_kwg, v_iters, d, blob, vin, n_new, wpos, c);
}

}  // namespace quant_detail

hipError_t launch_quantize_prefill(const Dims& d, const void* layout, const void* k, const void* v, int n_new,
                                   const int32_t* write_pos, const CachePtrs& c, hipStream_t s) {
  using namespace quant_detail;
  const uint8_t* blob = static_cast<const uint8_t*>(layout);
  const int lz = d.batch * d.n_lc;
  // rows per workgroup: small calls spread over more workgroups (one
  // sub-tile or value tile per wave, 4-wave workgroups up to 64K rows), large
  // ones amortise the 64 KB matrix staged in LDS over more rows
  const long rows = static_cast<long>(n_new) * d.n_kv * lz;
  const int k_iters = rows <= 256L * 256 ? 1 : (rows <= 4L * 256 * 512 ? 2 : 4);
  const int v_iters = rows <= 256L * 512 ? 1 : 2;
  const auto go = [&](auto kern, int w) {
    const int n_kwg = (n_new + w * kSub * k_iters - 1) / (w * kSub * k_iters);
    // value tiles per workgroup: w v_iters (a wave per tile), or 2 (short calls)
    const int vt_wg = w == kWavesLong ? w * v_iters : kWavesShort / 2;
    const int n_vwg = (n_new / kTile + 2 + vt_wg - 1) / vt_wg;
    const dim3 grid(n_kwg + n_vwg, d.n_kv, lz);
    hipLaunchKernelGGL(kern, grid, dim3(w * 64), 0, s, d, blob, k, v, n_new, write_pos, c, n_kwg, n_vwg, k_iters,
                       v_iters);
  };
  const bool bf = d.in_dtype == 1, short_call = rows <= 256L * 256;
  if (bf && d.k_words <= kSplitKWords && d.v_bits <= kSplitVBits) {
    const auto split = [&](auto kern, int w, int iters) {
      const int n_kwg = (n_new + w * kSplitRows * iters - 1) / (w * kSplitRows * iters);
      const int n_vwg = (n_new / kTile + 2 + w * iters - 1) / (w * iters);
      hipLaunchKernelGGL(kern, dim3(n_kwg + n_vwg, d.n_kv, lz), dim3(w * 64), 0, s, d, blob, k, v, n_new, write_pos, c,
                         n_kwg, iters, iters);
    };
    const auto by_width = [&](auto bv) {
      if (short_call) split(k_quant_rows_bf16<kWavesShort, bv.value>, kWavesShort, 1);
      else split(k_quant_rows_bf16<kWavesLong, bv.value>, kWavesLong, rows <= 4L * 256 * 512 ? 1 : 4);
    };
    if (d.v_bits == 1) by_width(std::integral_constant<int, 1>{});
    else if (d.v_bits == 2) by_width(std::integral_constant<int, 2>{});
    else if (d.v_bits == 3) by_width(std::integral_constant<int, 3>{});
    else by_width(std::integral_constant<int, kSplitVBits>{});
    return hipGetLastError();
  }
  if (short_call) {
    if (bf) go(k_quant_rows<true, kWavesShort>, kWavesShort);
    else go(k_quant_rows<false, kWavesShort>, kWavesShort);
  } else {
    if (bf) go(k_quant_rows<true, kWavesLong>, kWavesLong);
    else go(k_quant_rows<false, kWavesLong>, kWavesLong);
  }
  return hipGetLastError();
}

}  // namespace bgtq
