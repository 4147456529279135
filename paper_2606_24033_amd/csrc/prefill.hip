// Causal prefill attention over the packed cache (Sec. 4, prefill paragraph):
// each workgroup owns a tile of query rows, streams the packed K/V tiles of
// its (layer, sequence, KV head) up to the tile's last position, decodes each
// tile once into LDS for all of its query rows, and accumulates QK^T and PV
// with a causal mask under an online softmax.  No fp16 cache and no attention
// matrix is written.
//
// Two launches on the caller's stream:
//  1. k_prefill_qrot_bf16 (bf16 queries on 16-byte aligned buffers) or
//     k_prefill_qrot: the Q-side rotation of every query row into the key
//     stream order, qr[p] = log2 e (Pi_g q_g)_j / sqrt(d_g d_h) at stream
//     position p = g_pos[g] + j (fp32, into the caller's workspace);
//  2. k_prefill_attn: the attention, 256 query rows per workgroup (8 waves of
//     32 rows; 128 rows, two waves per 32, in short calls).  Decoded key tile:
//     radius x centroid, exact in fp16 hi + lo parts, so that hi/lo query x
//     hi/lo key (three MFMA passes, the lo x lo product left out) carries
//     ~fp32 precision through one full-width product per 16 coordinates; the
//     value tile holds the bare fp16 centroids (exact) and the value radius
//     enters the softmax weight.  Products run transposed, S^T = K Q^T and
//     O^T = V^T P^T, so that the softmax weights go from the S^T accumulators
//     straight into the B operand of the PV product (no trip through LDS).
//     The decoded tiles are double-buffered: while a tile's products run, the
//     same waves decode the next tile into the other buffer; one barrier per
//     tile.  Its epilogue: out = Pi_V^T o, with fp32 MFMAs.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "layout.h"
#include "mix.h"
#include "split.h"

namespace bgtq {
namespace prefill_detail {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

typedef float float16_t __attribute__((ext_vector_type(16)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;      // rotation kernel: 4 waves
constexpr int kAttnWaves = 8;      // attention kernel: 8 waves (2 per SIMD)
constexpr int kAttnThreads = kAttnWaves * 64;
constexpr int kWaveRows = 32;      // query rows (position x head) of a wave: one 32x32 column block
constexpr int kQrotRows = 512;     // query rows (position x head) per rotation workgroup
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegInf = -__builtin_huge_valf();
// ---- LDS map of the attention kernel (bytes)
constexpr int kKStride = 136;  // halves per decoded key row (128 + 8 pad)
constexpr int kVStride = 72;   // halves per decoded value row (64 + 8 pad: 16-byte aligned, conflict-free reads)
// decoded tile (two buffers): keys hi, lo [64 tokens][kKStride] fp16, values
// [128 dims][kVStride] fp16, value radii [64] fp16
constexpr int kDecKH = 0;
constexpr int kDecKL = kDecKH + 64 * kKStride * 2;
constexpr int kDecV = kDecKL + 64 * kKStride * 2;
constexpr int kDecVN = kDecV + 128 * kVStride * 2;
constexpr int kDecBytes = kDecVN + 64 * 2;
constexpr int kOffCb = 0;                        // fp16 codebooks
constexpr int kOffPair = kOffCb + 1024;          // pair tables of the widths 1 .. kMaxPair
constexpr int kMaxPair = 6;
// byte offset of the pair table of width b: 4^b entries of two fp16 centroids
__host__ __device__ constexpr int pair_offset(int b) { return 4 * (((1 << (2 * b)) - 4) / 3); }
// (the tables lie below 64 KB: their offsets fit the immediate of an LDS read)
constexpr int kOffDec = (kOffPair + pair_offset(kMaxPair + 1) + 15) / 16 * 16;
constexpr int kTileLds = kOffDec + 2 * kDecBytes;
constexpr int kRotVLds = kHeadDim * kHeadDim * 4;  // Pi_V staged for the epilogue
constexpr int kMergeLds = (kAttnWaves / 2) * 64 * 66 * 4;  // states of the waves that hand theirs over (KS = 2)
constexpr int kLdsBytes = kTileLds > kRotVLds ? (kTileLds > kMergeLds ? kTileLds : kMergeLds)
                                              : (kRotVLds > kMergeLds ? kRotVLds : kMergeLds);
static_assert(kLdsBytes <= 160 * 1024, "LDS of one workgroup");
static_assert(kDecBytes % 16 == 0 && kDecV % 16 == 0 && kOffDec % 16 == 0, "aligned buffers");
static_assert(2 * kCodebookEntries <= 1024, "codebook staging");

// Load of a T at a 32-bit byte offset from a wave-uniform base (the global
// load form with a scalar base and a 32-bit vector offset).
template <class T>
__device__ __forceinline__ T ld_at(const void* base, uint32_t byte_off) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + byte_off);
}

// r0, r1 = the values of lanes l % 32 and l % 32 + 32 (the two lanes that hold
// the same query row of an accumulator); gfx950 lane swap
__device__ __forceinline__ void swap32(float v, float& r0, float& r1) {
  unsigned x = __builtin_bit_cast(unsigned, v), y = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  r0 = __builtin_bit_cast(float, x);
  r1 = __builtin_bit_cast(float, y);
}
__device__ __forceinline__ float max2g(float v) {
  float a, b;
  swap32(v, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum2g(float v) {
  float a, b;
  swap32(v, a, b);
  return a + b;
}

__device__ __forceinline__ float ld_q(const void* q, size_t i, int in_dtype) {  // BGTQ_BF16 = 1
  if (in_dtype == 1) {
    const uint16_t b = static_cast<const uint16_t*>(q)[i];
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
  }
  return static_cast<const float*>(q)[i];
}

// ---------------------------------------------------------------- 1. rotation
// grid (ceil(n_q G / kQrotRows), n_kv, batch).  qr: [batch][n_q][Hq][128]
// fp32.  The rotation of a query row is one product with a 128 x 128 matrix
// in stream order, W[p][k] = log2 e / sqrt(d_g d_h) Pi_g[j][k - g_pos] for
// p = g_pos + j and k in the same group g (zero elsewhere), applied to the
// row gathered into stream order.  W is staged in LDS once per workgroup
// (transposed, Wt[k][p]); each wave multiplies 16-row tiles by it with fp32
// MFMAs (16x16x4: 32 steps of 4 coordinates x 8 tiles of 16 outputs).
__global__ __launch_bounds__(kThreads) void k_prefill_qrot(Dims d, const uint8_t* __restrict__ blob,
                                                           const void* __restrict__ q, int n_q,
                                                           float* __restrict__ qr) {
  __shared__ float wt[kHeadDim * kHeadDim];                  // Wt[k][p]
  __shared__ float qs[kThreads / 64][16][kHeadDim + 4];      // per wave: 16 rows in stream order
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kvh = blockIdx.y, seq = blockIdx.z;
  const int G = d.group, hq = d.n_kv * G;
  const int n_rows_blob = d.n_layers * d.n_kv;
  const RowMeta* M = reinterpret_cast<const RowMeta*>(blob + kOffRows) + (d.layer * d.n_kv + kvh);
  const float* rowrot = reinterpret_cast<const float*>(blob + layout_rowrot_offset(n_rows_blob)) +
                        static_cast<size_t>(d.layer * d.n_kv + kvh) * kRowRotFloats;
  for (int i = tid; i < kHeadDim * kHeadDim; i += kThreads) wt[i] = 0.f;
  __syncthreads();
  {
    // column p (thread & 127) of Wt: the rotation row j = p - g_pos of its group
    const int p = tid & 127;
    const int g = M->grp[p], p0 = M->g_pos[g], dg = M->g_dim[g], j = p - p0;
    int off = 0;
    for (int e = 0; e < g; ++e) off += M->g_dim[e] * M->g_dim[e];
    const float scale = kLog2e * rsqrtf(static_cast<float>(dg) * kHeadDim);
    for (int k = tid >> 7; k < dg; k += kThreads / kHeadDim)
      wt[(p0 + k) * kHeadDim + p] = rowrot[off + k * dg + j] * scale;  // Pi_dg transposed: [k dg + j] = Pi[j][k]
  }
  const int dimk = M->dim[lane], dimk2 = M->dim[lane + 64];  // stream position -> source dim
  __syncthreads();
  const int nr = n_q * G;
  const int r_wg = blockIdx.x * kQrotRows;
  float (*qw)[kHeadDim + 4] = qs[wave];
  for (int t0 = r_wg + wave * 16; t0 < min(r_wg + kQrotRows, nr); t0 += kThreads / 4) {
    // gather 16 rows into stream order (rows past the end are zero)
    for (int r = 0; r < 16; ++r) {
      const int row = t0 + r;
      float a = 0.f, b = 0.f;
      if (row < nr) {
        const int i = row / G, h = row - (row / G) * G;
        const size_t base = ((static_cast<size_t>(seq) * n_q + i) * hq + kvh * G + h) * kHeadDim;
        a = ld_q(q, base + dimk, d.in_dtype);
        b = ld_q(q, base + dimk2, d.in_dtype);
      }
      qw[r][lane] = a;
      qw[r][lane + 64] = b;
    }
    // one wave writes and reads its own rows: LDS operations of a wave
    // complete in order, so only the compiler must keep the order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float4_t acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
    const int ar = lane & 15, ak = lane >> 4;
#pragma unroll 4
    for (int st = 0; st < kHeadDim / 4; ++st) {
      const float a = qw[ar][4 * st + ak];
      const float* wrow = wt + (4 * st + ak) * kHeadDim + ar;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, wrow[16 * t], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = t0 + 4 * ak + i;
      if (row < nr) {
        const int qi = row / G, h = row - (row / G) * G;
        float* dst = qr + ((static_cast<size_t>(seq) * n_q + qi) * hq + kvh * G + h) * kHeadDim + ar;
#pragma unroll
        for (int t = 0; t < 8; ++t) dst[16 * t] = acc[t][i];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // reads of these rows before the next tile's writes
    __builtin_amdgcn_wave_barrier();
  }
}

// The same for bf16 queries on 16-byte aligned buffers: three exact bf16
// products with the key rotation on the natural dims (the gather into stream
// order folded in) and the scale applied to the sums.  A wave takes 32 rows;
// 4-wave workgroups for calls of up to 64K rows, which then spread over more
// CUs.  The traffic bounds it (256 B in, 512 B out per row).
// Against fp32 products (a 2-byte gather through LDS), both in turn in one
// run: 32768 positions x 32 heads 1.23 and 0.16 ms (5.0 TB/s), the attention
// behind it 15.4 and 14.9 ms, the whole call 16.55 and 14.93 ms; 1001 positions
// x 16 heads after 15003 rows, the call: 575 and 460 us.
template <int W>
__global__ __launch_bounds__(W * 64) void k_prefill_qrot_bf16(Dims d, const uint8_t* __restrict__ blob,
                                                              const void* __restrict__ q, int n_q, int iters,
                                                              float* __restrict__ qr) {
  using namespace split;
  __shared__ uint4_t wa[3][kMatOps];
  __shared__ float scale[kHeadDim];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tk = lane & 15, kk = lane >> 4;
  const int kvh = blockIdx.y, seq = blockIdx.z;
  const int G = d.group, hq = d.n_kv * G, nr = n_q * G;
  const int ri = d.layer * d.n_kv + kvh;
  const RowMeta* M = reinterpret_cast<const RowMeta*>(blob + kOffRows) + ri;
  if (tid < kHeadDim) scale[tid] = kLog2e * rsqrtf(static_cast<float>(M->g_dim[M->grp[tid]]) * kHeadDim);
  stage_split<W>(wa, reinterpret_cast<const float4*>(blob + layout_kdense_offset(d.n_layers * d.n_kv)) +
                         static_cast<size_t>(ri) * kMatF4,
                 tid);
  __syncthreads();
  for (int it = 0; it < iters; ++it) {
    const int r0 = ((blockIdx.x * iters + it) * W + wave) * kSplitRows;
    if (r0 >= nr) break;  // wave-uniform
    uint4_t x[2][4];
    size_t off[2];
    bool valid[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int r = r0 + kSub * s + tk, i = r / G, h = r - i * G;
      valid[s] = r < nr;
      off[s] = ((static_cast<size_t>(seq) * n_q + i) * hq + kvh * G + h) * kHeadDim;
      load_operands(q, off[s] + 32 * kk, valid[s], x[s]);
    }
#pragma unroll 2
    for (int t = 0; t < 8; ++t) {
      // this lane: stream positions 16 t + 4 kk .. + 3 of rows tk, 16 + tk
      float4_t z[2];
      split_product(wa, t, lane, x, z);
      const float4_t sc = *reinterpret_cast<const float4_t*>(&scale[16 * t + 4 * kk]);
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (valid[s]) *reinterpret_cast<float4_t*>(qr + off[s] + 16 * t + 4 * kk) = z[s] * sc;
    }
  }
}

// ---------------------------------------------------------------- 2. attention
// Lane roles in the products (32x32x16 f16 MFMAs; l32 = lane % 32, hf =
// lane / 32): the A operand comes from the decoded tile (token or dim l32 of
// a 32-block, 8 consecutive k from 8 hf), the B operand is the wave's 32 query
// rows (row l32, the same k), and an accumulator's register r holds token
// (S^T) or dim (O^T) 8 (r / 4) + 4 hf + r % 4 of its 32-block for row l32.
// The softmax weights of a lane are therefore, 8 registers at a time, a B
// operand of O^T = V^T P^T whose k runs over tokens {4 hf + i, 8 + 4 hf + i}
// of a 16-token step; the value tile stores the tokens of a step in that
// order (0-3, 8-11, 4-7, 12-15), so that its operand is one 16-byte read.

// Bits [POS, POS + LEN) of the little-endian word array w, placed at bit SH.
template <int POS, int LEN, int SH, int N>
__device__ __forceinline__ uint32_t field_at(const uint32_t (&w)[N]) {
  constexpr int wi = POS / 32, sh = POS % 32;
  static_assert(wi < N && SH + LEN <= 32, "field");
  uint32_t v;
  if constexpr (sh + LEN > 32) {
    static_assert(wi + 1 < N && sh >= SH, "field word");
    v = __builtin_amdgcn_alignbit(w[wi + 1], w[wi], sh - SH);
  } else if constexpr (sh >= SH) {
    v = w[wi] >> (sh - SH);
  } else {
    v = w[wi] << (SH - sh);
  }
  return v & (((1u << LEN) - 1u) << SH);
}

// Two consecutive BV-bit codes at bit POS of w -> two fp16 centroids.
template <int BV, int POS, int N>
__device__ __forceinline__ uint32_t value_pair(const uint8_t* smem, const uint32_t (&w)[N]) {
  if constexpr (BV <= kMaxPair) {
    return *reinterpret_cast<const uint32_t*>(smem + kOffPair + pair_offset(BV) + field_at<POS, 2 * BV, 2>(w));
  } else {
    const uint32_t c0 = *reinterpret_cast<const uint16_t*>(smem + kOffCb + 2 * cb_index(BV) + field_at<POS, BV, 1>(w));
    const uint32_t c1 =
        *reinterpret_cast<const uint16_t*>(smem + kOffCb + 2 * cb_index(BV) + field_at<POS + BV, BV, 1>(w));
    return c0 | (c1 << 16);
  }
}

// Key decode.  A key row is 32 items of 4 consecutive stream positions: two
// pairs, each inside one group (groups have even sizes), whose codes are one
// dense field of 2 bA + 2 bB <= 32 bits.  Lane = token; a wave decodes the
// items wave + 8 j, so that everything that describes an item is
// wave-uniform, and stores 8 bytes per item and token.
constexpr int kItemsPer = kHeadDim / 4 / kAttnWaves;
struct KeyItems {
  uint32_t word[kItemsPer];                     // byte offset of the first of the two words that are loaded
  uint32_t sh[kItemsPer];                       // first bit of the field in them
  uint32_t wa[kItemsPer], wb[kItemsPer];        // 2 bA, 2 bB
  uint32_t ta[kItemsPer], tb[kItemsPer];        // offsets of the widths' pair tables
  uint32_t sel_lo[kItemsPer], sel_hi[kItemsPer];  // byte selectors that pick (rA, rB) from the token's 8 radii:
                                                // groups 0-3 and 4-7, a radius in the other half selects zero
  bool wide;                                    // some width is above kMaxPair: codes looked up one by one
};
// Raw words of a thread's share of one tile.
template <int BV>
struct Raw {
  static constexpr int kVW = (BV + 1) / 2;  // words of 16 value codes
  uint2 k[kItemsPer];
  uint4 kn;
  uint32_t v[kVW];
  uint32_t vn;
};
__device__ __forceinline__ KeyItems key_items(const RowMeta* M, int wave, int kw) {
  KeyItems k;
  k.wide = false;
#pragma unroll
  for (int j = 0; j < kItemsPer; ++j) {
    const int p = 4 * (wave + kAttnWaves * j);
    const auto uni = [](uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))); };
    const uint32_t off = uni(M->bitoff[p]), ba = uni(M->width[p]), bb = uni(M->width[p + 2]), ga = uni(M->grp[p]),
                   gb = uni(M->grp[p + 2]);
    const uint32_t w0 = min(off >> 5, static_cast<uint32_t>(kw - 2));  // (a row has at least 4 words)
    const auto tab = [](uint32_t b) { return static_cast<uint32_t>(kOffPair) + 4 * (((1u << (2 * b)) - 4u) / 3u); };
    const auto sel = [](uint32_t g) { return 2 * (g & 3u) | (2 * (g & 3u) + 1) << 8; };
    k.word[j] = 4 * w0;
    k.sh[j] = off - 32 * w0;
    k.wa[j] = 2 * ba;
    k.wb[j] = 2 * bb;
    k.ta[j] = tab(ba);
    k.tb[j] = tab(bb);
    k.sel_lo[j] = (ga < 4 ? sel(ga) : 0x0C0Cu) | (gb < 4 ? sel(gb) : 0x0C0Cu) << 16;
    k.sel_hi[j] = (ga < 4 ? 0x0C0Cu : sel(ga)) | (gb < 4 ? 0x0C0Cu : sel(gb)) << 16;
    k.wide = k.wide || ba > kMaxPair || bb > kMaxPair;
  }
  return k;
}
// The centroids of the wave's items (c.x: pair A, c.y: pair B).
template <bool WIDE>
__device__ __forceinline__ void key_lookups(const uint8_t* smem, const KeyItems& it, const uint2 (&w)[kItemsPer],
                                            uint2 (&c)[kItemsPer]) {
#pragma unroll
  for (int j = 0; j < kItemsPer; ++j) {
    const uint32_t f = static_cast<uint32_t>((static_cast<uint64_t>(w[j].y) << 32 | w[j].x) >> it.sh[j]);
    if constexpr (!WIDE) {
      c[j].x = *reinterpret_cast<const uint32_t*>(smem + it.ta[j] + 4 * __builtin_amdgcn_ubfe(f, 0, it.wa[j]));
      c[j].y = *reinterpret_cast<const uint32_t*>(smem + it.tb[j] + 4 * __builtin_amdgcn_ubfe(f, it.wa[j], it.wb[j]));
    } else {
      const uint32_t ba = it.wa[j] >> 1, bb = it.wb[j] >> 1;
      const auto one = [&](uint32_t at, uint32_t b) {
        return static_cast<uint32_t>(*reinterpret_cast<const uint16_t*>(
            smem + kOffCb + 2 * ((1u << b) - 2u + __builtin_amdgcn_ubfe(f, at, b))));
      };
      c[j].x = one(0, ba) | one(ba, ba) << 16;
      c[j].y = one(2 * ba, bb) | one(2 * ba + bb, bb) << 16;
    }
  }
}
// Item j: centroids times the groups' radii, as fp16 hi and lo parts.  The
// product of two fp16 numbers has at most 22 significant bits: hi =
// fp16(r c) and the fused residual lo = fp16(r c - hi) carry all of them above
// fp16's subnormal step.  dst: the item's place in the token's decoded row.
__device__ __forceinline__ void key_store(uint8_t* dst, const KeyItems& it, int j, const uint4& radii, const uint2& c) {
  const uint32_t r =
      __builtin_amdgcn_perm(radii.y, radii.x, it.sel_lo[j]) | __builtin_amdgcn_perm(radii.w, radii.z, it.sel_hi[j]);
  const half2_t rr = __builtin_bit_cast(half2_t, r);
  const half2_t ra = {rr[0], rr[0]}, rb = {rr[1], rr[1]};
  const half2_t ca = __builtin_bit_cast(half2_t, c.x), cb = __builtin_bit_cast(half2_t, c.y);
  const half2_t ha = ra * ca, hb = rb * cb;
  const half2_t la = __builtin_elementwise_fma(ra, ca, -ha), lb = __builtin_elementwise_fma(rb, cb, -hb);
  *reinterpret_cast<uint2*>(dst + kDecKH) =
      make_uint2(__builtin_bit_cast(uint32_t, ha), __builtin_bit_cast(uint32_t, hb));
  *reinterpret_cast<uint2*>(dst + kDecKL) =
      make_uint2(__builtin_bit_cast(uint32_t, la), __builtin_bit_cast(uint32_t, lb));
}

// Value decode: thread = (dim tid % 128, 16-token step tid / 128); a holds
// tokens 0-3 and 8-11 of the step, b tokens 4-7 and 12-15.
template <int BV>
__device__ __forceinline__ void value_lookups(const uint8_t* smem, const Raw<BV>& raw, int quarter, uint4& a, uint4& b) {
  constexpr int NW = Raw<BV>::kVW;
  uint32_t w[NW];
  if constexpr (BV % 2 == 0) {
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = raw.v[i];
  } else {
    const int sh = 16 * (quarter & 1);  // uniform
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = __builtin_amdgcn_alignbit(i + 1 < NW ? raw.v[i + 1] : 0u, raw.v[i], sh);
  }
  a.x = value_pair<BV, 0 * BV>(smem, w);
  a.y = value_pair<BV, 2 * BV>(smem, w);
  b.x = value_pair<BV, 4 * BV>(smem, w);
  b.y = value_pair<BV, 6 * BV>(smem, w);
  a.z = value_pair<BV, 8 * BV>(smem, w);
  a.w = value_pair<BV, 10 * BV>(smem, w);
  b.z = value_pair<BV, 12 * BV>(smem, w);
  b.w = value_pair<BV, 14 * BV>(smem, w);
}
template <int BV>
__device__ __forceinline__ void store_values(uint8_t* dec, const Raw<BV>& raw, int tid, int quarter, const uint4& a,
                                             const uint4& b) {
  uint4* dst = reinterpret_cast<uint4*>(dec + kDecV + (tid & 127) * (2 * kVStride) + 32 * quarter);
  dst[0] = a;
  dst[1] = b;
  // every wave stores the 64 value radii it loaded (the same ones; no branch)
  reinterpret_cast<uint16_t*>(dec + kDecVN)[tid & 63] = static_cast<uint16_t>(raw.vn);
}

// What bounds it: per 64-token tile a SIMD's two waves issue 128 MFMAs of 32
// cycles and 570 other VALU instructions, and meet at one barrier.  On the
// 32K-token Llama-shaped layer (14.9 ms; 23.0 ms with 16x16x32 products and a
// per-code decode through raw words in LDS) the matrix cores are busy 61 % of
// the cycles and the VALU port 52 %; with the softmax and the decode taken out
// (the products, their LDS reads and the barrier stay) it takes 11.5 ms.  The
// waves' softmax and decode phases are only partly hidden behind each other's
// products.  Three passes of the key product and the one of the value product
// make 17.6 TFLOP of matrix work, 1.18 PFLOP/s.
// Tried and slower or equal: two barriers per tile with the halves in
// alternate phases (19.0 ms), the decode spread between the products (18.2),
// four waves of 64 rows, one per SIMD (spills), 32-token blocks (16.4).
//
// grid (n_tiles, n_kv, batch), tiles in reverse order (the longest first).
// KS = 1: a workgroup owns 8 x 32 query rows.  KS = 2: 4 x 32 rows, waves w
// and w + 4 taking the two 32-token halves of every tile for the same rows
// (their states are merged at the end).
template <int BV, int KS>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_prefill_attn(
    Dims d, const uint8_t* __restrict__ blob, const float* __restrict__ qr, int n_q,
    const int32_t* __restrict__ q_pos0, int max_pos, CachePtrs c, float* __restrict__ out) {
  constexpr int kRows = kAttnWaves / KS * kWaveRows, NB = 2 / KS;  // rows of the workgroup; token blocks of a wave
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int n_tiles = gridDim.x;
  const int qt = n_tiles - 1 - static_cast<int>(blockIdx.x);
  const int kvh = blockIdx.y, seq = blockIdx.z;
  const int G = d.group, hq = d.n_kv * G, cap = d.capacity, kw = d.k_words;
  const RowMeta* M = reinterpret_cast<const RowMeta*>(blob + kOffRows) + (d.layer * d.n_kv + kvh);
  const int nslot = (M->n_groups + 1) & ~1;
  const int pos0 = q_pos0[seq];
  const int rw = KS == 1 ? wave : wave & 3;       // the wave's row block
  const int blk0 = KS == 1 ? 0 : wave >> 2;       // its first token block of a tile

  // this lane's query row (position index ri, head rh)
  const int r0 = qt * kRows + rw * kWaveRows;
  const int ri = (r0 + l32) / G, rh = r0 + l32 - ri * G;
  const int pos = max(0, min(pos0 + min(ri, n_q - 1), max_pos));
  // the wave's first (smallest) position: its first row
  const int pos_min = max(0, min(pos0 + min(r0 / G, n_q - 1), max_pos));
  // the workgroup's last position bounds its key loop
  const int i_last = min(n_q - 1, (qt * kRows + kRows - 1) / G);
  const int pos_last = max(0, min(pos0 + i_last, max_pos));
  const int n_kt = pos_last / kKeyTile + 1;

  // query operands (B of S^T = K Q^T): dims 16 ks + 8 hf .. +7 of the row,
  // fp16 hi and lo parts
  half8_t qh[8], ql[8];
  {
    const bool valid = ri < n_q;
    const float* src = qr + ((static_cast<size_t>(seq) * n_q + min(ri, n_q - 1)) * hq + kvh * G + rh) * kHeadDim;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const float4 a = *reinterpret_cast<const float4*>(src + 16 * ks + 8 * hf);
      const float4 b = *reinterpret_cast<const float4*>(src + 16 * ks + 8 * hf + 4);
      const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = valid ? v[e] : 0.f;
        const _Float16 h = static_cast<_Float16>(x);
        qh[ks][e] = h;
        ql[ks][e] = static_cast<_Float16>(x - static_cast<float>(h));
      }
    }
  }
  const KeyItems items = key_items(M, wave, kw);
  // codebooks and pair tables (entry i of width b holds the centroids of codes
  // i % 2^b and i / 2^b), of every width: 5460 entries.  Calls of a tile or a
  // few carry that and are still shorter than with the per-code decode, which
  // needed no tables: one position 27 against 42 us the call, 64 positions 30
  // against 82 us, 64 sequences of 16 positions 71 against 105 us (8 KV heads x 4).
  {
    const uint16_t* c16 = reinterpret_cast<const uint16_t*>(blob + kOffC16);
    uint16_t* cbs = reinterpret_cast<uint16_t*>(smem + kOffCb);
    for (int i = tid; i < kCodebookEntries; i += kAttnThreads) cbs[i] = c16[i];
    __syncthreads();
#pragma unroll
    for (int b = 1; b <= kMaxPair; ++b)
      for (int i = tid; i < (1 << (2 * b)); i += kAttnThreads)
        *reinterpret_cast<uint32_t*>(smem + kOffPair + pair_offset(b) + 4 * i) =
            cbs[cb_index(b) + (i & ((1 << b) - 1))] | (static_cast<uint32_t>(cbs[cb_index(b) + (i >> b)]) << 16);
  }

  const size_t row = (static_cast<size_t>(d.layer) * d.batch + seq) * d.n_kv + kvh;
  const uint8_t* kc = reinterpret_cast<const uint8_t*>(c.k_codes + row * cap * kw);
  const uint8_t* kn = reinterpret_cast<const uint8_t*>(c.k_norms + row * kMaxGroups * cap);
  const uint8_t* vc = reinterpret_cast<const uint8_t*>(c.v_codes + row * (cap / kTile) * kHeadDim * BV);
  const uint16_t* vnp = c.v_norms + row * cap;

  float m_run = kNegInf, l_run = 0.f;
  float16_t o[4];
#pragma unroll
  for (int cc = 0; cc < 4; ++cc)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[cc][i] = 0.f;

  // Raw words of one tile (every token of a tile is below the capacity, a
  // multiple of 64): straight from memory to the registers of the lane that
  // decodes them.
  const int quarter = wave >> 1;  // 16-token step of the value decode
  // Per-thread addresses are recomputed for each tile from an opaque copy of
  // the thread index: hoisted out of the loop they would take the registers
  // that the products need.
  const auto opaque_tid = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  Raw<BV> raw;
  const auto load_raw = [&](int ta) {
    const int tt = opaque_tid();
    const uint8_t* ks = kc + static_cast<size_t>(ta) * kw * 4;
    const uint8_t* ns = kn + static_cast<size_t>(ta) * nslot * 2;
    uint32_t k_at = static_cast<uint32_t>((tt & 63) * kw * 4), n_at = static_cast<uint32_t>((tt & 63) * nslot * 2);
    uint32_t v_lane = static_cast<uint32_t>((tt & 127) * BV * 4), vn_lane = static_cast<uint32_t>((tt & 63) * 2);
#pragma unroll
    for (int j = 0; j < kItemsPer; ++j) {
      raw.k[j].x = ld_at<uint32_t>(ks + items.word[j], k_at);
      raw.k[j].y = ld_at<uint32_t>(ks + items.word[j] + 4, k_at);
    }
    // (a token's 16 bytes of radii stay inside the row's 8 slots per token)
    raw.kn.x = ld_at<uint32_t>(ns, n_at);
    raw.kn.y = ld_at<uint32_t>(ns + 4, n_at);
    raw.kn.z = ld_at<uint32_t>(ns + 8, n_at);
    raw.kn.w = ld_at<uint32_t>(ns + 12, n_at);
    // 16 codes from bit 16 BV (quarter % 2) of the dim's words in value tile quarter / 2
    constexpr int NW = Raw<BV>::kVW;
    const uint8_t* vs = vc + (static_cast<size_t>(ta / kTile) + (quarter >> 1)) * kHeadDim * BV * 4 +
                        4 * (BV * (quarter & 1) / 2);
#pragma unroll
    for (int i = 0; i < NW; ++i) raw.v[i] = ld_at<uint32_t>(vs + 4 * i, v_lane);
    raw.vn = ld_at<uint16_t>(vnp + ta, vn_lane);
  };
  // the thread's share of the decode of the tile whose raw words it holds
  const auto decode = [&](uint8_t* dec) {
    const int tt = opaque_tid();
    uint4 va, vb;
    uint2 code[kItemsPer];
    if (items.wide) key_lookups<true>(smem, items, raw.k, code);
    else key_lookups<false>(smem, items, raw.k, code);
    value_lookups<BV>(smem, raw, quarter, va, vb);
    uint8_t* dst = dec + (tt & 63) * (2 * kKStride) + 8 * wave;
#pragma unroll
    for (int j = 0; j < kItemsPer; ++j) key_store(dst + 8 * kAttnWaves * j, items, j, raw.kn, code[j]);
    store_values<BV>(dec, raw, tt, quarter, va, vb);
  };

  float16_t s[NB];  // S^T of the wave's token blocks
  // S^T = K Q^T of the tile in dcur, three passes: hi hi, lo_k hi_q, hi_k
  // lo_q.  One step = 16 coordinates of one token block; its operands are read
  // two steps ahead (sched_barrier: left alone, the compiler reads an operand
  // right before its product and waits out the LDS latency).
  const auto products_qk = [&](const uint8_t* dcur) {
    const int tt = opaque_tid();
    const uint8_t* kb = dcur + (32 * blk0 + (tt & 31)) * (2 * kKStride) + ((tt & 32) >> 1);
    half8_t ka[3][2];
    const auto read_keys = [&](int u) {  // step u: coordinates 16 (u / NB) .. of block u % NB
      const uint8_t* at = kb + u % NB * 32 * 2 * kKStride + 32 * (u / NB);
      ka[u % 3][0] = *reinterpret_cast<const half8_t*>(at + kDecKH);
      ka[u % 3][1] = *reinterpret_cast<const half8_t*>(at + kDecKL);
    };
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[n][i] = 0.f;
    read_keys(0);
    read_keys(1);
#pragma unroll
    for (int u = 0; u < 8 * NB; ++u) {
      if (u + 2 < 8 * NB) read_keys(u + 2);
      __builtin_amdgcn_sched_barrier(0);
      const int n = u % NB, ks = u / NB;
      s[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka[u % 3][0], qh[ks], s[n], 0, 0, 0);
      s[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka[u % 3][1], qh[ks], s[n], 0, 0, 0);
      s[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka[u % 3][0], ql[ks], s[n], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Causal mask and online softmax (base 2) of tile kt, then O^T += V^T P^T.
  // The mask is applied only where a token of the wave's blocks can lie past a
  // row of the wave.  A tile that raises no running maximum of the wave (one
  // vote) skips the cross-lane maximum and the rescale, which changes no
  // result.
  const auto softmax_pv = [&](const uint8_t* dcur, int t0) {
    const int tt = opaque_tid(), hf4 = (tt & 32) >> 3;  // 4 hf
    if (t0 + 32 * (blk0 + NB) - 1 > pos_min) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int tok = t0 + 32 * (blk0 + n) + 8 * (i >> 2) + hf4 + (i & 3);
          s[n][i] = tok > pos ? kNegInf : s[n][i];
        }
    }
    uint2 vr[4];  // value radii of the lane's tokens of one block
    const auto read_radii = [&](int n) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        vr[q] = *reinterpret_cast<const uint2*>(dcur + kDecVN + 2 * (32 * (blk0 + n) + 8 * q + hf4));
    };
    // (four chains: one chain of dependent maxima would wait out their latency)
    float mp[4];
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
      mp[c4] = fmaxf(s[0][4 * c4], s[0][4 * c4 + 1]);
      mp[c4] = fmaxf(fmaxf(mp[c4], s[0][4 * c4 + 2]), s[0][4 * c4 + 3]);
      if constexpr (NB == 2) {
        mp[c4] = fmaxf(fmaxf(mp[c4], s[1][4 * c4]), s[1][4 * c4 + 1]);
        mp[c4] = fmaxf(fmaxf(mp[c4], s[1][4 * c4 + 2]), s[1][4 * c4 + 3]);
      }
    }
    const float mx = fmaxf(fmaxf(mp[0], mp[1]), fmaxf(mp[2], mp[3]));
    if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
      const float mn = fmaxf(m_run, max2g(mx));
      // (m_run stays -inf only while every token so far is masked)
      const float corr = m_run == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m_run - mn);
      m_run = mn;
      l_run *= corr;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) o[cc] *= corr;
    }
    const float mref = m_run == kNegInf ? 0.f : m_run;
    // exp2 is the hardware instruction: its arguments are <= 0 here and a
    // result below the normal range (flushed to 0) is negligible
    float ps = 0.f;
    half8_t pb[NB][2];
    const auto weights = [&](int n) {
      uint32_t pw[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[i] = __builtin_amdgcn_exp2f(s[n][4 * q + i] - mref);
        }
        ps += (p[0] + p[1]) + (p[2] + p[3]);
        pw[2 * q] = mix_pair(p[0], p[1], vr[q].x);
        pw[2 * q + 1] = mix_pair(p[2], p[3], vr[q].y);
      }
      pb[n][0] = __builtin_bit_cast(half8_t, make_uint4(pw[0], pw[1], pw[2], pw[3]));
      pb[n][1] = __builtin_bit_cast(half8_t, make_uint4(pw[4], pw[5], pw[6], pw[7]));
    };
    // 16 tokens and 4 dim blocks at a time; the operands of a step are read
    // one step ahead, and the second block's exponentials run beside the
    // first one's products
    const uint8_t* vb = dcur + kDecV + (tt & 31) * (2 * kVStride) + 64 * blk0 + 4 * hf4;
    half8_t va[2][4];
    const auto read_values = [&](int st16) {
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
        va[st16 & 1][cc] = *reinterpret_cast<const half8_t*>(vb + 32 * cc * (2 * kVStride) + 32 * st16);
    };
    read_radii(0);
    read_values(0);
    __builtin_amdgcn_sched_barrier(0);
    weights(0);
#pragma unroll
    for (int st16 = 0; st16 < 2 * NB; ++st16) {
      if (NB == 2 && st16 == 0) read_radii(1);
      if (st16 + 1 < 2 * NB) read_values(st16 + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
        o[cc] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[st16 & 1][cc], pb[st16 >> 1][st16 & 1], o[cc], 0, 0, 0);
      if (NB == 2 && st16 == 0) weights(1);
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run += ps;
  };

  // Pipeline: tile kt's products run on decoded buffer kt % 2 while the same
  // waves decode tile kt + 1 (its raw words are in registers) into the other
  // buffer and load tile kt + 2's raw words.  Waves 0-3 decode before their
  // products and waves 4-7 after them, so that of a SIMD's two waves one has
  // matrix work while the other decodes.  One barrier per tile separates a
  // buffer's writes from its reads on either side.  After the last tile the
  // waves decode stale words into a buffer that nobody reads and load the last
  // tile again.
  const auto tile_start = [&](int kt) { return min(kt, n_kt - 1) * kKeyTile; };
  load_raw(0);
  __syncthreads();
  decode(smem + kOffDec);
  load_raw(tile_start(1));
  __syncthreads();
  // Waves 4-7 take the SIMD's issue slots first, throughout: with equal
  // priorities (or a higher one for the product phases of both) the two waves
  // of a SIMD share the matrix core and reach their softmax together, leaving
  // it idle (17.4 -> 16.2 ms on a 32K-token Llama-shaped layer).
  if (wave >= 4) __builtin_amdgcn_s_setprio(2);
  for (int kt = 0; kt < n_kt; ++kt) {
    const uint8_t* const dcur = smem + kOffDec + (kt & 1) * kDecBytes;
    uint8_t* const dnxt = smem + kOffDec + (~kt & 1) * kDecBytes;
    if (wave < 4) {
      decode(dnxt);
      load_raw(tile_start(kt + 2));
    }
    products_qk(dcur);
    softmax_pv(dcur, kt * kKeyTile);
    if (wave >= 4) {
      decode(dnxt);
      load_raw(tile_start(kt + 2));
    }
    __syncthreads();
  }

  // ---- KS = 2: waves 4-7 hand their states over to waves 0-3
  l_run = sum2g(l_run);
  if constexpr (KS == 2) {
    float* mg = reinterpret_cast<float*>(smem) + (wave & 3) * 66 * 64 + lane;
    if (wave >= 4) {
      mg[0] = m_run;
      mg[64] = l_run;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int i = 0; i < 16; ++i) mg[64 * (2 + 16 * cc + i)] = o[cc][i];
    }
    __syncthreads();
    if (wave < 4) {
      const float m2 = mg[0], l2 = mg[64], mn = fmaxf(m_run, m2);
      const float e1 = m_run == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m_run - mn);
      const float e2 = m2 == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m2 - mn);
      l_run = l_run * e1 + l2 * e2;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cc][i] = o[cc][i] * e1 + mg[64 * (2 + 16 * cc + i)] * e2;
    }
    __syncthreads();
  }

  // ---- epilogue: o / (l sqrt(d_h)), then out = Pi_V^T o (fp32 MFMAs over Pi_V staged in LDS)
  {
    // the codes' 1/sqrt(d_h) (value radius n_V over sqrt(d_h) times a unit-variance centroid)
    const float inv = l_run > 0.f ? 0.08838834764831845f / l_run : 0.f;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) o[cc] *= inv;
  }
  float* rv = reinterpret_cast<float*>(smem);
  {
    const float4* src = reinterpret_cast<const float4*>(blob + kOffRotV);
    for (int i = tid; i < kHeadDim * kHeadDim / 4; i += kAttnThreads) reinterpret_cast<float4*>(rv)[i] = src[i];
  }
  __syncthreads();
  if (KS == 2 && wave >= 4) return;
#pragma unroll 1
  for (int c2 = 0; c2 < 4; ++c2) {
    float16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        // A[d'][k = hf] = Pi_V[32 cc + 8 (i / 4) + 4 hf + i % 4][d'], B[k][row] = o[cc][i]
        const float a = rv[(32 * cc + 8 * (i >> 2) + 4 * hf + (i & 3)) * kHeadDim + 32 * c2 + l32];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, o[cc][i], acc, 0, 0, 0);
      }
    if (ri < n_q) {
      float* dst = out + ((static_cast<size_t>(seq) * n_q + ri) * hq + kvh * G + rh) * kHeadDim + 32 * c2 + 4 * hf;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(dst + 8 * q) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    }
  }
}

template <int BV>
hipError_t launch_attn(const Dims& d, const uint8_t* blob, const float* qr, int n_q, const int32_t* q_pos0,
                       int max_pos, const CachePtrs& c, float* out, hipStream_t s) {
  const long nr = static_cast<long>(n_q) * d.group;
  const auto go = [&](auto kern, int rows) {
    hipLaunchKernelGGL(kern, dim3((nr + rows - 1) / rows, d.n_kv, d.batch), dim3(kAttnThreads), 0, s, d, blob, qr,
                       n_q, q_pos0, max_pos, c, out);
  };
  // 128-row workgroups while they all fit the 256 CUs at once: half the rows
  // take half the time per tile (1001 positions x 8 heads x 2 KV heads after
  // 15003 rows: 0.46 against 0.70 ms).  Above that every tile would be decoded
  // twice as often for the same products (2048 positions x 4 heads x 8 KV
  // heads: 0.19 against 0.15 ms with 256 rows; 32768 positions: 17.2 against
  // 14.7 ms).
  constexpr int rows1 = kAttnWaves * kWaveRows, rows2 = rows1 / 2;
  if ((nr + rows2 - 1) / rows2 * d.n_kv * d.batch <= 256) go(k_prefill_attn<BV, 2>, rows2);
  else go(k_prefill_attn<BV, 1>, rows1);
  return hipGetLastError();
}

}  // namespace prefill_detail

hipError_t launch_prefill_attn(const Dims& d, const void* layout, const void* q, int n_q,
                               const int32_t* q_pos0, int max_pos, const CachePtrs& c, float* qr_ws,
                               float* out, hipStream_t s) {
  using namespace prefill_detail;
  const uint8_t* blob = static_cast<const uint8_t*>(layout);
  const int nr = n_q * d.group;
  const bool aligned = (reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(qr_ws)) % 16 == 0;
  if (d.in_dtype == 1 && aligned) {
    const long rows = static_cast<long>(nr) * d.n_kv * d.batch;
    const auto go = [&](auto kern, int w, int iters) {
      const int per = w * split::kSplitRows * iters;
      hipLaunchKernelGGL(kern, dim3((nr + per - 1) / per, d.n_kv, d.batch), dim3(w * 64), 0, s, d, blob, q, n_q, iters,
                         qr_ws);
    };
    // 4-wave workgroups up to 64K rows, where 16-wave ones would leave CUs
    // idle; above, 16 waves share one staging of the matrix, and above 512K rows
    // four passes of the workgroup do.  us of the rotation with 4 waves / 16
    // waves / 16 waves and four passes: 16K rows 11 / 16 / 44, 32K 16 / 19 / 48,
    // 64K 22 / 18 / 45, 96K 28 / 18 / 45, 512K 171 / 106 / 90, 640K 198 / 119 /
    // 159, 1M 308 / 212 / 172 (the true crossings lie near 48K and, by whole
    // rounds of workgroups, between 256K and 1M rows).
    if (rows <= 256L * 256) go(k_prefill_qrot_bf16<4>, 4, 1);
    else go(k_prefill_qrot_bf16<16>, 16, rows <= 4L * 256 * 512 ? 1 : 4);
  } else {
    const dim3 g1((nr + kQrotRows - 1) / kQrotRows, d.n_kv, d.batch);
    hipLaunchKernelGGL(k_prefill_qrot, g1, dim3(kThreads), 0, s, d, blob, q, n_q, qr_ws);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (d.v_bits) {
    case 1: return launch_attn<1>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 2: return launch_attn<2>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 3: return launch_attn<3>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 4: return launch_attn<4>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 5: return launch_attn<5>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 6: return launch_attn<6>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    case 7: return launch_attn<7>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
    default: return launch_attn<8>(d, blob, qr_ws, n_q, q_pos0, max_pos, c, out, s);
  }
}

}  // namespace bgtq
