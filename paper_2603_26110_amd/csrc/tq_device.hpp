// Device-side building blocks shared by the quantize and decode kernels.
//
// Cache layout (64-slot tiles, 2048 bytes per tile per tensor):
//   K tile, token-major: 16-byte half c (codes 32c..32c+31) of slot-in-tile r
//        at byte (c*64 + r)*16. One lane per token loads its 32 bytes with two
//        128-bit loads; each wave-wide load covers 1 KiB contiguously. Key word
//        w holds dimensions 8w..8w+7: 3-bit index of dimension 8w+j in bits
//        3j..3j+2, its QJL sign bit in bit 24+j.
//   V tile, dimension-major: 16-byte half c (slots 32c..32c+31) of dimension i
//        at byte (c*64 + i)*16. One lane per dimension loads the 64 codes of its
//        dimension for the whole tile with two 128-bit loads. A value nibble is
//        idx | sign << 3; nibble j of a 32-bit word sits at bits 4j..4j+3.
//   Scalars: 4 x fp16 per slot [n_k, g_k, n_v, g_v] at byte slot*8.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace tq {

constexpr int kDim = 64;
constexpr int kTile = 64;
constexpr int kTileBytes = 2048;   // 64 slots x 32 bytes
constexpr int kPairs = 32;
constexpr int kXcds = 8;           // blocks go to the 8 XCDs round-robin

// Flags (values fixed by the public header).
constexpr uint32_t kVRotate = 1u << 0;
constexpr uint32_t kVQjl = 1u << 1;
constexpr uint32_t kQjlPaper = 1u << 2;
constexpr uint32_t kRopeHalf = 1u << 3;
constexpr uint32_t kInputRotated = 1u << 4;
constexpr uint32_t kOutF32 = 1u << 5;

// sqrt(pi/2) / m with m = 64 projection rows (QJL estimator scale).
constexpr float kQjlAlpha = 0.019583033395554691f;

__device__ __forceinline__ float load_in(const void* p, int64_t i, bool f16) {
  if (f16) return __half2float(reinterpret_cast<const __half*>(p)[i]);
  return reinterpret_cast<const float*>(p)[i];
}

// Norms are stored as fp16 with round-to-nearest-even, saturated at 65504.
__device__ __forceinline__ uint32_t store_norm(float x) {
  x = (x > 65504.0f) ? 65504.0f : x;
  return (uint32_t)__half_as_ushort(__float2half_rn(x));
}

__device__ __forceinline__ float half_bits_to_float(uint32_t bits) {
  return __half2float(__ushort_as_half((unsigned short)(bits & 0xFFFFu)));
}

// Key word of dimensions 8w..8w+7: 3-bit index of dimension 8w+j in bits
// 3j..3j+2, its QJL sign bit in bit 24+j. Value words hold eight 4-bit
// nibbles idx | sign << 3.
__device__ __forceinline__ uint32_t key_code_bits(uint32_t idx, uint32_t sign, int j) {
  return (idx << (3 * j)) | (sign << (24 + j));
}

// Byte offset of 16-byte half c of row r (slot for K, dimension for V) in a tile.
__device__ __forceinline__ int64_t tile_half_offset(int64_t tile, int c, int r) {
  return tile * kTileBytes + (int64_t)(c * kTile + r) * 16;
}

// Fixed-order binary32 steps of the quantizer for one vector held in registers
// (this file is compiled with -ffp-contract=off and correctly rounded sqrtf and
// division, the HIP defaults; fmaf is the only fused operation)
// by one lane: the norm and residual-norm fma chains run over i ascending, so
// any kernel that calls this on the same x^ produces the same bits.
//   xh[64]   rotated vector over `scale` (overwritten by the residual r)
//   scale    a power of two, which no rounding of these steps depends on
//   thr, lev the table's midpoints {t0, t2, t4, t6, t1, t3, t5} and its levels,
//            in LDS
//   words[8] out: index of dimension 8w+j in bits width*j of word w
// The eight levels and seven midpoints of one table as named register values.
// Named members (no arrays) keep the level choice a chain of selects between
// registers; an array indexed inside a loop gets folded into an indexed load
// from private memory, which the compiler then spills to LDS or scratch.
struct Levels {
  float c0, c1, c2, c3, c4, c5, c6, c7;
  float t0, t1, t2, t3, t4, t5, t6;
};

__device__ __forceinline__ Levels load_levels(const float* lut) {
  Levels L;
  L.c0 = lut[0]; L.c1 = lut[1]; L.c2 = lut[2]; L.c3 = lut[3];
  L.c4 = lut[4]; L.c5 = lut[5]; L.c6 = lut[6]; L.c7 = lut[7];
  L.t0 = 0.5f * (L.c0 + L.c1); L.t1 = 0.5f * (L.c1 + L.c2); L.t2 = 0.5f * (L.c2 + L.c3);
  L.t3 = 0.5f * (L.c3 + L.c4); L.t4 = 0.5f * (L.c4 + L.c5); L.t5 = 0.5f * (L.c5 + L.c6);
  L.t6 = 0.5f * (L.c6 + L.c7);
  return L;
}

// Strictly ascending levels (false for any NaN level). Kernels skip a
// (layer, head) whose table fails this: the midpoint rule assumes it.
__device__ __forceinline__ bool levels_ascending(const Levels& L) {
  return (L.c0 < L.c1) & (L.c1 < L.c2) & (L.c2 < L.c3) & (L.c3 < L.c4) & (L.c4 < L.c5) &
         (L.c5 < L.c6) & (L.c6 < L.c7);
}

// Nearest level of u by the midpoints (ties go to the lower level): returns
// the level, its index in *idx.
// The levels are passed as separate values, which callers pin in registers
// once (TQ_PIN_LEVELS): the selects then pick between register values, where a
// select between two loads of a table would become one load at a computed
// offset, from private memory.
#define TQ_PIN_LEVELS(L)                                                                  \
  float L##_0 = L.c0, L##_1 = L.c1, L##_2 = L.c2, L##_3 = L.c3, L##_4 = L.c4, L##_5 = L.c5, \
        L##_6 = L.c6, L##_7 = L.c7;                                                       \
  asm volatile("" : "+v"(L##_0), "+v"(L##_1), "+v"(L##_2), "+v"(L##_3), "+v"(L##_4),     \
               "+v"(L##_5), "+v"(L##_6), "+v"(L##_7))
#define TQ_LEVELS(L) L, L##_0, L##_1, L##_2, L##_3, L##_4, L##_5, L##_6, L##_7

__device__ __forceinline__ float nearest_level(float u, const Levels& L, float c0, float c1,
                                               float c2, float c3, float c4, float c5, float c6,
                                               float c7, uint32_t* idx) {
  uint32_t i = 0;
  float lv = c0;
  bool a;
  a = u > L.t0; i += a ? 1u : 0u; lv = a ? c1 : lv;
  a = u > L.t1; i += a ? 1u : 0u; lv = a ? c2 : lv;
  a = u > L.t2; i += a ? 1u : 0u; lv = a ? c3 : lv;
  a = u > L.t3; i += a ? 1u : 0u; lv = a ? c4 : lv;
  a = u > L.t4; i += a ? 1u : 0u; lv = a ? c5 : lv;
  a = u > L.t5; i += a ? 1u : 0u; lv = a ? c6 : lv;
  a = u > L.t6; i += a ? 1u : 0u; lv = a ? c7 : lv;
  *idx = i;
  return lv;
}

// The index alone, #{m : u > t_m} (the same count as nearest_level's), of four
// values at a time, for a caller that reads the level itself from a table in
// LDS. The comparisons write three scalar register pairs and VCC, and each is
// used at once, so no lane mask stays live across the elements of a vector (64
// unrolled select chains keep so many masks live that they spill).
// The count is the length of the prefix of thresholds below u (they are
// non-decreasing), found in three steps: b2 = [t3 < u], b1 =
// [t(b2 ? 5 : 1) < u] and b0 = [t(4 b2 + 2 b1) < u], each bit added into
// the count by a carry (a NaN u compares false throughout, like the
// count). The second threshold is selected in registers (t1 and t5 as
// vector operands: a select that reads a mask cannot also read a scalar);
// the third, t(2 i) for i = 2 b2 + b1, is read from {t0, t2, t4, t6} in LDS.
// levels_half gives i, levels_full the counts from i and those thresholds.
// (A vector instruction may read a mask that another wrote only after two wait
// states, which the compiler does not see here: the four values take turns.)
__device__ __forceinline__ void levels_half(uint32_t* i, const float* u, float t1, float t3, float t5) {
  float a0, a1, a2, a3;
  uint64_t m0, m1, m2;
  asm("v_cmp_lt_f32_e64 %8, %12, %14\n\t"
      "v_cmp_lt_f32_e64 %9, %12, %15\n\t"
      "v_cmp_lt_f32_e64 %10, %12, %16\n\t"
      "v_cmp_lt_f32 vcc, %12, %17\n\t"
      "v_cndmask_b32_e64 %0, 0, 1, %8\n\t"
      "v_cndmask_b32_e64 %4, %11, %13, %8\n\t"
      "v_cndmask_b32_e64 %1, 0, 1, %9\n\t"
      "v_cndmask_b32_e64 %5, %11, %13, %9\n\t"
      "v_cndmask_b32_e64 %2, 0, 1, %10\n\t"
      "v_cndmask_b32_e64 %6, %11, %13, %10\n\t"
      "v_cndmask_b32_e64 %3, 0, 1, vcc\n\t"
      "v_cndmask_b32 %7, %11, %13, vcc\n\t"
      "v_cmp_lt_f32_e64 %8, %4, %14\n\t"
      "v_cmp_lt_f32_e64 %9, %5, %15\n\t"
      "v_cmp_lt_f32_e64 %10, %6, %16\n\t"
      "v_cmp_lt_f32 vcc, %7, %17\n\t"
      "v_addc_co_u32_e64 %0, %8, %0, %0, %8\n\t"
      "v_addc_co_u32_e64 %1, %9, %1, %1, %9\n\t"
      "v_addc_co_u32_e64 %2, %10, %2, %2, %10\n\t"
      "v_addc_co_u32 %3, vcc, %3, %3, vcc"
      : "=&v"(i[0]), "=&v"(i[1]), "=&v"(i[2]), "=&v"(i[3]), "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3), "=&s"(m0),
        "=&s"(m1), "=&s"(m2)
      : "v"(t1), "v"(t3), "v"(t5), "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3])
      : "vcc");
}

__device__ __forceinline__ void levels_full(uint32_t* i, const float* u, const float* tb) {
  uint64_t m0, m1, m2;
  asm("v_cmp_lt_f32_e64 %4, %7, %11\n\t"
      "v_cmp_lt_f32_e64 %5, %8, %12\n\t"
      "v_cmp_lt_f32_e64 %6, %9, %13\n\t"
      "v_cmp_lt_f32 vcc, %10, %14\n\t"
      "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"
      "v_addc_co_u32_e64 %1, %5, %1, %1, %5\n\t"
      "v_addc_co_u32_e64 %2, %6, %2, %2, %6\n\t"
      "v_addc_co_u32 %3, vcc, %3, %3, vcc"
      : "+v"(i[0]), "+v"(i[1]), "+v"(i[2]), "+v"(i[3]), "=&s"(m0), "=&s"(m1), "=&s"(m2)
      : "v"(tb[0]), "v"(tb[1]), "v"(tb[2]), "v"(tb[3]), "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3])
      : "vcc");
}

// Sixteen values loaded before any of them is used: the wave waits for its
// LDS reads once per sixteen.
__device__ __forceinline__ void arrive16(float (&v)[16]) {
  asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]),
               "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]), "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15]));
}

struct QuantOut {
  uint32_t n16, g16;
  float g;                 // ||r|| in binary32 (before the fp16 store)
};

__device__ __forceinline__ QuantOut quantize_lane(float (&xh)[kDim], float scale, const float* thr, const float* lev,
                                                  uint32_t width, uint32_t (&words)[8]) {
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < kDim; ++i) s = fmaf(xh[i], xh[i], s);
  const float n = sqrtf(s);
  const float inv = (n == 0.0f) ? 0.0f : 8.0f / n;
  const float t1 = thr[4], t3 = thr[5], t5 = thr[6];
#pragma unroll
  for (int i0 = 0; i0 < kDim; i0 += 16) {
    uint32_t idx[16];
    float rd[16];
#pragma unroll
    for (int j = 0; j < 16; j += 4) {
#pragma unroll
      for (int e = j; e < j + 4; ++e) xh[i0 + e] *= inv;   // u_i
      levels_half(&idx[j], &xh[i0 + j], t1, t3, t5);
#pragma unroll
      for (int e = j; e < j + 4; ++e) rd[e] = thr[idx[e]];
    }
    arrive16(rd);
#pragma unroll
    for (int j = 0; j < 16; j += 4) {
      levels_full(&idx[j], &xh[i0 + j], &rd[j]);
#pragma unroll
      for (int e = j; e < j + 4; ++e) rd[e] = lev[idx[e]];   // the level c[idx]
    }
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      uint32_t word = idx[8 * w + 7];
#pragma unroll
      for (int j = 6; j >= 0; --j) word = (word << width) | idx[8 * w + j];
      asm volatile("" : "+v"(word));   // (packed here: a later place would keep all indices live)
      words[(i0 >> 3) + w] = word;
    }
    arrive16(rd);
#pragma unroll
    for (int j = 0; j < 16; ++j) xh[i0 + j] -= rd[j];   // residual r_i
  }
  float gs = 0.0f;
#pragma unroll
  for (int i = 0; i < kDim; ++i) gs = fmaf(xh[i], xh[i], gs);
  const float g = sqrtf(gs);
  QuantOut o;
  o.n16 = store_norm(n * scale);
  o.g16 = store_norm(g);
  o.g = g;
  return o;
}

// The 64 lanes' values of a wave, for sums that every lane forms over all of
// them (decode: a tile's token weights; appends: a vector's elements). Lane t
// holds w_t; two lane swaps give four registers R_j holding lanes
// 16j .. 16j+15 in every 16-lane row (v_permlane32_swap exchanges the upper
// half of one register with the lower half of another, v_permlane16_swap the
// odd rows of one with the even rows of another). An FMA then reads w_{16j+k}
// through a DPP row broadcast of lane k (row_newbcast), so no value costs an
// instruction of its own. (A DPP read needs two wait states after the vector
// instruction that wrote the register, which the compiler does not see here.)
struct LaneSpread {
  float r[4];
};

__device__ __forceinline__ LaneSpread spread_lanes(float w) {
  const int wi = __float_as_int(w);
  const auto h = __builtin_amdgcn_permlane32_swap(wi, wi, false, false);   // rows 0 1 0 1 | 2 3 2 3
  const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);   // 0 0 0 0 | 1 1 1 1
  const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);   // 2 2 2 2 | 3 3 3 3
  LaneSpread tw;
  tw.r[0] = __int_as_float(lo[0]);
  tw.r[1] = __int_as_float(lo[1]);
  tw.r[2] = __int_as_float(hi[0]);
  tw.r[3] = __int_as_float(hi[1]);
  return tw;
}

// acc += w_{16j+K} * c, the weight taken from register R_j by a row broadcast.
template <int K>
__device__ __forceinline__ void fma_row_bcast(float& acc, float rj, float c) {
  asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
      : "+v"(acc) : "v"(rj), "v"(c), "i"(K));
}

// Wave-wide reductions (64 lanes).
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace tq
