// Prefill-side quantizer: RoPE -> Pi rotation -> per-vector norm -> 3-bit
// table codes -> residual -> QJL sign bits -> packed cache (TurboESM Sec. 3.1
// prefill steps 1, 3, 4; Sec. 3.3; Sec. 3.4; Sec. 4.2).
//
// Three kernels:
//   quantize_tiles_kernel   for prefill-sized T: the keys and values of 32
//                           tokens per wave; the rotations x^ = Pi x' of
//                           these 64 vectors and the projections S r run on
//                           the matrix cores (fp16 MFMA on hi/lo parts), one
//                           lane per vector runs the quantizer steps.
//   quantize_batch_kernel   many short sequences: a wave takes four vectors at a
//                           time, one lane per dimension, and a block's waves
//                           share the staged Pi and S.
//   quantize_vectors_kernel one wave per vector (one lane per dimension; the
//                           key and the value of a token-head in parallel), for
//                           decode-step appends with small T; its rotation is
//                           an fma chain over k ascending.
// All run the quantizer steps (norm, levels, residual, projected signs) in
// the fixed binary32 order of quantize_lane / quantize_wave, so identical x^
// give identical bits; for raw inputs the prefill's rotation sums in another
// order than the other two's, so a code can differ where x^ sits within rounding of a threshold.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "tq_append.hpp"
#include "tq_device.hpp"
#include "tq_internal.hpp"

namespace tq {

// ---------------------------------------------------------------- RoPE table
// cs[p][m] = (cos, sin)(p * base^(-2m/64)), fp64 before rounding (Eq. 2).
__global__ void rope_table_kernel(float* cs, int positions, double base) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)positions * kPairs) return;
  const int p = (int)(e / kPairs), m = (int)(e % kPairs);
  const double theta = pow(base, -2.0 * m / (double)kDim);
  const double ang = (double)p * theta;
  cs[2 * e + 0] = (float)cos(ang);
  cs[2 * e + 1] = (float)sin(ang);
}

hipError_t launch_rope_table(float* cs, int positions, double base, hipStream_t st) {
  const int64_t n = (int64_t)positions * kPairs;
  const int threads = 256;
  const int blocks = (int)((n + threads - 1) / threads);
  hipLaunchKernelGGL(rope_table_kernel, dim3(blocks), dim3(threads), 0, st, cs, positions, base);
  return hipGetLastError();
}

// ------------------------------------------- matrix-core products of 64 rows
// Two dense 64 x 64 x 64 products per wave run on the matrix cores: the
// rotation x^ = Pi x' of the keys and values of the wave's 32 tokens and the
// QJL projection S r of their residuals. Both use v_mfma_f32_32x32x16_f16
// (fp16 inputs, fp32 sums) with each fp32 operand split into fp16 parts
// hi = fp16(v), lo = fp16(v - hi) and three products hi*hi + hi*lo + lo*hi,
// which carries a product to about 2^-21 relative. Each vector is first scaled
// by a power of two (exact) so that its largest entry lies in [1, 2), and each
// row of S to norm 8 (the split takes the exact product), which keeps the parts
// in fp16's range. Values in fp16 are their own high part: they are neither
// scaled nor split, and have no low part.
// Instruction layout (lane l, n = l % 32, h = l / 32; verified on gfx950):
//   A lane values A[n][8h + j], B lane values B[8h + j][n] (j = 0..7),
//   D register r D[8 (r/4) + 4h + r%4][n].
// Block 0 of the B operand (nb = 0) holds the 32 keys and block 1 the 32
// values. Step q (0..3) contracts k = 16q + 8h + j: a lane's B values at step
// q are 8 consecutive dimensions of its token (one 16-byte load of fp16 input)
// and its A values 8 consecutive columns of a row of the staged matrix (one
// 16-byte LDS read per part). The result leaves lane half h the dimensions
// {8q + 4h + j, j < 4} of key n and of value n; one v_permlane32_swap per
// register pair then hands lane l < 32 all 64 values of key l and lane l >= 32
// those of value l - 32.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kGroup = 32;                   // tokens per wave
constexpr float kSignBand = 0x1p-15f;        // projected_signs' guard band

// 16-byte chunk c (columns 8c .. 8c + 7) of row r of a staged 64 x 64 matrix
// of fp16 lies at chunk position c ^ (r / 2 % 8) of its row: the 16 rows read
// together fall on all 64 banks once, without padding.
__device__ __forceinline__ int staged_at(int r, int c) { return r * kDim + ((c ^ ((r >> 1) & 7)) << 3); }

// Blocks of a pair of products: D[mb][nb], rows 32 mb .. and vectors of block nb.
typedef f32x16 Blocks[2][2];

// hi = fp16(v sc), lo = fp16(v sc - hi), sc a power of two (v sc exact): one
// mixed-precision fma each, as pairs in one register. (The s_nop: a matrix
// instruction may not read a register in the two wait states after a vector
// instruction wrote it, and the compiler does not look into the block.)
__device__ __forceinline__ void split8(const float* v, float sc, half8& hi, half8& lo) {
  uint32_t h[4], l[4];
  asm("v_fma_mixlo_f16 %0, %8, %16, 0\n\t"
      "v_fma_mixlo_f16 %1, %10, %16, 0\n\t"
      "v_fma_mixlo_f16 %2, %12, %16, 0\n\t"
      "v_fma_mixlo_f16 %3, %14, %16, 0\n\t"
      "v_fma_mixhi_f16 %0, %9, %16, 0\n\t"
      "v_fma_mixhi_f16 %1, %11, %16, 0\n\t"
      "v_fma_mixhi_f16 %2, %13, %16, 0\n\t"
      "v_fma_mixhi_f16 %3, %15, %16, 0\n\t"
      "v_fma_mixlo_f16 %4, %8, %16, -%0 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixlo_f16 %5, %10, %16, -%1 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixlo_f16 %6, %12, %16, -%2 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixlo_f16 %7, %14, %16, -%3 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %4, %9, %16, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %5, %11, %16, -%1 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %6, %13, %16, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %7, %15, %16, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "s_nop 1"
      : "=&v"(h[0]), "=&v"(h[1]), "=&v"(h[2]), "=&v"(h[3]), "=&v"(l[0]), "=&v"(l[1]), "=&v"(l[2]), "=&v"(l[3])
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(sc));
  hi = __builtin_bit_cast(half8, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(half8, make_uint4(l[0], l[1], l[2], l[3]));
}

// 2^(1 - e) for m = f 2^e, f in [0.5, 1): m times it lies in [1, 2); 1 for m = 0.
// At most 2^126, so that it and its reciprocal are normal numbers: a subnormal
// m then lands below 1, in multiples of 2^-23, which two fp16 parts hold
// exactly.
__device__ __forceinline__ float unit_scale(float m) {
  const float s = ldexpf(1.0f, min(1 - __builtin_amdgcn_frexp_expf(m), 126));
  return m > 0.0f ? s : 1.0f;
}

// Step Q of acc[mb] (+)= rows 32 mb .. of the matrix (parts mh, ml) times block
// 0 (b0h, b0l) and, with TWO, block 1 (b1h and, with LO1, b1l); step 0 starts
// from zero. The blocks take turns, so that a product does not wait for the
// one before it.
template <int Q, bool TWO, bool LO1>
__device__ __forceinline__ void product_step(Blocks& acc, int mb, const _Float16* mh, const _Float16* ml, int lane,
                                             half8 b0h, half8 b0l, half8 b1h, half8 b1l) {
  int o = staged_at(lane & 31, 2 * Q + (lane >> 5));
  asm volatile("" : "+v"(o));
  // (rows 32 apart have the same chunk order)
  const half8 ah = *reinterpret_cast<const half8*>(mh + o + 32 * mb * kDim);
  const half8 al = *reinterpret_cast<const half8*>(ml + o + 32 * mb * kDim);
  const f32x16 zero = {};
  acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b0h, Q == 0 ? zero : acc[mb][0], 0, 0, 0);
  if (TWO) acc[mb][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b1h, Q == 0 ? zero : acc[mb][1], 0, 0, 0);
  acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b0l, acc[mb][0], 0, 0, 0);
  if (TWO && LO1) acc[mb][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b1l, acc[mb][1], 0, 0, 0);
  acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, b0h, acc[mb][0], 0, 0, 0);
  if (TWO) acc[mb][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, b1h, acc[mb][1], 0, 0, 0);
}

// f(Q) for Q = 0 .. 3 as compile-time constants.
template <class F>
__device__ __forceinline__ void four_steps(F f) {
  f(std::integral_constant<int, 0>{});
  f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{});
  f(std::integral_constant<int, 3>{});
}

// D blocks -> lane l holds all 64 rows of its vector (key l, or value l - 32).
__device__ __forceinline__ void to_lane_per_vector(Blocks& acc, float (&out)[kDim]) {
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[mb][0][r]),
                                                       __float_as_uint(acc[mb][1][r]), false, false);
      const int d = 32 * mb + 8 * (r >> 2) + (r & 3);
      out[d] = __uint_as_float(sw[0]);       // row set of lane half 0
      out[d + 4] = __uint_as_float(sw[1]);   // row set of lane half 1
    }
}

// A lane's part of key and value j0 + n as loaded (dimensions 16q + 8h + j),
// and the key's RoPE (cos, sin).
template <bool F16>
struct RawRows {
  uint4 k[F16 ? 4 : 8], v[F16 ? 4 : 8];
  float4 cs[8];
};

// A token past the sequence's end or with a position outside the table is
// loaded at the nearest valid one (its result is not stored), so that no load
// waits for a branch.
template <bool F16>
__device__ __forceinline__ void load_rows(RawRows<F16>& raw, const QuantArgs& a, int64_t row, int pos, int lane) {
  const int hh = lane >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (F16) {
      raw.k[q] = *reinterpret_cast<const uint4*>(reinterpret_cast<const __half*>(a.k) + row + 16 * q + 8 * hh);
    } else {
      const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(a.k) + row + 16 * q + 8 * hh);
      raw.k[2 * q] = p[0];
      raw.k[2 * q + 1] = p[1];
    }
  }
  // (cos, sin) of two pairs per float4: pairs 8q + 4h + {0..3} of (2m, 2m + 1),
  // or the angles 16q + 8h + {0..7}, q < 2, of (d, d + 32)
  const bool half = (a.flags & kRopeHalf) != 0;
  const float4* cs4 = reinterpret_cast<const float4*>(a.rope_cs + (int64_t)pos * 2 * kPairs) + (half ? 4 : 2) * hh;
  if (half) {
#pragma unroll
    for (int e = 0; e < 8; ++e) raw.cs[e] = cs4[8 * (e >> 2) + (e & 3)];
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) raw.cs[e] = cs4[4 * (e >> 1) + (e & 1)];
  }
  if (a.flags & kVRotate) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (F16) {
        raw.v[q] = *reinterpret_cast<const uint4*>(reinterpret_cast<const __half*>(a.v) + row + 16 * q + 8 * hh);
      } else {
        const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(a.v) + row + 16 * q + 8 * hh);
        raw.v[2 * q] = p[0];
        raw.v[2 * q + 1] = p[1];
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < (F16 ? 4 : 8); ++q) raw.v[q] = make_uint4(0, 0, 0, 0);
  }
}

template <bool F16>
__device__ __forceinline__ void unpack_rows(float (&xv)[32], const uint4* raw) {
#pragma unroll
  for (int e = 0; e < (F16 ? 4 : 8); ++e) {
    const uint32_t w[4] = {raw[e].x, raw[e].y, raw[e].z, raw[e].w};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      if (F16) {
        xv[8 * e + 2 * p] = half_bits_to_float(w[p]);
        xv[8 * e + 2 * p + 1] = half_bits_to_float(w[p] >> 16);
      } else {
        xv[4 * e + p] = __uint_as_float(w[p]);
      }
    }
  }
}

// x c + y for x the half HI of an fp16 pair; NEG: x c - y.
template <int HI, bool NEG = false>
__device__ __forceinline__ float mix(uint32_t pair, float c, float y) {
  float r;
  if constexpr (HI && NEG)
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(c), "v"(y));
  else if constexpr (HI)
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(c), "v"(y));
  else if constexpr (NEG)
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(c), "v"(y));
  else
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(c), "v"(y));
  return r;
}

// RoPE of a lane's part of a key (both pairings keep a pair inside the lane:
// (2m, 2m + 1) inside a group of 8, (d, d + 32) in groups q and q + 2):
// x'_a = x_a c - x_b s, x'_b = x_a s + x_b c, as fma(x_a, c, -(x_b s)) and
// fma(x_a, s, x_b c). fp16 inputs enter the fmas as they are.
template <bool F16>
__device__ __forceinline__ void rope_rows(float (&xv)[32], const uint4* raw, const float4 (&cs)[8], bool half) {
  if constexpr (F16) {
    uint32_t w[16];                            // pairs of dimensions 2i, 2i + 1 of the lane's 32
#pragma unroll
    for (int q = 0; q < 4; ++q) { w[4 * q] = raw[q].x; w[4 * q + 1] = raw[q].y; w[4 * q + 2] = raw[q].z; w[4 * q + 3] = raw[q].w; }
    if (!half) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float c = (i & 1) ? cs[i >> 1].z : cs[i >> 1].x, s = (i & 1) ? cs[i >> 1].w : cs[i >> 1].y;
        xv[2 * i] = mix<0, true>(w[i], c, mix<1>(w[i], s, 0.0f));
        xv[2 * i + 1] = mix<0>(w[i], s, mix<1>(w[i], c, 0.0f));
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {            // angles of dimensions 2i and 2i + 1
        const float4 c = cs[i];
        xv[2 * i] = mix<0, true>(w[i], c.x, mix<0>(w[8 + i], c.y, 0.0f));
        xv[16 + 2 * i] = mix<0>(w[i], c.y, mix<0>(w[8 + i], c.x, 0.0f));
        xv[2 * i + 1] = mix<1, true>(w[i], c.z, mix<1>(w[8 + i], c.w, 0.0f));
        xv[17 + 2 * i] = mix<1>(w[i], c.w, mix<1>(w[8 + i], c.z, 0.0f));
      }
    }
    return;
  }
  unpack_rows<F16>(xv, raw);
  if (!half) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float4 c = cs[e];
      const float x0 = xv[4 * e], x1 = xv[4 * e + 1], x2 = xv[4 * e + 2], x3 = xv[4 * e + 3];
      xv[4 * e] = fmaf(x0, c.x, -(x1 * c.y)); xv[4 * e + 1] = fmaf(x0, c.y, x1 * c.x);
      xv[4 * e + 2] = fmaf(x2, c.z, -(x3 * c.w)); xv[4 * e + 3] = fmaf(x2, c.w, x3 * c.z);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float4 c = cs[e];
      const float xa = xv[2 * e], xb = xv[16 + 2 * e], ya = xv[2 * e + 1], yb = xv[16 + 2 * e + 1];
      xv[2 * e] = fmaf(xa, c.x, -(xb * c.y)); xv[16 + 2 * e] = fmaf(xa, c.y, xb * c.x);
      xv[2 * e + 1] = fmaf(ya, c.z, -(yb * c.w)); xv[16 + 2 * e + 1] = fmaf(ya, c.w, yb * c.z);
    }
  }
}

// The scale that brings a vector's largest entry into [1, 2).
__device__ __forceinline__ float vector_scale(const float (&xv)[32]) {
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < 32; ++k) m = fmaxf(m, fabsf(xv[k]));
  return unit_scale(fmaxf(m, __shfl_xor(m, 32, 64)));   // (the other 32 entries sit in lane l ^ 32)
}

// x^ of the lane's vector in out[64] (Pi staged as fp16 parts), over the
// returned power of two: the vector's scale, left in, since scaling by a power
// of two changes no rounding of the norm and of u = 8 x^ / n, and taken out
// (1 returned) where some vector's scale is so far from 1 that squares could
// leave fp32's range.
template <bool F16>
__device__ __forceinline__ float rotate_rows(float (&out)[kDim], const RawRows<F16>& raw, const _Float16* pih,
                                             const _Float16* pil, bool half, int lane) {
  half8 kh[4], kl[4], vh[4], vl[4];
  float sk, sv = 1.0f;
  {
    float xv[32];
    rope_rows<F16>(xv, raw.k, raw.cs, half);
    sk = vector_scale(xv);
#pragma unroll
    for (int q = 0; q < 4; ++q) split8(&xv[8 * q], sk, kh[q], kl[q]);
  }
  if constexpr (F16) {
#pragma unroll
    for (int q = 0; q < 4; ++q) vh[q] = __builtin_bit_cast(half8, raw.v[q]);
  } else {
    float xv[32];
    unpack_rows<F16>(xv, raw.v);
    sv = vector_scale(xv);
#pragma unroll
    for (int q = 0; q < 4; ++q) split8(&xv[8 * q], sv, vh[q], vl[q]);
  }
  Blocks acc;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
    four_steps([&](auto q) {
      product_step<q, true, !F16>(acc, mb, pih, pil, lane, kh[q], kl[q], vh[q], F16 ? vh[q] : vl[q]);
    });
  to_lane_per_vector(acc, out);
  const float inv = 1.0f / (lane < 32 ? sk : sv);   // a power of two: exact
  if (__builtin_amdgcn_ballot_w64(!(inv >= 0x1p-40f && inv <= 0x1p40f)) == 0) return inv;
#pragma unroll
  for (int d = 0; d < kDim; ++d) out[d] *= inv;
  return 1.0f;
}

// A vector as it is (pre-rotated inputs, values without TQ_V_ROTATE).
template <bool F16>
__device__ __forceinline__ void load_vector(float (&x)[kDim], const void* src, int64_t row) {
#pragma unroll
  for (int i = 0; i < kDim; i += 8) {
    if (F16) {
      const uint4 w = *reinterpret_cast<const uint4*>(reinterpret_cast<const __half*>(src) + row + i);
      const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        x[i + 2 * p] = half_bits_to_float(ww[p]);
        x[i + 2 * p + 1] = half_bits_to_float(ww[p] >> 16);
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; u += 4) {
        const float4 f = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(src) + row + i + u);
        x[i + u] = f.x; x[i + u + 1] = f.y; x[i + u + 2] = f.z; x[i + u + 3] = f.w;
      }
    }
  }
}

// A load at a wave-uniform address as a scalar load.
template <class T>
__device__ __forceinline__ T scalar_load(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

// (word << 1) | sign of v.
__device__ __forceinline__ uint32_t push_sign(uint32_t word, float v) {
  return __builtin_amdgcn_alignbit(word, __float_as_uint(v), 31);
}

// min(|a|, |b|, m). (Not inline assembly: its operands come from matrix
// instructions, whose latency the compiler waits out only for its own.)
__device__ __forceinline__ float min_abs3(float a, float b, float m) { return fminf(fminf(fabsf(a), fabsf(b)), m); }

// Nibble k of the low 16 bits to the low nibble of byte k.
__device__ __forceinline__ uint32_t nibbles_to_bytes(uint32_t x) {
  x = (x | (x << 8)) & 0x00FF00FFu;
  return (x | (x << 4)) & 0x0F0F0F0Fu;
}

// Projected QJL sign bits of the wave's residuals (lane l: r of its key, or
// with BOTH its key or value): bit i = !(p_i < 0) for p_i the binary32 fma
// chain over k ascending of S[i][k] r_k (the exact quantizer step).
// p~ = (sigma_i S_i) . (s r) comes from the matrix cores (sigma_i makes the
// row's norm 8; the power of two s brings ||r|| = g into [1, 2)), and its sign
// is taken where |p~_i| > kSignBand max_i ||sigma_i S_i|| ||s r||.
// There it is the chain's, whatever order and rounding the matrix cores sum a
// row's 192 products in. In units of ||sigma_i S_i|| ||s r||: where the signs
// differ the exact sum is next to 0, so its partial sums are at most 1/2
// (Cauchy-Schwarz on the two parts); one addition per product, truncated to
// fp32, then errs by up to 192 x 2^-24 = 2^-16.4, the split products by
// 2^-20.4, the fp16 spacing below 2^-14 by 2^-21 and the chain by 2^-19:
// 2^-16.1 in all, and kSignBand is twice that. (Rows of equal norm keep the
// band no wider than each row needs: 1024 tokens of 20 heads 12.2 us, 13.1 with
// rows scaled by powers of two.) The smallest
// |p~_i| tells whether any coordinate lies inside that band (snmax: the
// largest row norm, infinite if a row is not finite); only then are the rows
// found, and recomputed with the chain from S in memory for all the wave's
// vectors (every lane's bit of a recomputed row is the chain's).
// The residuals reach the B layout through v_permlane32_swap pairs
// (16q + j, 16q + 8 + j). With keys alone the result stays where it is: lane
// half h has the signs of the dimensions 8w + 4h + j of key n, which the
// halves exchange as one register.
template <bool BOTH>
__device__ __forceinline__ uint64_t projected_signs(float (&x)[kDim], float g, const _Float16* sh, const _Float16* sl,
                                                    float snmax, const float* S, int lane) {
  const float sc = unit_scale(g);
  const float sc_other = __shfl_xor(sc, 32, 64), g_other = __shfl_xor(g, 32, 64);
  const float sk = lane < 32 ? sc : sc_other, sv = lane < 32 ? sc_other : sc;   // of key n and value n
  // Step q's operands are built just before its products; the swaps are undone
  // only where the chain below needs the vectors again.
  auto swap_pairs = [&](int q) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[16 * q + j]),
                                                       __float_as_uint(x[16 * q + 8 + j]), false, false);
      x[16 * q + j] = __uint_as_float(sw[0]);       // key n, dimension 16q + 8h + j
      x[16 * q + 8 + j] = __uint_as_float(sw[1]);   // value n, dimension 16q + 8h + j
    }
  };
  Blocks acc;
  four_steps([&](auto q) {
    half8 h0, l0, h1{}, l1{};
    swap_pairs(q);
    split8(&x[16 * q], sk, h0, l0);
    if (BOTH) split8(&x[16 * q + 8], sv, h1, l1);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) product_step<q, BOTH, BOTH>(acc, mb, sh, sl, lane, h0, l0, h1, l1);
  });
  uint64_t bits, any = 0;
  if constexpr (BOTH) {
    float p[kDim];
    to_lane_per_vector(acc, p);
    const float band = snmax * (g * sc) * kSignBand;
    float least[4];                            // of dimensions 16 e .. 16 e + 15
    uint32_t neg[2];
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      least[e] = INFINITY;
      if (e & 1) neg[e >> 1] = 0;
#pragma unroll
      for (int i = 16 * e + 15; i > 16 * e; i -= 2) {
        neg[e >> 1] = push_sign(push_sign(neg[e >> 1], p[i]), p[i - 1]);
        least[e] = min_abs3(p[i], p[i - 1], least[e]);
      }
    }
    bits = ~(((uint64_t)neg[1] << 32) | neg[0]);
    const float low = fminf(fminf(least[0], least[1]), fminf(least[2], least[3]));
    if (__builtin_amdgcn_ballot_w64(!(low > band)) != 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (__builtin_amdgcn_ballot_w64(!(least[e] > band)) == 0) continue;
#pragma unroll
        for (int i = 16 * e; i < 16 * e + 16; ++i)
          any |= (uint64_t)(__builtin_amdgcn_ballot_w64(!(fabsf(p[i]) > band)) != 0) << i;
      }
    }
  } else {
    const float band = snmax * ((lane < 32 ? g : g_other) * sk) * kSignBand;
    float least[4];                            // of registers 8 e .. 8 e + 7
    uint32_t neg = 0;                          // nibble w: dimensions 8 w + 4 h + j
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      least[e] = INFINITY;
#pragma unroll
      for (int r = 8 * e + 7; r > 8 * e; r -= 2) {
        const float hi = acc[r >> 4][0][r & 15], lo = acc[(r - 1) >> 4][0][(r - 1) & 15];
        neg = push_sign(push_sign(neg, hi), lo);
        least[e] = min_abs3(hi, lo, least[e]);
      }
    }
    const uint32_t other = __shfl_xor(neg, 32, 64);
    bits = ~(((uint64_t)(nibbles_to_bytes(neg >> 16) | (nibbles_to_bytes(other >> 16) << 4)) << 32) |
             (nibbles_to_bytes(neg & 0xFFFFu) | (nibbles_to_bytes(other & 0xFFFFu) << 4)));
    const float low = fminf(fminf(least[0], least[1]), fminf(least[2], least[3]));
    if (__builtin_amdgcn_ballot_w64(!(low > band)) != 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (__builtin_amdgcn_ballot_w64(!(least[e] > band)) == 0) continue;
#pragma unroll
        for (int r = 8 * e; r < 8 * e + 8; ++r) {
          const uint64_t in = __builtin_amdgcn_ballot_w64(!(fabsf(acc[r >> 4][0][r & 15]) > band));
          const int d = 8 * (r >> 2) + (r & 3);
          any |= (uint64_t)((uint32_t)in != 0u) << d | (uint64_t)((uint32_t)(in >> 32) != 0u) << (d + 4);
        }
      }
    }
  }
  // rows inside the band: the fixed-order chain (wave-uniform row), over
  // vectors as the swaps left them: with keys alone, lane half h holds the
  // dimensions 16q + 8h + j, and the running sum of key n moves between lanes
  // n and n + 32 every eight elements (both halves run along; lane n ends with
  // the chain).
  if constexpr (BOTH) {
    if (any) {
#pragma unroll
      for (int q = 0; q < 4; ++q) swap_pairs(q);
    }
  }
  while (any) {
    const int i = __builtin_ctzll(any);
    any &= any - 1;
    float acc_i = 0.0f;
#pragma unroll
    for (int k = 0; k < kDim; ++k) {
      if (!BOTH && k > 0 && k % 8 == 0) acc_i = __shfl_xor(acc_i, 32, 64);
      acc_i = fmaf(scalar_load(S + i * kDim + k), x[BOTH ? k : 16 * (k / 16) + k % 8], acc_i);
    }
    if (!BOTH) acc_i = __shfl_xor(acc_i, 32, 64);
    bits = (bits & ~(1ull << i)) | ((uint64_t)((acc_i < 0.0f) ? 0u : 1u) << i);
  }
  return bits;
}

// 8 x 8 nibbles: nibble e of word d <- nibble d of word e.
__device__ __forceinline__ void transpose_nibbles(uint32_t (&m)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {                // halves: words e and e + 4
    const uint32_t x = m[e], y = m[e + 4];
    m[e] = __builtin_amdgcn_perm(y, x, 0x05040100u);
    m[e + 4] = __builtin_amdgcn_perm(y, x, 0x07060302u);
  }
#pragma unroll
  for (int e0 = 0; e0 < 4; ++e0) {             // bytes: words e and e + 2, e = 0, 1, 4, 5
    const int e = (e0 & 1) + 4 * (e0 >> 1);
    const uint32_t x = m[e], y = m[e + 2];
    m[e] = __builtin_amdgcn_perm(y, x, 0x06020400u);
    m[e + 2] = __builtin_amdgcn_perm(y, x, 0x07030501u);
  }
#pragma unroll
  for (int e = 0; e < 8; e += 2) {             // nibbles: words e and e + 1
    const uint32_t x = m[e], y = m[e + 1];
    m[e] = (x & 0x0F0F0F0Fu) | ((y & 0x0F0F0F0Fu) << 4);
    m[e + 1] = ((x >> 4) & 0x0F0F0F0Fu) | (y & 0xF0F0F0F0u);
  }
}

// All four bits of nibble j set where bit j of the low byte is.
__device__ __forceinline__ uint32_t nibble_mask(uint32_t m) {
  m = (m | (m << 12)) & 0x000F000Fu;
  m = (m | (m << 6)) & 0x03030303u;
  m = (m | (m << 3)) & 0x11111111u;
  return m * 15u;
}

// The groups of 32 tokens of a (layer, head), numbered through the sequences
// in order. In a ragged call sequence b has ceil(T_b / 32) of them; lane i of
// a wave then holds the running count of groups up to sequence first + i of a
// window of 64 sequences, and a group's sequence is found by one ballot (the
// window moves where the group lies outside it). Where there are more windows
// than one, the block's waves first count their groups into LDS, so that a
// window is found there (60000 sequences, one in 50 with 64 tokens, one head:
// 55 us; 694 with windows walked one after the other, 211 in blocks of their own
// per sequence).
constexpr int kMaxWindows = 1024;            // (the host keeps B below 2^16)

struct GroupCursor {
  int first, base, end;   // the window's first sequence; groups before and up to the end of the window
  int upto, own;          // per lane: groups up to and of sequence first + lane

  // Groups of sequence b.
  __device__ __forceinline__ static int groups(const QuantArgs& a, int b) {
    return b < a.B ? (min(max(a.tokens[b], 0), a.T) + kGroup - 1) / kGroup : 0;
  }

  // The window that holds a group, found in the groups before each one.
  __device__ __forceinline__ void find(const QuantArgs& a, const int* before, int windows, int group, int lane) {
    int lo = 0, hi = windows - 1;              // the last window with at most `group` before it
    while (lo < hi) {
      const int half = (lo + hi + 1) >> 1;
      if (__builtin_amdgcn_readfirstlane(before[half]) <= group) lo = half; else hi = half - 1;
    }
    window(a, 64 * lo, __builtin_amdgcn_readfirstlane(before[lo]), lane);
  }

  __device__ __forceinline__ void window(const QuantArgs& a, int f, int before, int lane) {
    first = f;
    base = before;
    own = groups(a, f + lane);
    upto = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int w = __shfl_up(upto, o, 64);
      upto += lane >= o ? w : 0;
    }
    upto += before;
    end = __builtin_amdgcn_readlane(upto, 63);
  }
};

// ---------------------------------------------------- lane-per-vector kernel
// One block of 12 waves per compute unit takes an equal, contiguous share of
// the call's groups of 32 tokens, numbered (layer, head) by (layer, head). It
// stages S once and Pi and the tables of up to four (layer, head)s at a time;
// its waves then take the groups of these in turn, with no barrier between
// (layer, head)s.
//
// What bounds it: the vector ALU, 1,690 instructions per group at three waves
// per SIMD (168 registers): 60 % of the issue slots over 1024 tokens of 33
// layers (the matrix cores are busy 18 %), and what three waves leave uncovered
// of their load and LDS latencies. Keys and values side by side in one wave
// (half the lanes each) make one instruction stream of both, halve the registers
// of the projected signs (only keys have them), and a group's keys and values end
// together; that the value lanes run the residual steps unused costs less.
// Four waves per SIMD would need 128 registers: the compiler then spills 40,
// and the spills' 78 MB of traffic cost more than the fourth wave gives (131
// against 112 us in blocks of 4 waves). At 168 the forms with V signs, whose
// projections double, spill 21 to 24 (88 to 100 B of scratch per lane), the fp32
// one without V signs 1, the others none; all keep 11 to 33 scalars in vector
// lanes.
// fp16, 20 heads, repeated on the same buffers: 1024 tokens of 33 layers 95 us
// (with V signs 122), of one layer 12.2 us, one layer of 64 sequences of 50 to
// 1024 tokens 100 us; 115 (161), 20.0 and 198 us in blocks of 4 waves of which
// each took 64 tokens of one sequence, first the keys and then the values: partly
// filled blocks and a chain twice as long.
constexpr int kPackWaves = 12;
constexpr int kPackThreads = kPackWaves * 64;
constexpr int kPackHeads = 4;       // (layer, head)s staged at a time
constexpr int kComputeUnits = 256;
constexpr int kVtPitch = 9;         // words per token in a wave's transpose buffer
constexpr int kVtDims8 = 36;        // words per 8 dimensions in it, after the transpose

template <bool F16, bool VQJL, bool ROTATED>
__global__ __launch_bounds__(kPackThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void quantize_tiles_kernel(QuantArgs a, int blocks, int groups_per_seq, DivMagic div_seq, DivMagic div_h) {
  __shared__ __attribute__((aligned(16))) _Float16 s_pih[kPackHeads][kDim * kDim];   // Pi, fp16 parts
  __shared__ __attribute__((aligned(16))) _Float16 s_pil[kPackHeads][kDim * kDim];
  __shared__ __attribute__((aligned(16))) _Float16 s_sh[kDim * kDim];                // sigma_i S_i, fp16 parts
  __shared__ __attribute__((aligned(16))) _Float16 s_sl[kDim * kDim];
  __shared__ float s_Sn[kDim];                                                        // ||sigma_i S_i||
  __shared__ __attribute__((aligned(16))) uint32_t s_vt[kPackWaves][8 * kVtDims8];
  __shared__ float s_lev[kPackHeads][2][8];                                           // K and V levels
  __shared__ float s_thr[kPackHeads][2][8];                                           // their t0, t2, t4, t6, t1, t3, t5
  __shared__ int s_asc[kPackHeads][2];                                                // strictly ascending
  __shared__ int s_before[kMaxWindows + 1];                                           // groups before a window
  // The thread's and the lane's number from a copy that the compiler cannot
  // carry over: what is derived from them is formed where it is used, instead
  // of staying live (and spilled) through the loops.
  auto thread_of = [&]() {
    int t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"((int)threadIdx.x));
    return t;
  };
  auto lane_of = [&]() { return thread_of() & 63; };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr bool rotated = ROTATED;
  const bool paper = (a.flags & kQjlPaper) != 0;

  // ---- the block's share of the groups. Blocks go to the 8 XCDs round-robin;
  // each XCD gets one contiguous eighth of the shares.
  GroupCursor cur{};
  int per_head = a.B * groups_per_seq;
  const int windows = (a.B + 63) >> 6;
  if (a.tokens) {
    if (windows == 1) {
      cur.window(a, 0, 0, lane_of());
      per_head = cur.end;
    } else {
      for (int w = wave; w < windows; w += kPackWaves) {
        int n = GroupCursor::groups(a, 64 * w + lane_of());
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);
        s_before[w] = n;
      }
      __syncthreads();
      if (wave == 0) {                         // each lane a run of windows
        const int lane = lane_of(), run = (windows + 63) >> 6, w0 = min(lane * run, windows);
        const int w1 = min(w0 + run, windows);
        int own = 0;
        for (int w = w0; w < w1; ++w) own += s_before[w];
        int upto = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int n = __shfl_up(upto, o, 64);
          upto += lane >= o ? n : 0;
        }
        int before = upto - own;
        for (int w = w0; w < w1; ++w) {
          const int n = s_before[w];
          s_before[w] = before;
          before += n;
        }
        if (lane == 63) s_before[windows] = upto;
      }
      __syncthreads();
      per_head = __builtin_amdgcn_readfirstlane(s_before[windows]);
    }
    if (per_head == 0) return;
  }
  const uint32_t share = (blockIdx.x % kXcds) * ((uint32_t)blocks / kXcds) + blockIdx.x / kXcds;
  const uint64_t total = (uint64_t)per_head * (uint32_t)(a.H * a.nlayers);
  const uint64_t begin = total * share / (uint32_t)blocks;
  int64_t left = (int64_t)(total * (share + 1) / (uint32_t)blocks - begin);
  uint32_t head = (uint32_t)(begin / (uint32_t)per_head);       // nlayers x H, relative to layer0
  int g0 = (int)(begin - (uint64_t)head * (uint32_t)per_head);  // the share starts at its group g0

  bool first = true;
  while (left > 0) {
    // (layer, head)s head .. head + nheads - 1: `count` groups from g0 of the first one on
    const int64_t reach = (left + g0 + per_head - 1) / per_head;
    const int nheads = (int)min(reach, (int64_t)kPackHeads);
    const int count = (int)min(left, (int64_t)nheads * per_head - g0);
    const int64_t lh0 = (int64_t)a.layer0 * a.H + head;
    if (!first) __syncthreads();               // the heads before are done with
    for (int u = thread_of(); u < nheads * 512; u += kPackThreads) {
      const int hd = u >> 9, r = (u & 511) >> 3, c = u & 7;
      const float4* src = reinterpret_cast<const float4*>(a.pi + (lh0 + hd) * kDim * kDim + r * kDim + 8 * c);
      const float4 x = src[0], y = src[1];
      const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
      half8 hi, lo;
      split8(v, 1.0f, hi, lo);
      *reinterpret_cast<half8*>(s_pih[hd] + staged_at(r, c)) = hi;
      *reinterpret_cast<half8*>(s_pil[hd] + staged_at(r, c)) = lo;
    }
    if (const int t = thread_of(); t < 2 * nheads) {
      const int hd = t >> 1, v = t & 1;
      const Levels L = load_levels((v ? a.lut_v : a.lut_k) + (lh0 + hd) * 8);
      float* lev = s_lev[hd][v];
      float* thr = s_thr[hd][v];
      // (a level of 0 as -0: then u - c is +0 for u of either zero)
      const auto of = [](float c) { return c == 0.0f ? -0.0f : c; };
      lev[0] = of(L.c0); lev[1] = of(L.c1); lev[2] = of(L.c2); lev[3] = of(L.c3);
      lev[4] = of(L.c4); lev[5] = of(L.c5); lev[6] = of(L.c6); lev[7] = of(L.c7);
      thr[0] = L.t0; thr[1] = L.t2; thr[2] = L.t4; thr[3] = L.t6; thr[4] = L.t1; thr[5] = L.t3; thr[6] = L.t5;
      s_asc[hd][v] = levels_ascending(L) ? 1 : 0;
    }
    // The rows of S scaled by sigma_i, and their norms, by the
    // last four waves: four threads per row, which combine their maxima and
    // sums by shuffles.
    if (const int t = thread_of() - (kPackThreads - 256); first && t >= 0) {
      const int r = t >> 2, c0 = 16 * (t & 3);
      const float4* s4 = reinterpret_cast<const float4*>(a.qjl_s) + r * 16 + c0 / 4;
      float sv[16];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float4 q4 = s4[u];
        sv[4 * u] = q4.x; sv[4 * u + 1] = q4.y; sv[4 * u + 2] = q4.z; sv[4 * u + 3] = q4.w;
      }
      float mx = 0.0f;
#pragma unroll
      for (int k = 0; k < 16; ++k) mx = fmaxf(mx, fabsf(sv[k]));
      mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
      float sig = unit_scale(mx);              // row r's scale (the same in its four threads)
      float ss = 0.0f;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const float v = sv[k] * sig;
        ss = fmaf(v, v, ss);
      }
      ss += __shfl_xor(ss, 1, 64);
      ss += __shfl_xor(ss, 2, 64);
      // Norm 8, so that the largest row's is every row's (rows whose norm is
      // not of the usual size keep the power of two).
      const float norm = sqrtf(ss), even = ss >= 1.0f && ss < 0x1p20f && sig < 0x1p100f ? 8.0f / norm : 1.0f;
      sig *= even;
      if ((t & 3) == 0) s_Sn[r] = norm * even; // bounds the guard band only
#pragma unroll
      for (int k = 0; k < 16; k += 8) {
        half8 hi, lo;
        split8(sv + k, sig, hi, lo);
        *reinterpret_cast<half8*>(s_sh + staged_at(r, (c0 + k) >> 3)) = hi;
        *reinterpret_cast<half8*>(s_sl + staged_at(r, (c0 + k) >> 3)) = lo;
      }
    }
    first = false;
    __syncthreads();
    float snmax = s_Sn[lane_of()];
    snmax = snmax < INFINITY ? snmax : INFINITY;   // (NaN: a row that is not finite)
    snmax = wave_max(snmax);

    for (int item = wave; item < count; item += kPackWaves) {
      int group = g0 + item, hd = 0;
      while (group >= per_head) { group -= per_head; ++hd; }   // (at most three times)
      // a (layer, head) whose K or V table is not strictly ascending is not written
      if (!__builtin_amdgcn_readfirstlane(s_asc[hd][0] & s_asc[hd][1])) continue;
      const int64_t lh = lh0 + hd;
      const int li = (int)div_magic((int)head + hd, div_h), h = (int)head + hd - li * a.H;
      // the group's sequence and tokens
      int b, j0, Tb;
      if (a.tokens) {
        const int lane = lane_of();
        if (group < cur.base || group >= cur.end) cur.find(a, s_before, windows, group, lane);
        const int i = __builtin_ctzll(__builtin_amdgcn_ballot_w64(cur.upto > group));
        b = cur.first + i;
        j0 = (group - __builtin_amdgcn_readlane(cur.upto - cur.own, i)) * kGroup;
        Tb = min(max(scalar_load(a.tokens + b), 0), a.T);
      } else {
        b = (int)div_magic(group, div_seq);
        j0 = (group - b * groups_per_seq) * kGroup;
        Tb = a.T;
      }
      const int64_t sbase = scalar_load(a.slot0 + b);
      const int pbase = scalar_load(a.pos0 + b);
      uint8_t* kreg = a.k_codes + lh * a.slots * 32;
      uint8_t* vreg = a.v_codes + lh * a.slots * 32;
      int lane = lane_of();
      bool is_v = lane >= 32;

      // ---- x^: keys after RoPE and rotation, values rotated like them unless
      // TQ_V_ROTATE is off; pre-rotated inputs as they are
      float x[kDim];
      float sc = 1.0f;
      auto row_of = [&]() { return ((((int64_t)li * a.B + b) * a.T + min(j0 + (lane & 31), Tb - 1)) * a.H + h) * kDim; };
      if (rotated) {
        load_vector<false>(x, is_v ? a.v : a.k, row_of());
      } else {
        RawRows<F16> raw;
        load_rows(raw, a, ((((int64_t)li * a.B + b) * a.T + min(j0 + (lane & 31), Tb - 1)) * a.H + h) * kDim,
                  min(max(pbase + min(j0 + (lane & 31), Tb - 1), 0), a.rope_positions - 1), lane);
        sc = rotate_rows(x, raw, s_pih[hd], s_pil[hd], (a.flags & kRopeHalf) != 0, lane);
        if (!(a.flags & kVRotate)) {
          if (is_v) {
            load_vector<F16>(x, a.v, row_of());
            sc = 1.0f;
          }
        }
      }

      // ---- norm, levels, residual, signs: words of 8 dimensions, three bits
      // each for keys and four for values
      uint32_t words[8];
      const QuantOut qo = quantize_lane(x, sc, s_thr[hd][is_v ? 1 : 0], s_lev[hd][is_v ? 1 : 0], is_v ? 4u : 3u, words);
      uint64_t sb;
      if (!paper) {
        sb = projected_signs<VQJL>(x, qo.g, s_sh, s_sl, snmax, a.qjl_s, lane);
      } else {
        uint32_t neg[2] = {0u, 0u};            // (the sign of r, never -0; a NaN of either sign is not below 0)
#pragma unroll
        for (int i = kDim - 1; i >= 0; --i) neg[i >> 5] = push_sign(neg[i >> 5], fminf(x[i], INFINITY));
        sb = ~(((uint64_t)neg[1] << 32) | neg[0]);
      }

      // The lane's token: written or not, its slot (formed here, so that
      // nothing of it stays live through the products).
      lane = lane_of();
      is_v = lane >= 32;
      const int jl = j0 + (lane & 31);
      const int64_t base = sbase + j0;         // the slot of the group's first token
      const int64_t slot = sbase + jl;
      const bool ok = jl < Tb && slot >= 0 && slot < a.slots &&
                      (rotated || (pbase + jl >= 0 && pbase + jl < a.rope_positions));
      const uint32_t okmask = (uint32_t)__builtin_amdgcn_ballot_w64(ok);   // (both halves alike)
      if (!is_v) {
#pragma unroll
        for (int w = 0; w < 8; ++w) words[w] |= (uint32_t)(sb >> (8 * w)) << 24;
        if (ok) {
          const int64_t ct = slot >> 6;
          const int r = (int)(slot & 63);
          *reinterpret_cast<uint4*>(kreg + tile_half_offset(ct, 0, r)) = make_uint4(words[0], words[1], words[2], words[3]);
          *reinterpret_cast<uint4*>(kreg + tile_half_offset(ct, 1, r)) = make_uint4(words[4], words[5], words[6], words[7]);
        }
      } else if (VQJL) {
#pragma unroll
        for (int w = 0; w < 8; ++w) words[w] |= nibble_mask((uint32_t)(sb >> (8 * w)) & 0xFFu) & 0x88888888u;
      }
      if (ok) {
        const uint32_t g16 = (VQJL || !is_v) ? qo.g16 : 0u;
        reinterpret_cast<uint32_t*>(a.scalars + (lh * a.slots + slot) * 4)[is_v ? 1 : 0] = qo.n16 | (g16 << 16);
      }

      // ---- V is stored dimension-major: transpose the group's 32 x 64 nibbles
      // through the wave's LDS buffer, in blocks of 8 tokens x 8 dimensions
      // (lane (w, k) of the lower half: dimensions 8w .., tokens 8k ..), so
      // that lane i gets the 16 bytes of dimension i. The pitches keep every
      // access off a bank that another lane uses.
      uint32_t* s_w = s_vt[wave];
      if (is_v) {
#pragma unroll
        for (int w = 0; w < 8; ++w) s_w[(lane & 31) * kVtPitch + w] = words[w];
      }
      wave_sync_lds();
      uint32_t m[8];
      {
        const int w = (lane & 31) >> 2, k = lane & 3;
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = s_w[(8 * k + e) * kVtPitch + w];
        transpose_nibbles(m);                  // m[d]: dimension 8w + d, token 8k + e in nibble e
        wave_sync_lds();
        if (!is_v) {
#pragma unroll
          for (int d = 0; d < 8; ++d) s_w[w * kVtDims8 + 4 * d + k] = m[d];
        }
      }
      wave_sync_lds();
      const uint4 dim = *reinterpret_cast<const uint4*>(s_w + (lane >> 3) * kVtDims8 + 4 * (lane & 7));
      wave_sync_lds();                         // (the next group writes the buffer)
      if (okmask == ~0u && (base & 31) == 0) {
        *reinterpret_cast<uint4*>(vreg + tile_half_offset(base >> 6, (int)((base & 63) >> 5), lane)) = dim;
      } else if (okmask != 0u) {
        // any slots: words of 8 slots, of which `sh` precede the group's first token
        const int sh = (int)(base & 7);
        const int64_t G0 = (base - sh) / 8;    // (exact: base may be below 0)
        const uint32_t d[6] = {0u, dim.x, dim.y, dim.z, dim.w, 0u};
        const uint64_t in = (uint64_t)okmask << sh;
#pragma unroll
        for (int g = 0; g < 5; ++g) {
          const uint32_t mask = nibble_mask((uint32_t)(in >> (8 * g)) & 0xFFu);
          if (mask == 0u) continue;
          const uint32_t word = sh ? (d[g + 1] << (4 * sh)) | (d[g] >> (32 - 4 * sh)) : d[g + 1];
          const int64_t G = G0 + g;
          store_v_word(reinterpret_cast<uint32_t*>(vreg + tile_half_offset(G >> 3, (int)((G & 7) >> 2), lane) + (G & 3) * 4),
                       word, mask);
        }
      }
    }
    left -= count;
    head += nheads;
    g0 = 0;
  }
}

// Blocks of a launch: one per compute unit, or one per group where there are
// fewer (an upper bound in a ragged call); a multiple of 8 (the XCDs).
static int pack_blocks(int64_t groups) {
  return (int)((std::min<int64_t>(groups, kComputeUnits) + kXcds - 1) / kXcds * kXcds);
}

// ----------------------------------------------- wave-per-vector kernel
// Coalesced copy of a 64 x 64 row-major matrix into its staged form, in two
// steps so that the loads can be issued early: thread t holds float4 number
// t + 128 j (row e / 16, columns 4 (e % 16) .. 4 (e % 16) + 3).
struct MatrixSlice {
  float4 v[8];
};

__device__ __forceinline__ void load_slice(const float* __restrict__ m, MatrixSlice& sl, int t) {
#pragma unroll
  for (int j = 0; j < 8; ++j) sl.v[j] = reinterpret_cast<const float4*>(m)[t + 128 * j];
}

__device__ __forceinline__ void store_slice(const MatrixSlice& sl, float* m, int t) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int e = t + 128 * j;
    stage_row4(m, e >> 4, (e & 15) * 4, sl.v[j]);
  }
}

template <bool F16>
__global__ __launch_bounds__(128) void quantize_vectors_kernel(QuantArgs a, uint32_t total) {
  __shared__ VectorSmem sm;
  const int wave = threadIdx.x >> 6, i = threadIdx.x & 63;
  const uint32_t th = blockIdx.x;   // the host keeps the token-head count below 2^31
  if (th >= total) return;
  const bool is_v = wave == 1;
  const uint32_t h = th % (uint32_t)a.H;
  uint32_t rest = th / (uint32_t)a.H;
  const uint32_t j = rest % (uint32_t)a.T;
  rest /= (uint32_t)a.T;
  const uint32_t b = rest % (uint32_t)a.B;
  const uint32_t li = rest / (uint32_t)a.B;
  const int l = a.layer0 + (int)li;
  const int64_t lh = (int64_t)l * a.H + h;
  const bool rotated = (a.flags & kInputRotated) != 0;
  const bool paper = (a.flags & kQjlPaper) != 0;
  const int ksign = paper ? 2 : 1;
  const int sign_mode = is_v ? ((a.flags & kVQjl) ? ksign : 0) : ksign;
  const bool any_rotate = !rotated;                       // keys rotate unless pre-rotated
  const bool rotate = !rotated && (!is_v || (a.flags & kVRotate));
  const bool any_proj = !paper;                           // keys use the projection unless paper
  const int64_t row = ((((int64_t)li * a.B + b) * a.T + j) * a.H + h) * kDim;

  // ---- loads that do not depend on the slot, issued first
  float x = load_in(is_v ? a.v : a.k, row + i, F16);
  const Levels L = load_levels((is_v ? a.lut_v : a.lut_k) + lh * 8);
  const Levels Lo = load_levels((is_v ? a.lut_k : a.lut_v) + lh * 8);
  MatrixSlice pi_sl, s_sl;
  if (any_rotate) load_slice(a.pi + lh * kDim * kDim, pi_sl, threadIdx.x);
  if (any_proj) load_slice(a.qjl_s, s_sl, threadIdx.x);
  const int64_t slot = a.slot0[b] + j;
  const int pos = a.pos0[b] + (int)j;
  const int Tb = a.tokens ? min(max(a.tokens[b], 0), a.T) : a.T;
  // block-uniform exits (before any barrier); a (layer, head) whose K or V
  // table is not strictly ascending is not written
  if ((int)j >= Tb) return;               // beyond the sequence's tokens (a ragged call)
  if (slot < 0 || slot >= a.slots) return;
  if (!levels_ascending(L) || !levels_ascending(Lo)) return;
  if (!rotated && (pos < 0 || pos >= a.rope_positions)) return;
  const bool half = (a.flags & kRopeHalf) != 0;
  float2 cs = make_float2(1.0f, 0.0f);
  if (!is_v && !rotated) {
    const int m = half ? (i & 31) : (i >> 1);
    cs = reinterpret_cast<const float2*>(a.rope_cs + (int64_t)pos * 2 * kPairs)[m];
  }
  if (any_rotate) store_slice(pi_sl, sm.pi, threadIdx.x);
  if (any_proj) store_slice(s_sl, sm.s, threadIdx.x);
  __syncthreads();

  // ---- RoPE (keys), rotation, quantizer, store
  if (!is_v && !rotated) x = rope_wave(x, cs, half, i);
  append_wave<Pitch68>(x, is_v, rotate, L, sm.pi, sm.s, sm.x[wave], sm.r[wave], sign_mode, slot, lh,
                       a.k_codes, a.v_codes, a.scalars, a.slots, i);
}

// ------------------------------------------- wave-per-four-vectors kernel
// Rows lie 68 floats apart, so that the reads of four rows at one column do
// not meet in a bank.
constexpr int kVecPitch = kDim + 4;

constexpr int kRowChunks = 8;       // 16-byte chunks of a row in registers at a time

// Row i of a 64 x 64 matrix staged in `m` (Swz16) times NT vectors held one
// element per lane: fma chains over k ascending (row_dot's). The row is read
// once for all of them, and their elements reach the chains through row
// broadcasts: reading them from LDS too (one 16-byte broadcast per four
// elements and vector) made its return path the bound.
template <int K0, int NT, int... K4>
__device__ __forceinline__ void row_dots_steps(const float4 (&mr)[kRowChunks], const LaneSpread (&v)[NT],
                                               float (&acc)[NT], std::integer_sequence<int, K4...>) {
  auto step = [&](auto k4, const float4& m) {
    constexpr int K = 4 * (K0 + k4.value), J = K / 16;
#pragma unroll
    for (int t = 0; t < NT; ++t) fma_row_bcast<K % 16>(acc[t], v[t].r[J], m.x);
#pragma unroll
    for (int t = 0; t < NT; ++t) fma_row_bcast<K % 16 + 1>(acc[t], v[t].r[J], m.y);
#pragma unroll
    for (int t = 0; t < NT; ++t) fma_row_bcast<K % 16 + 2>(acc[t], v[t].r[J], m.z);
#pragma unroll
    for (int t = 0; t < NT; ++t) fma_row_bcast<K % 16 + 3>(acc[t], v[t].r[J], m.w);
  };
  (step(std::integral_constant<int, K4>{}, mr[K4]), ...);
}

template <int NT>
__device__ __forceinline__ void row_dots(const float* m, int i, float (&x)[NT]) {
  const float4* m4 = reinterpret_cast<const float4*>(m);
  float4 mr[kRowChunks];
#pragma unroll
  for (int k4 = 0; k4 < kRowChunks; ++k4) mr[k4] = m4[Swz16::chunk(i, k4)];
  LaneSpread v[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    v[t] = spread_lanes(x[t]);
    x[t] = 0.0f;
  }
  // (the two wait states before a DPP read)
#pragma unroll
  for (int t = 0; t < NT; ++t)
    asm volatile("s_nop 1" : "+v"(v[t].r[0]), "+v"(v[t].r[1]), "+v"(v[t].r[2]), "+v"(v[t].r[3]));
  constexpr auto steps = std::make_integer_sequence<int, kRowChunks>{};
  row_dots_steps<0>(mr, v, x, steps);
#pragma unroll
  for (int k4 = 0; k4 < kRowChunks; ++k4) mr[k4] = m4[Swz16::chunk(i, kRowChunks + k4) + after(x[0])];
  row_dots_steps<kRowChunks>(mr, v, x, steps);
}

// A block stages Pi and S of one (layer, head) once (direct 16-byte copies
// into LDS) for a chunk of its tokens, the sequences' tokens counted through;
// waves 0 .. 3 take their keys and waves 4 .. 7 their values, four at a time
// (one lane per dimension). The steps of each vector are append_wave's, in its
// order, so the bytes are quantize_vectors_kernel's; four vectors share the
// reads of the matrix rows, and their norm chains run in different lanes (lane
// t runs vector t's).
//
// What bounds it: the vector ALU, 63 % of the issue slots at four waves per SIMD
// (60 tokens x 1440 (layer, head)s), and the waits between the fma chains. At the
// 128 registers of four waves it spills 24 (100 B of scratch per lane) and keeps
// 41 scalars in vector lanes. fp16, 60 tokens x 1440 (layer, head)s 115 us, 8 tokens of 64 sequences
// x 20 heads 23.5 us; 324 and 39.1 us in quantize_vectors_kernel, whose blocks
// stage 32 KB per token and merge every value nibble by two atomics of its own
// (alone 65 of the 180 us that this kernel took with them).
constexpr int kVecWaves = 8;
constexpr int kVecTokens = 4;       // per wave

template <bool F16>
__global__ __launch_bounds__(kVecWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
void quantize_batch_kernel(QuantArgs a, int total_blocks, int per_xcd, int chunk_tokens, DivMagic div_chunks,
                           DivMagic div_t, DivMagic div_h, int chunks) {
  constexpr int NT = kVecTokens;
  __shared__ __attribute__((aligned(16))) float s_pi[kDim * kDim];   // Swz16
  __shared__ __attribute__((aligned(16))) float s_s[kDim * kDim];
  __shared__ __attribute__((aligned(16))) float s_x[kVecWaves][NT * kVecPitch];
  const int work = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (work >= total_blocks) return;
  const int head = (int)div_magic(work, div_chunks);     // nlayers x H, relative to layer0
  const int chunk = work - head * chunks;
  const int li = (int)div_magic(head, div_h), h = head - li * a.H;
  const int64_t lh = (int64_t)a.layer0 * a.H + head;
  const int i = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool is_v = wave >= kVecWaves / 2;
  const bool rotated = (a.flags & kInputRotated) != 0;
  const bool paper = (a.flags & kQjlPaper) != 0;
  const int ksign = paper ? 2 : 1;
  const int sign_mode = is_v ? ((a.flags & kVQjl) ? ksign : 0) : ksign;
  const bool rotate = !rotated && (!is_v || (a.flags & kVRotate));
  const bool half = (a.flags & kRopeHalf) != 0;
  {
    typedef __attribute__((address_space(3))) void* lds_ptr;
    const float* pig = a.pi + lh * kDim * kDim;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c0 = (wave + kVecWaves * j) * 64;
      if (!rotated)                                      // keys rotate unless pre-rotated
        __builtin_amdgcn_global_load_lds(pig + Swz16::source(c0 + i) * 4, (lds_ptr)(s_pi + c0 * 4), 16, 0, 0);
      if (!paper)                                        // keys use the projection unless paper
        __builtin_amdgcn_global_load_lds(a.qjl_s + Swz16::source(c0 + i) * 4, (lds_ptr)(s_s + c0 * 4), 16, 0, 0);
    }
  }
  const int all = a.B * a.T;
  const int stop = min(all, (chunk + 1) * chunk_tokens);
  // Four tokens from n0 on: written or not, their slots, and the lane's element
  // and RoPE (cos, sin) of each. Loaded ahead: the first ones with the staging,
  // the next ones while the ones before are quantized.
  float x_in[NT];
  float2 cs[NT];
  int64_t slot_in[NT];
  uint32_t ok_in = 0;
  auto fetch = [&](int n0) {
    ok_in = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = min(n0 + t, all - 1);
      const int b = (int)div_magic(n, div_t), j = n - b * a.T;
      const int Tb = a.tokens ? min(max(scalar_load(a.tokens + b), 0), a.T) : a.T;
      const int pos = scalar_load(a.pos0 + b) + j;
      const int64_t slot = scalar_load(a.slot0 + b) + j;
      slot_in[t] = slot;
      x_in[t] = 0.0f;
      cs[t] = make_float2(1.0f, 0.0f);
      if (n0 + t < stop && j < Tb && slot >= 0 && slot < a.slots &&
          (rotated || (pos >= 0 && pos < a.rope_positions))) {
        ok_in |= 1u << t;
        const int64_t row = ((((int64_t)li * a.B + b) * a.T + j) * a.H + h) * kDim;
        x_in[t] = load_in(is_v ? a.v : a.k, row + i, F16);
        if (!is_v && !rotated)
          cs[t] = reinterpret_cast<const float2*>(a.rope_cs + (int64_t)pos * 2 * kPairs)[half ? (i & 31) : (i >> 1)];
      }
    }
  };
  int n0 = chunk * chunk_tokens + (wave & 3) * NT;
  fetch(n0);
  const Levels L = load_levels((is_v ? a.lut_v : a.lut_k) + lh * 8);
  const Levels Lo = load_levels((is_v ? a.lut_k : a.lut_v) + lh * 8);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // a (layer, head) whose K or V table is not strictly ascending is not written
  if (!levels_ascending(L) || !levels_ascending(Lo)) return;

  float* xs = s_x[wave];
  const float* own = xs + (i & (NT - 1)) * kVecPitch;
  for (; n0 < stop; n0 += 4 * NT) {
    float x[NT];
    int64_t slot[NT];
    const uint32_t ok = ok_in;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      x[t] = !is_v && !rotated ? rope_wave(x_in[t], cs[t], half, i) : x_in[t];
      slot[t] = slot_in[t];
    }
    fetch(n0 + 4 * NT);
    // ---- rotation
    if (rotate) row_dots<NT>(s_pi, i, x);
    // ---- norm, levels, residual
#pragma unroll
    for (int t = 0; t < NT; ++t) xs[t * kVecPitch + i] = x[t];
    wave_sync_lds();
    const float n_own = sqrtf(sum_squares<8>(own));
    const float inv_own = (n_own == 0.0f) ? 0.0f : 8.0f / n_own;
    wave_sync_lds();
    TQ_PIN_LEVELS(L);
    uint32_t nib[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float u = x[t] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv_own), t));
      const float lv = nearest_level(u, TQ_LEVELS(L), &nib[t]);
      x[t] = u - lv;
      xs[t * kVecPitch + i] = x[t];
    }
    wave_sync_lds();
    const float g_own = sqrtf(sum_squares<8>(own));
    const uint32_t scal_own = store_norm(n_own) | ((sign_mode == 0 ? 0u : store_norm(g_own)) << 16);
    // ---- signs
    if (sign_mode == 1) {
      row_dots<NT>(s_s, i, x);
#pragma unroll
      for (int t = 0; t < NT; ++t) nib[t] |= ((x[t] < 0.0f) ? 0u : 1u) << 3;
    } else if (sign_mode == 2) {
#pragma unroll
      for (int t = 0; t < NT; ++t) nib[t] |= ((x[t] < 0.0f) ? 0u : 1u) << 3;
    }
    wave_sync_lds();                                     // xs is written again by the next tokens
    // ---- stores; values of tokens in the same eight slots together
    if (!is_v) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (ok & (1u << t))
          store_key(nib[t], (uint32_t)__builtin_amdgcn_readlane((int)scal_own, t), slot[t], lh, a.k_codes, a.scalars,
                    a.slots, i);
    } else {
      uint32_t word = 0, mask = 0;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (!(ok & (1u << t))) continue;
        const int sh = 4 * (int)(slot[t] & 7);
        word |= nib[t] << sh;
        mask |= 15u << sh;
        const int u = t + 1 < NT ? t + 1 : t;
        if (u == t || !(ok & (1u << u)) || (slot[u] >> 3) != (slot[t] >> 3)) {
          store_value_nibbles(word, mask, slot[t] >> 3, lh, a.v_codes, a.slots, i);
          word = 0;
          mask = 0;
        }
      }
      if (i < NT && (ok & (1u << i))) {
        int64_t s = slot[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) s = i == t ? slot[t] : s;
        reinterpret_cast<uint32_t*>(a.scalars + (lh * a.slots + s) * 4)[1] = scal_own;
      }
    }
  }
}

// Its tokens per block: a pass takes 16 of a (layer, head); as many passes as
// bring the blocks down to the two per compute unit that run at once (a pass
// more costs less than a second staging).
static int batch_chunk(int64_t heads, int64_t tokens) {
  const int64_t passes = (tokens + 15) / 16;
  const int64_t per_head = std::max<int64_t>(1, std::min(passes, 2 * (int64_t)kComputeUnits / heads));
  return (int)((passes + per_head - 1) / per_head * 16);
}

// Whether quantize_batch_kernel takes a call of short sequences: from 12 tokens
// per (layer, head) on, where the token-heads fill its passes. A pass costs it
// about the same however few of its 16 tokens there are; up to one block per
// compute unit it waits on nothing else. Without the rotation or the projection
// (`without` of the two) the other kernel has less to stage per token, and the
// line lies higher. One token per sequence (fp16, us, this kernel /
// quantize_vectors_kernel): one block per compute unit at most, 180 heads x 12
// tokens 11 / 12, 140 x 16 12 / 12; one pass of more blocks, 140 x 18 15 / 13,
// 180 x 18 16 / 15, 220 x 17 16 / 17, 340 x 12 16 / 18; two passes, 260 x 20
// 24 / 21, 300 x 20 25 / 24, 340 x 20 25 / 27, 400 x 17 24 / 27. In the
// per-element form 180 x 16 12.4 / 11.6, 256 x 12 12.4 / 12.2, 20 x 200 15.5 /
// 14.6, 256 x 20 15.7 / 17.5, 340 x 20 23.5 / 22.4, 400 x 20 25.2 / 25.6.
static bool batch_pays(int64_t heads, int64_t tokens, int without) {
  const int64_t passes = batch_chunk(heads, tokens) / 16, blocks = heads * ((tokens + 16 * passes - 1) / (16 * passes));
  const int64_t least = passes == 1 && blocks <= kComputeUnits ? (without == 1 ? 3100 : 2048)
                                                               : (600 + 3000 * passes) * (4 + without) / 4;
  return tokens >= 12 && heads * tokens >= least;
}

hipError_t launch_quantize(const QuantArgs& a, hipStream_t st) {
  const bool f16 = a.f16 && !(a.flags & kInputRotated);
  if (a.T >= 64) {
    const int per_seq = (int)(((int64_t)a.T + kGroup - 1) / kGroup);
    const int blocks = pack_blocks((int64_t)per_seq * a.B * a.H * a.nlayers);
    const DivMagic div_seq = make_div_magic((uint32_t)per_seq), div_h = make_div_magic((uint32_t)a.H);
    const bool vq = (a.flags & kVQjl) != 0;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kPackThreads), 0, st, a, blocks, per_seq, div_seq, div_h);
    };
    if (a.flags & kInputRotated)
      vq ? launch(quantize_tiles_kernel<false, true, true>) : launch(quantize_tiles_kernel<false, false, true>);
    else if (f16)
      vq ? launch(quantize_tiles_kernel<true, true, false>) : launch(quantize_tiles_kernel<true, false, false>);
    else
      vq ? launch(quantize_tiles_kernel<false, true, false>) : launch(quantize_tiles_kernel<false, false, false>);
  } else {
    const int64_t heads = (int64_t)a.nlayers * a.H, tokens = (int64_t)a.B * a.T;
    const uint32_t total = (uint32_t)(heads * tokens);
    const int without = ((a.flags & kInputRotated) != 0) + ((a.flags & kQjlPaper) != 0);
    if (batch_pays(heads, tokens, without)) {
      const int chunk = batch_chunk(heads, tokens);
      const int chunks = (int)((tokens + chunk - 1) / chunk), blocks = (int)(heads * chunks);
      const int per_xcd = (blocks + kXcds - 1) / kXcds;
      auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)per_xcd * kXcds), dim3(kVecWaves * 64), 0, st, a, blocks, per_xcd,
                           chunk, make_div_magic((uint32_t)chunks), make_div_magic((uint32_t)a.T),
                           make_div_magic((uint32_t)a.H), chunks);
      };
      f16 ? launch(quantize_batch_kernel<true>) : launch(quantize_batch_kernel<false>);
      return hipGetLastError();
    }
    if (f16)
      hipLaunchKernelGGL(quantize_vectors_kernel<true>, dim3(total), dim3(128), 0, st, a, total);
    else
      hipLaunchKernelGGL(quantize_vectors_kernel<false>, dim3(total), dim3(128), 0, st, a, total);
  }
  return hipGetLastError();
}

}  // namespace tq
