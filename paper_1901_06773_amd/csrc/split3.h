// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values: h = bf16(x), m = bf16(x - h), l = x - h - m
// (8 significant bits each, 24 in all; both differences are exact).  A product is then
//   a*b = ah*bh + (ah*bm + am*bh) + (ah*bl + am*bm + al*bh) + terms below 2^-25 of |a*b|,
// six v_mfma_f32_32x32x16_bf16 (32 cycles each) where the fp32 instruction needs eight of 64 cycles
// (v_mfma_f32_32x32x2_f32) for the same 32 x 32 x 16 products, with the same fp32 accumulators.
// The terms left out are smaller than the rounding of one fp32 addition, and the sum is rounded 6 times per
// 16 products instead of 16 times.
//
// The parts are taken of the value times 2^24.  bf16 has the exponents of fp32 but 16 bits less: below 2^-110 the lowest part of a
// value would fall under the smallest bf16 (2^-133) and the value be held in fewer than 24 bits (2e-3 of it lost at
// 2^-125); times 2^24 every part of every fp32 value, subnormal ones included, is a normal bf16.  The sums come out times
// 2^48 and are taken back when they are finished.  Values and sums that leave the range at the other end (infinities, NaN,
// values from 2^104 and sums from 2^80 on) end up non-finite in the accumulator; the kernels then redo the tile in fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace acc {

typedef float x3_v16f __attribute__((ext_vector_type(16)));
typedef float x3_v4f __attribute__((ext_vector_type(4)));
typedef unsigned x3_v4u __attribute__((ext_vector_type(4)));
typedef unsigned x3_v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t x3_pack(float a, float b) {   // two bf16, round to nearest even
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  typedef float v2f __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));
}

constexpr float kX3Scale = 16777216.f;                                // 2^24, of every value
constexpr float kX3Unscale = 1.f / (kX3Scale * kX3Scale);             // of the sums of products

// the three parts of two values (times kX3Scale), packed in pairs
__device__ __forceinline__ void x3_split(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  a *= kX3Scale;
  b *= kX3Scale;
  h = x3_pack(a, b);
  const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
  m = x3_pack(ra, rb);
  l = x3_pack(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
}

__device__ __forceinline__ x3_v16f x3_mfma(const x3_v4u& a, const x3_v4u& b, x3_v16f c) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
#else
  return c;  // the host pass never runs this
#endif
}

// One of the products of an MB x NB group of 32 x 32 blocks: part PA of a times part PB of b (0 = h, 1 = m,
// 2 = l); consecutive instructions work on different accumulators where there are several.
template <int PA, int PB, int MB, int NB>
__device__ __forceinline__ void x3_product(const x3_v4u (&a)[3][MB], const x3_v4u (&b)[3][NB], x3_v16f (&acc)[MB][NB]) {
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = x3_mfma(a[PA][i], b[PB][j], acc[i][j]);
}

// true in every lane of the wave if any accumulator of any lane is an infinity or a NaN
template <int MB, int NB>
__device__ __forceinline__ bool x3_any_nonfinite(const x3_v16f (&acc)[MB][NB]) {
#if defined(__HIP_DEVICE_COMPILE__)
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) t = fmaf(acc[i][j][v], 0.f, t);      // 0, or NaN from then on
  return __any(t != 0.f);
#else
  return false;
#endif
}

}  // namespace acc
