// bf16 operand planes of the matrix products (device side).
//
// bf16-GEMM mode: one plane, the value rounded to nearest even. fp32 mode: three planes
// p1 + p2 + p3 = v exactly (8 significant bits each of the 24), and a product is the six
// bf16 products p1q1 + p1q2 + p2q1 + p1q3 + p2q2 + p3q1 accumulated in fp32; what is left out is
// below 2^-25 of |v||w|, half an ulp of one fp32 product. The bf16 MFMAs have 16 times the rate of the
// fp32 ones, so six of them take 3/8 of the time. A plane ends at bf16's smallest number, 2^-133, so values
// below about 1e-35 keep 2^-134 of absolute precision (gradients of 1e-34: dx 1.5e-6 off, normwise per step).
#pragma once
#include "common.h"

template <int S>
__device__ __forceinline__ void split_bf16(float v, bf16_t (&p)[S]) {
  p[0] = f32_to_bf16_bits(v);
  if constexpr (S == 3) {
    // a finite value that rounds to infinity keeps its upper half; infinities and NaN have no rest
    const uint32_t bits = __float_as_uint(v);
    const bool finite = (bits & 0x7f800000u) != 0x7f800000u;
    if (finite && (p[0] & 0x7f80u) == 0x7f80u) p[0] = (bf16_t)(bits >> 16);
    const float r = finite ? v - bf16_bits_to_f32(p[0]) : 0.f;
    p[1] = f32_to_bf16_bits(r);
    p[2] = f32_to_bf16_bits(r - bf16_bits_to_f32(p[1]));
  }
}

// Eight values to one 16-byte granule per plane.
template <int S>
__device__ __forceinline__ void split_granule(const float (&v)[8], uint4 (&g)[S]) {
  uint32_t w[S][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bf16_t lo[S], hi[S];
    split_bf16<S>(v[2 * j], lo);
    split_bf16<S>(v[2 * j + 1], hi);
#pragma unroll
    for (int s = 0; s < S; ++s) w[s][j] = (uint32_t)lo[s] | ((uint32_t)hi[s] << 16);
  }
#pragma unroll
  for (int s = 0; s < S; ++s) g[s] = uint4{w[s][0], w[s][1], w[s][2], w[s][3]};
}

// acc[j] += the plane products of one K step of A fragment a[j] and B fragment b. The MFMA aligns
// its addends to the largest and cuts off (towards minus infinity) what falls below a few guard
// bits, so small products on a large accumulator, or large products on a small one, lose up to
// 2^-27 of the large one each time, always to the same side: the gradient sums over tens of
// thousands of nodes show it (db of 81k nodes: 3.6e-6 off instead of 0.5e-6). The small products
// of a step are therefore added up apart from the large ones, both from zero, and joined to the
// sum by ordinary additions.
template <int N>
__device__ __forceinline__ void mfma_planes_add(const bf16x8 (&a)[N][3], const bf16x8 (&b)[3], f32x4 (&acc)[N]) {
  f32x4 lo[N], hi[N];
#pragma unroll
  for (int j = 0; j < N; ++j) lo[j] = mfma_bf16_16x16x32(a[j][2], b[0], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
  for (int j = 0; j < N; ++j) lo[j] = mfma_bf16_16x16x32(a[j][1], b[1], lo[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) lo[j] = mfma_bf16_16x16x32(a[j][0], b[2], lo[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) lo[j] = mfma_bf16_16x16x32(a[j][1], b[0], lo[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) lo[j] = mfma_bf16_16x16x32(a[j][0], b[1], lo[j]);
#pragma unroll
  for (int j = 0; j < N; ++j) hi[j] = mfma_bf16_16x16x32(a[j][0], b[0], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] += hi[j] + lo[j];
}

// Recurrent products (h U and dA U^T, whose U stays in registers). bf16-GEMM mode: one bf16 plane.
// fp32 mode: two fp16 planes of the value times a power of two that brings the largest of its unit
// (U), row piece (dA) or of all states (h, |h| < 1) just under 2^15: p1 + p2 holds 22 to 24
// significant bits down to 2^-17 of the largest and 2^-40 of the largest below that, and a product
// is p1q1 + p1q2 + p2q1, three MFMAs and two thirds of the registers of the bf16 planes.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
constexpr int kHExp = 15;                // exponent of the scale of h
constexpr float kHScale = 32768.f;
// A row piece's inverse scale is kept as 2^-(s + kDaExp) and a unit's as 2^(kDaExp - s): both are fp32
// numbers, and the sums over the pieces, in units of the largest weight, overflow only with dA itself.
constexpr int kDaExp = 14;

template <int NP>
__device__ __forceinline__ void split_rec(float v, float scale, uint16_t (&p)[NP]) {
  if constexpr (NP == 1) {
    p[0] = f32_to_bf16_bits(v);
  } else {
    const float s = v * scale;
    const _Float16 a = (_Float16)s;
    p[0] = __builtin_bit_cast(uint16_t, a);
    // (an infinity has no rest)
    const float r = s - (float)a;
    p[1] = __builtin_bit_cast(uint16_t, (_Float16)(__builtin_isfinite(s) ? r : 0.f));
  }
}
template <int NP>
__device__ __forceinline__ void split_rec_granule(const float (&v)[8], float scale, uint4 (&g)[NP]) {
  uint32_t w[NP][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint16_t lo[NP], hi[NP];
    split_rec<NP>(v[2 * j], scale, lo);
    split_rec<NP>(v[2 * j + 1], scale, hi);
#pragma unroll
    for (int s = 0; s < NP; ++s) w[s][j] = (uint32_t)lo[s] | ((uint32_t)hi[s] << 16);
  }
#pragma unroll
  for (int s = 0; s < NP; ++s) g[s] = uint4{w[s][0], w[s][1], w[s][2], w[s][3]};
}
// Exponent s of the power of two that brings a largest magnitude m into [2^14, 2^15): -113 .. 127 (0
// for zero). At 127 (m below 2^-112) the largest ends under 2^14, and every fp32 number of its size is
// still a whole number of fp16's smallest steps. A non-finite m gets -114: no finite value becomes
// infinite. 2^s and 2^-s are fp32 numbers (2^-127 a subnormal one); the two inverse scales of a product
// together need not be, so they are applied one after the other or as a sum of exponents.
__device__ __forceinline__ int rec_exp(float m) {
  const int e = (int)((__float_as_uint(m) >> 23) & 0xffu);
  return m == 0.f ? 0 : min(127 + 14 - e, 127);
}
__device__ __forceinline__ float rec_scale(int s) { return __uint_as_float((uint32_t)(127 + s) << 23); }
__device__ __forceinline__ float rec_ldexp(float v, int e) { return __builtin_amdgcn_ldexpf(v, e); }
// acc += the products of K chunk c. fp32 mode: the first plane of A is stored negated in odd chunks
// and its products subtracted, so that what the MFMA cuts off, always towards minus infinity,
// cancels between chunks; those of the second plane gather in lo.
__device__ __forceinline__ f32x4 mfma_f16_16x16x32(const uint4& x, const uint4& y, f32x4 z) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), z, 0, 0, 0);
}
template <int NP>
__device__ __forceinline__ void mfma_rec(int c, const uint4 (&a)[NP], const uint4 (&b)[NP], f32x4& acc, f32x4& lo) {
  if constexpr (NP == 1) {
    acc = mfma_bf16_16x16x32(__builtin_bit_cast(bf16x8, a[0]), __builtin_bit_cast(bf16x8, b[0]), acc);
  } else {
    f32x4 hi = mfma_f16_16x16x32(a[0], b[1], f32x4{0.f, 0.f, 0.f, 0.f});
    lo = mfma_f16_16x16x32(a[1], b[0], lo);
    hi = mfma_f16_16x16x32(a[0], b[0], hi);
    if (c & 1) acc -= hi;
    else acc += hi;
  }
}
// The same of the first planes alone, fp32 mode. A product with an infinity in it is NaN where the
// fp32 one is infinite, because the infinity also meets the other operand's second plane, of
// either sign or zero. The sum of the first planes' products is infinite or NaN as the fp32 sum is (but
// for values so far below the largest of their scale, 2^-40, that their first plane is 0). So a wave
// that finds NaN among its results takes those from here, on the fragments it has: no other wave
// needs to know.
__device__ __forceinline__ void mfma_rec_first(int c, const uint4& a, const uint4& b, f32x4& acc) {
  const f32x4 hi = mfma_f16_16x16x32(a, b, f32x4{0.f, 0.f, 0.f, 0.f});
  if (c & 1) acc -= hi;
  else acc += hi;
}
__device__ __forceinline__ bool has_nan(const f32x4& v) { return v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3]; }
// Fragments of an odd chunk: the first plane negated.
__device__ __forceinline__ uint4 rec_negated(uint4 v) {
  return uint4{v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u};
}
