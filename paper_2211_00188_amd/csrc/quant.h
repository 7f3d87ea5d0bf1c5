// Arithmetic of the b-bit stochastic quantiser shared by the kernels: the Philox dither, the quotient
// |v| / a, the code and the decoded magnitude of one coordinate.
#pragma once
#include "devutil.h"

namespace adacgd {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): counter (c0..c3), key (k0,k1) -> 4 words
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// dither u in [0,1) of coordinate l: word l%4 of the block l/4, top 24 bits
__device__ __forceinline__ float dither_of(uint32_t word) { return (float)(word >> 8) * 5.9604644775390625e-8f; }

// b-bit stochastic quantiser of one coordinate from t = fl(|v| / a): the magnitude code xi (as a float) and
// the decoded magnitude fl(xi c).  s = magnitude levels, c = fl(a / (s (1+omega))).
__device__ __forceinline__ float quant_mag(float t, float s, float c, float u, float* xi_out) {
  const float r = t * s;              // the second of the two rounded fp32 operations
  const float fl = floorf(r);
  const float pfrac = r - fl;
  const float xi = fl + ((u < pfrac) ? 1.f : 0.f);
  *xi_out = xi;
  return xi * c;
}

// ... with the sign of v: returns the signed code and the decoded value.
__device__ __forceinline__ float quant_ratio(float v, float t, float s, float c, float u, int* code) {
  float xi;
  const float mag = quant_mag(t, s, c, u, &xi);
  *code = (__float_as_uint(v) >> 31) ? -(int)xi : (int)xi;
  return copysignf(mag, v);
}

// The same with a = max |v| (> 0) given.
__device__ __forceinline__ float quant_one(float v, float a, float s, float c, float u, int* code) {
  return quant_ratio(v, fabsf(v) / a, s, c, u, code);
}

}  // namespace adacgd
