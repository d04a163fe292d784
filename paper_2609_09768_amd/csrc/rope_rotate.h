// Rotation of cached keys to their new positions, in float64 and rounded once
// to bfloat16 (device side only): shared by the adjustment kernel, whose file
// says why it rounds as it does, and by the check layer's fused adjustment
// and deviation.
#pragma once

#include "bf16_util.h"

namespace kvc {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two float32 values to packed bfloat16, nearest with ties to even.
__device__ __forceinline__ uint32_t pack_bf16_rne(uint32_t a, uint32_t b) {
  const f32x2_t v = {__uint_as_float(a), __uint_as_float(b)};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// float32 bits on a bfloat16 midpoint (low 16 bits 0x8000)
__device__ __forceinline__ bool on_midpoint(uint32_t f) { return (f & 0xFFFFu) == 0x8000u; }

// Move a float32 that sits on a bfloat16 midpoint one unit towards the
// float64 value r it was rounded from (nothing if it equals r).
__device__ __forceinline__ uint32_t off_midpoint(uint32_t f, double r) {
  if (!on_midpoint(f)) return f;
  const double d = (double)__uint_as_float(f);
  if (d == r) return f;
  return fabs(d) > fabs(r) ? f - 1u : f + 1u;  // magnitude down or up, sign kept
}

// Rotates the 8 pairs of a unit and rounds them, 4 pairs at a time: fewer
// live registers, so that with one tile per workgroup (no loop) the kernel
// fits 96 registers and five waves per SIMD instead of four (2-3 % faster
// on cold buffers).
__device__ __forceinline__ void rotate8(const uint4& a, const uint4& b, const double* c,
                                        const double* s, uint4& oa, uint4& ob) {
  uint32_t pa[4], pb[4];
#pragma unroll
  for (int g0 = 0; g0 < 8; g0 += 4) {
    double ra[4], rb[4];
    uint32_t fa[4], fb[4];
    int mid = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = g0 + i;
      const double x = (double)bf16x8_elem(a, e);
      const double y = (double)bf16x8_elem(b, e);
      ra[i] = fma(x, c[e], -(y * s[e]));
      rb[i] = fma(y, c[e], x * s[e]);
      fa[i] = __float_as_uint((float)ra[i]);
      fb[i] = __float_as_uint((float)rb[i]);
      mid |= (int)on_midpoint(fa[i]) | (int)on_midpoint(fb[i]);
    }
    if (__builtin_expect(mid, 0)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        fa[i] = off_midpoint(fa[i], ra[i]);
        fb[i] = off_midpoint(fb[i], rb[i]);
      }
    }
    pa[g0 / 2] = pack_bf16_rne(fa[0], fa[1]);
    pa[g0 / 2 + 1] = pack_bf16_rne(fa[2], fa[3]);
    pb[g0 / 2] = pack_bf16_rne(fb[0], fb[1]);
    pb[g0 / 2 + 1] = pack_bf16_rne(fb[2], fb[3]);
  }
  oa = make_uint4(pa[0], pa[1], pa[2], pa[3]);
  ob = make_uint4(pb[0], pb[1], pb[2], pb[3]);
}

}  // namespace kvc
