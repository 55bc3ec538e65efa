// Float operands of the bfloat16 matrix cores: splitting in registers and the
// six-term product (see gemm.hip for its accuracy).
#pragma once

#include "split.h"

namespace nmfk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Eight floats (scaled by SPLIT_SCALE) as three bfloat16 operand registers.
struct Split8 { u32x4 h, m, l; };

__device__ __forceinline__ void split2(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  x0 *= SPLIT_SCALE;
  x1 *= SPLIT_SCALE;
  h = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{x0, x1}, bf16x2));
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{r0, r1}, bf16x2));
  const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
  l = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{s0, s1}, bf16x2));
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  Split8 s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    unsigned h, m, l;
    split2(x[2 * i], x[2 * i + 1], h, m, l);
    s.h[i] = h;
    s.m[i] = m;
    s.l[i] = l;
  }
  return s;
}

// acc[j] += the product of a with b[j] (SPLIT_UNSCALE of it is the result),
// smallest terms first.
template <int N>
__device__ __forceinline__ void split_mma(const Split8& a, const Split8 (&b)[N], f32x4 (&acc)[N]) {
#define TERM(PA, PB) \
  _Pragma("unroll") for (int j = 0; j < N; ++j) acc[j] = mfma_bf16(a.PA, b[j].PB, acc[j]);
  TERM(l, h) TERM(h, l) TERM(m, m) TERM(m, h) TERM(h, m) TERM(h, h)
#undef TERM
}

}  // namespace nmfk
