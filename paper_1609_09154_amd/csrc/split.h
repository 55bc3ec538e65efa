// Floats as exact sums of three bfloat16 values, and the packed layout in
// which the dense products (gemm.hip) read their factor operand.
#pragma once

#include "common.h"

namespace nmfk {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Operands are split after scaling by 2^16, and their products scaled back by
// 2^-32 (both exact): the last bit of any float, 2^-149 at the least, is then a
// whole multiple of the smallest bfloat16 (2^-133), so that no split loses bits,
// however small the entry. Unscaled, entries below 2^-110 did: with a factor
// near 2^-122 and A near 2^40 a product was off by 1e-5.
constexpr float SPLIT_SCALE = 65536.f, SPLIT_UNSCALE = 1.f / 4294967296.f;

// 2^16 x = h + m + l (bits of three bfloat16 values) for every x of magnitude
// below 2^111: h is 2^16 x rounded to nearest even (cut off instead where
// rounding would overflow), m the remainder rounded, l the rest. Larger
// entries, infinities and NaN have h infinite or NaN and m = l = 0.
__device__ __forceinline__ void split_bf16x3(float x, unsigned& h, unsigned& m, unsigned& l) {
  x *= SPLIT_SCALE;
  const unsigned u = __float_as_uint(x), a = u & 0x7fffffffu;
  unsigned hh = u + 0x7fffu + ((u >> 16) & 1u);
  if (a >= 0x7f7f8000u) hh = a > 0x7f800000u ? u | 0x400000u : u;
  hh &= 0xffff0000u;
  const float r = a < 0x7f800000u ? x - __uint_as_float(hh) : 0.f;
  const unsigned ur = __float_as_uint(r), mm = (ur + 0x7fffu + ((ur >> 16) & 1u)) & 0xffff0000u;
  const unsigned uq = __float_as_uint(r - __uint_as_float(mm));
  h = hh >> 16;
  m = mm >> 16;
  l = (uq + 0x7fffu + ((uq >> 16) & 1u)) >> 16;
}

// Packed factor (rows x KP floats): for each group of 8 rows, plane h, then m,
// then l, each KP chunks (one per column) of the 8 rows' values, 16 bytes a
// chunk. Rows are padded with zeros to a multiple of 32 (one product step).
__host__ __device__ inline int64_t split_groups(int64_t rows) { return cdiv(rows, 32) * 4; }

// The chunks of column i of group k8 from its 8 values.
__device__ __forceinline__ void store_split_chunk(const float (&x)[8], int64_t k8, int KP, int i,
                                                  u32x4* __restrict__ out) {
  u32x4 w[3];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    unsigned a[3], b[3];
    split_bf16x3(x[2 * v], a[0], a[1], a[2]);
    split_bf16x3(x[2 * v + 1], b[0], b[1], b[2]);
#pragma unroll
    for (int p = 0; p < 3; ++p) w[p][v] = a[p] | b[p] << 16;
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) out[(k8 * 3 + p) * KP + i] = w[p];
}

}  // namespace nmfk
