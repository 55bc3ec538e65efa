// Reduced-precision products for dense A: P = A H^T and R = A^T W of
// Algorithm 1 on the gfx950 matrix cores with float accumulation, for A
// stored in bfloat16 or in FP8 E4M3. The factors stay float; before each
// product the factor operand is packed, transposed, into the same format
// (round to nearest even): bfloat16 directly; FP8 after dividing each rank
// column by the smallest power of two that brings its largest entry to at
// most 448 (the E4M3 maximum), the power being multiplied back into that
// output column.
//
// Both products are computed as D (M x N, float) = X Y^T with X (M x K) A or
// its transpose, read in A's own layout, and Y (N x K) the packed factor, K
// contiguous. A H^T (NT) has K contiguous in X too: each K step covers one
// 128-byte line of a row, and lane (g = l / 16, c = l % 16) of a wave needs bytes
// 32 g .. 32 g + 31 of row c of each of its row tiles. For FP8 those 32 values
// are the operand of v_mfma_scale_f32_16x16x128_f8f6f4 (lane l: row l % 16, K
// values 32 (l / 16) .. + 31). For bfloat16 they feed two
// v_mfma_f32_16x16x32_bf16 (lane l: row l % 16, eight K values from
// 8 (l / 16)): values 0..7 the first, 8..15 the second; the factor operand
// gets the same K permutation, so the sum is unchanged. The two 16-byte loads
// of a tile read eight whole lines each (lane (g, c): row c % 8, then row
// 8 + c % 8, bytes 32 g + 16 (c / 8)), and lanes c and c + 8 trade halves
// afterwards (unpair): whole lines per instruction read at 7.1 TB/s on this
// card, and halves of sixteen lines at 6.1. 131072 x 65536 at k = 100: FP8
// 1.71 -> 1.39 ms a product, bfloat16 3.35 -> 2.86.
//
// A^T W (TN) has the output side contiguous: for the same K values lane (g, c)
// reads four (or eight, lp_wide) neighbouring columns of each row, one column
// for each of its tiles, and regroups the values of four columns from along the row to along K
// in registers (v_perm_b32: one per two bfloat16 values, one per two FP8
// values). No transposed copy of A is made: at 24000 x 16400 bfloat16 that
// copy took 360 of the call's 569 us, and it held as much memory again as A.
//
// At rank k the product does k (bfloat16) or 2k (FP8) flops per byte of A,
// far below the ridge of either format, so the kernel is built to keep HBM
// busy: A is read once with non-temporal loads, several K steps deep; the
// factor slice of each K step (N rows x 128 bytes) is loaded once per
// workgroup into LDS and shared by its four waves.
#include <type_traits>

#include "common.h"
#include "grid.h"
#include "kernels.h"

namespace nmfk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ i32x8 join32(u32x4 a, u32x4 b) {
  return __builtin_bit_cast(i32x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// bfloat16 bits of x, rounded to nearest even (NaN stays a quiet NaN).
__device__ __forceinline__ uint16_t to_bf16_rne(float x) {
  const unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// FP8 E4M3 bits of x (sign, 4 exponent bits with bias 7, 3 fraction bits;
// largest finite 448, no infinities), rounded to nearest even and saturating
// at 448. |x| is rounded to a multiple of its binade's spacing (2^(e-3) for
// 2^e <= |x| < 2^(e+1), e >= -6, and 2^-9 below 2^-6); the scalings by powers
// of two are exact, so the only rounding is the one to an integer.
__device__ __forceinline__ uint8_t to_fp8_e4m3_rne(float x) {
  const unsigned sgn = (__float_as_uint(x) >> 24) & 0x80u;
  const float a = fabsf(x);
  if (!(a == a)) return 0x7f;
  if (a >= 448.f) return (uint8_t)(sgn | 0x7eu);
  int e = (int)((__float_as_uint(a) >> 23) & 0xffu) - 127;
  e = e < -6 ? -6 : e;
  const float q = rintf(ldexpf(a, 3 - e));     // multiples of 2^(e-3)
  if (q == 0.f) return (uint8_t)sgn;
  if (e == -6 && q < 8.f) return (uint8_t)(sgn | (unsigned)q);  // subnormal: q 2^-9
  // q in [8, 16]: 16 carries into the next binade
  const int qi = (int)q;
  const int ee = qi == 16 ? e + 1 : e;
  const int f = qi == 16 ? 0 : qi - 8;
  return (uint8_t)(sgn | ((unsigned)(ee + 7) << 3) | (unsigned)f);
}

constexpr int SB = 128;        // bytes of each row per K step
constexpr int BWAVES = 4;      // waves per workgroup

template <int MT> struct XFrag { u32x4 v[MT][2]; };

// MT neighbouring elements of a row, at any alignment.
template <typename TE, int MT> struct Run;
template <> struct Run<uint16_t, 4> {
  typedef unsigned V __attribute__((ext_vector_type(2), aligned(2)));
};
template <> struct Run<uint8_t, 4> {
  typedef unsigned V __attribute__((ext_vector_type(1), aligned(1)));
};
template <> struct Run<uint8_t, 8> {
  typedef unsigned V __attribute__((ext_vector_type(2), aligned(1)));
};

// The operands of four tiles from runs of four columns: r[q] is row q of the
// lane's K values (16 rows for bfloat16, 32 for FP8); tile t's operand holds
// column t along K.
__device__ __forceinline__ void regroup(const Run<uint16_t, 4>::V (&r)[16], XFrag<4>& f) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned a = r[8 * h + 2 * i][t >> 1], b = r[8 * h + 2 * i + 1][t >> 1];
        f.v[t][h][i] = __builtin_amdgcn_perm(b, a, (t & 1) ? 0x07060302u : 0x05040100u);
      }
}
// FP8: the operands of tiles 4 H .. 4 H + 3.
template <int H, typename V>
__device__ __forceinline__ void regroup(const V (&r)[32], XFrag<4>& f) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    // bytes (rows 4 q .. 4 q + 3) x (columns 4 H .. 4 H + 3), transposed
    const unsigned a = r[4 * q][H], b = r[4 * q + 1][H], c = r[4 * q + 2][H], d = r[4 * q + 3][H];
    const unsigned ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u);  // a0 b0 a1 b1
    const unsigned ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);  // a2 b2 a3 b3
    const unsigned cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u);
    const unsigned cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    f.v[0][q >> 2][q & 3] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    f.v[1][q >> 2][q & 3] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    f.v[2][q >> 2][q & 3] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
    f.v[3][q >> 2][q & 3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
  }
}

// The operands of MT tiles from row pieces loaded in pairs: x.v[t][h] of lane
// (g, c) is bytes 32 g + 16 (c / 8) of row 8 h + c % 8; the operand's two
// halves are bytes 32 g and 32 g + 16 of row c, so lanes c and c + 8 trade one
// half each (DPP row_ror:8; bank masks 0xC and 0x3 are lanes 8..15 and 0..7).
template <int MT>
__device__ __forceinline__ void unpair(const XFrag<MT>& x, XFrag<MT>& f) {
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = (int)x.v[t][0][i], b = (int)x.v[t][1][i];
      f.v[t][0][i] = (unsigned)__builtin_amdgcn_update_dpp(a, b, 0x128, 0xf, 0xC, false);
      f.v[t][1][i] = (unsigned)__builtin_amdgcn_update_dpp(b, a, 0x128, 0xf, 0x3, false);
    }
}

// TE: stored element (uint16_t bfloat16 bits or uint8_t FP8 E4M3 bits).
// NT 16-column tiles (N = 16 NT), MT 16-row tiles per wave, STAGES K steps of
// X in registers (STAGES - 1 in flight while one is multiplied), WPE waves per
// SIMD to leave room for. FP8 outputs: column j is multiplied by colscale[j].
// TR: X is given as its transpose (K x M, ldx between its rows), M >= MT and
// ldx < TN_MAX_LD, so that a lane's offset within a step fits 32 bits.
constexpr int64_t TN_MAX_LD = (int64_t)1 << 24;
template <typename TE, int NT, bool TR, int MT, int STAGES, int WPE>
__global__ __launch_bounds__(64 * BWAVES, WPE) void gemm_lp_kernel(
    const TE* __restrict__ X, int64_t ldx, const TE* __restrict__ Y, int64_t ldy,
    const float* __restrict__ colscale, float* __restrict__ D, int64_t ldd, int64_t dsplit,
    int64_t M, int64_t K, int64_t kchunk) {
  constexpr bool FP8 = sizeof(TE) == 1;
  constexpr int BK = SB / (int)sizeof(TE);    // K values per step
  constexpr int LE = 32 / (int)sizeof(TE);    // K values per lane per step
  constexpr int VE = 16 / (int)sizeof(TE);    // K values per 16-byte load
  constexpr int YLD = BK + VE;                // LDS row pitch (16 bytes of padding)
  constexpr int NR = 16 * NT;                 // factor rows (the padded rank)
  constexpr int YCH = SB / 16;                // 16-byte chunks per factor row per step
  constexpr int YRP = 256 / YCH;              // factor rows staged per pass
  constexpr int YPASS = (NR + YRP - 1) / YRP;
  // LDS rows NR..YPASS*YRP-1 take the copies of the last pass past the
  // factor's end (their global row is clamped): no branch in the staging.
  __shared__ __attribute__((aligned(16))) TE Ys[2][YPASS * YRP * YLD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int64_t m0 = (int64_t)blockIdx.x * (16 * MT * BWAVES) + wave * 16 * MT;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  D += (int64_t)blockIdx.y * dsplit;

  // TR: columns col0 .. col0 + MT - 1, moved back where they would pass the
  // last one (two lanes then hold, and store, the same column)
  typedef typename Run<TE, TR ? MT : 4>::V RunV;
  const TE* xr[TR ? 1 : MT][2];
  uint32_t xo = 0;   // TR: the lane's offset from the (uniform) step rows
  if constexpr (TR) {
    int64_t col0 = m0 + MT * c;
    col0 = col0 < M - MT ? col0 : M - MT;
    xo = (uint32_t)((int64_t)(LE * g) * ldx + col0);
  } else {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int64_t row = m0 + 16 * t + 8 * h + (c & 7);
        row = row < M ? row : M - 1;
        xr[t][h] = X + row * ldx + LE * g + VE * (c >> 3);
      }
  }
  // factor staging: thread tid copies chunk (tid % YCH) of rows tid / YCH + YRP p
  const int ych = tid % YCH, yrow0 = tid / YCH;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int64_t nfull = (kend - kbeg) / BK;
  // a step's X: the operands (NT), or the runs they are regrouped from (TN)
  struct Runs { RunV r[LE]; };
  typedef typename std::conditional<TR, Runs, XFrag<MT>>::type XStep;
  XStep xf[STAGES];
  u32x4 yv[2][YPASS];  // factor slices of the next two steps, in registers

  auto load_x = [&](XStep& f, int64_t k0) {
    if constexpr (TR) {
#pragma unroll
      for (int u = 0; u < LE; ++u)
        f.r[u] = __builtin_nontemporal_load(
            reinterpret_cast<const RunV*>(X + (k0 + u) * ldx + xo));
    } else {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          f.v[t][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(xr[t][h] + k0));
    }
  };
  auto load_y = [&](u32x4 (&v)[YPASS], int64_t k0) {
#pragma unroll
    for (int p = 0; p < YPASS; ++p) {
      const int r = yrow0 + p * YRP;
      const int rg = r < NR ? r : NR - 1;
      v[p] = *reinterpret_cast<const u32x4*>(Y + (int64_t)rg * ldy + k0 + VE * ych);
    }
  };
  auto store_y = [&](const u32x4 (&v)[YPASS], int buf) {
#pragma unroll
    for (int p = 0; p < YPASS; ++p) {
      const int r = yrow0 + p * YRP;
      *reinterpret_cast<u32x4*>(&Ys[buf][r * YLD + VE * ych]) = v[p];
    }
  };
  // tiles t0 .. of the wave times the slice in buf
  auto multiply = [&](const auto& f, int buf, auto t0) {
    constexpr int T0 = decltype(t0)::value, N = sizeof(f.v) / sizeof(f.v[0]);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const TE* yp = &Ys[buf][(16 * j + c) * YLD + LE * g];
      const u32x4 b0 = *reinterpret_cast<const u32x4*>(yp);
      const u32x4 b1 = *reinterpret_cast<const u32x4*>(yp + VE);
#pragma unroll
      for (int t = 0; t < N; ++t) {
        if constexpr (FP8) {
          // operand formats 0 (E4M3) and no block scales: a plain FP8 product
          acc[T0 + t][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              join32(f.v[t][0], f.v[t][1]), join32(b0, b1), acc[T0 + t][j], 0, 0, 0, 0, 0, 0);
        } else {
          acc[T0 + t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f.v[t][0]),
                                                              as_bf16x8(b0), acc[T0 + t][j], 0, 0, 0);
          acc[T0 + t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(f.v[t][1]),
                                                              as_bf16x8(b1), acc[T0 + t][j], 0, 0, 0);
        }
      }
    }
  };

  typedef std::integral_constant<int, 0> First;
  typedef std::integral_constant<int, 4> Second;
  auto compute = [&](const XStep& x, int buf) {
    if constexpr (TR) {
      XFrag<4> f;
      if constexpr (FP8) regroup<0>(x.r, f);
      else regroup(x.r, f);
      multiply(f, buf, First{});
      if constexpr (MT == 8) {
        regroup<1>(x.r, f);
        multiply(f, buf, Second{});
      }
    } else {
      XFrag<MT> f;
      unpair(x, f);
      multiply(f, buf, First{});
    }
  };

  // Memory loads complete in issue order as far as the wait counter is
  // concerned, so each step issues the factor slice it will need two steps
  // later before the matrix rows it will need STAGES - 1 steps later: the
  // slice written to LDS at the end of a step was issued a full step earlier,
  // ahead of the newest row loads, and waiting for it leaves those in flight.
  static_assert(STAGES % 2 == 0, "the unrolled ring also indexes the two factor slices");
  if (nfull > 0) {
    load_y(yv[0], kbeg);
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nfull) load_x(xf[s], kbeg + s * BK);
    if (nfull > 1) load_y(yv[1], kbeg + BK);
    store_y(yv[0], 0);
    __syncthreads();
    // Steady state: every prefetch is in range, so the unrolled body has no
    // branch between a load and its use and the wait counts stay exact.
    // STAGES is even, so ring and buffer indices are constants.
    constexpr int AHEAD = STAGES - 1 > 2 ? STAGES - 1 : 2;
    int64_t s = 0;
    for (; s + STAGES + AHEAD <= nfull; s += STAGES) {
#pragma unroll
      for (int u = 0; u < STAGES; ++u) {
        const int64_t st = s + u;
        load_y(yv[u & 1], kbeg + (st + 2) * BK);
        load_x(xf[(u + STAGES - 1) % STAGES], kbeg + (st + STAGES - 1) * BK);
        // keep the prefetches ahead of this step's matrix-core work
        __builtin_amdgcn_sched_barrier(0);
        compute(xf[u], u & 1);
        store_y(yv[(u + 1) & 1], (u + 1) & 1);
        __syncthreads();
      }
    }
    // Drain: the last steps, with the loads past the end skipped.
    for (; s < nfull; s += STAGES) {
#pragma unroll
      for (int u = 0; u < STAGES; ++u) {
        const int64_t st = s + u;
        if (st < nfull) {
          if (st + 2 < nfull) load_y(yv[u & 1], kbeg + (st + 2) * BK);
          const int64_t pre = st + STAGES - 1;
          if (pre < nfull) load_x(xf[(u + STAGES - 1) % STAGES], kbeg + pre * BK);
          compute(xf[u], u & 1);
          if (st + 1 < nfull) store_y(yv[(u + 1) & 1], (u + 1) & 1);
          __syncthreads();
        }
      }
    }
  }
  // K tail (fewer than BK values left): element loads, zero beyond kend
  const int64_t kt = kbeg + nfull * BK;
  if (kt < kend) {
    XFrag<MT> f;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      TE e[LE];
      const int64_t row = m0 + 16 * t + c;
      const TE* xt = X + (row < M ? row : M - 1) * ldx + LE * g;
#pragma unroll
      for (int q = 0; q < LE; ++q) {
        const bool in = kt + LE * g + q < kend;
        if constexpr (TR) e[q] = in ? X[(kt + q) * ldx + xo + t] : (TE)0;
        else e[q] = in ? xt[kt + q] : (TE)0;
      }
      u32x4 w[2];
      __builtin_memcpy(w, e, sizeof(w));
      f.v[t][0] = w[0];
      f.v[t][1] = w[1];
    }
    for (int e = tid; e < NR * BK; e += 64 * BWAVES) {
      const int r = e / BK, kk = e % BK;
      Ys[0][r * YLD + kk] = (kt + kk < kend) ? Y[(int64_t)r * ldy + kt + kk] : (TE)0;
    }
    __syncthreads();
    multiply(f, 0, First{});
  }
  // store: element r of tile (t, j) is row 4 g + r, column c
  float cs[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) cs[j] = FP8 ? colscale[16 * j + c] : 1.f;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int64_t row = TR ? m0 + MT * (4 * g + r) : m0 + 16 * t + 4 * g + r;
      bool in = row < M;
      if constexpr (TR) {
        row = (row < M - MT ? row : M - MT) + t;
        in = m0 < M;
      }
      if (in) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
          D[row * ldd + 16 * j + c] = FP8 ? acc[t][j][r] * cs[j] : acc[t][j][r];
      }
    }
}

// Ft (KP x rows, row pitch ldt) = bfloat16(F^T) for F rows x KP float.
__global__ __launch_bounds__(256) void pack_bf16_t_kernel(const float* __restrict__ F,
                                                         int64_t rows, int KP,
                                                         uint16_t* __restrict__ Ft, int64_t ldt) {
  __shared__ float tile[32][33];
  const int64_t r0 = (int64_t)blockIdx.x * 32;
  const int c0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8) {
    const int64_t r = r0 + i;
    const int cc = c0 + tx;
    tile[i][tx] = (r < rows && cc < KP) ? F[r * KP + cc] : 0.f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int cc = c0 + i;
    const int64_t r = r0 + tx;
    if (cc < KP && r < rows) Ft[(int64_t)cc * ldt + r] = to_bf16_rne(tile[tx][i]);
  }
}

// FP8 packing, pass 1: maxbits[j] = bits of max_r |F[r][j]| (non-negative
// floats order like their bit patterns), KP a multiple of 4 up to 128;
// maxbits starts at 0. Thread (ty, c) of a block reads 16-byte chunks c of
// rows ty, ty + R, ... of the block's slices (R = 256 / (KP / 4) rows per
// pass, four passes in flight), the block reduces its maxima in LDS and
// raises each column's word once.
__global__ __launch_bounds__(256) void colmax_kernel(const float* __restrict__ F, int64_t rows,
                                                     int KP, unsigned* __restrict__ maxbits) {
  __shared__ unsigned part[256 * 4];
  const int q = KP / 4;           // float4 chunks per row
  const int R = 256 / q;          // rows per pass
  const int tid = threadIdx.x;
  const int c = tid % q, ty = tid / q;
  unsigned mx[4] = {0u, 0u, 0u, 0u};
  if (ty < R) {
    const int64_t stride = (int64_t)gridDim.x * R;
    for (int64_t r0 = (int64_t)blockIdx.x * R + ty; r0 < rows; r0 += 4 * stride) {
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t r = r0 + u * stride;
        v[u] = r < rows ? *reinterpret_cast<const f32x4*>(F + r * KP + 4 * c)
                        : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx[e] = max(mx[e], __float_as_uint(fabsf(v[u][e])));
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[tid * 4 + e] = mx[e];
  __syncthreads();
  if (tid < KP) {
    // column tid is element tid % 4 of chunk tid / 4, held by threads ty q + tid / 4
    unsigned m = 0;
    for (int t = 0; t < R; ++t) m = max(m, part[(t * q + tid / 4) * 4 + tid % 4]);
    if (m) atomicMax(&maxbits[tid], m);
  }
}

__global__ void zero_u32_kernel(unsigned* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Exponent p of the column scale 2^p: the smallest integer with
// 448 2^p >= mx (0 for mx = 0). With mx = f 2^E, f in [0.5, 1), and
// 448 = 0.875 2^9: p = E - 9 if f <= 0.875, else E - 8. No rounding.
__device__ __forceinline__ int fp8_col_exp(unsigned maxbits) {
  const float mx = __uint_as_float(maxbits);
  if (!(mx > 0.f)) return 0;
  int E;
  const float f = frexpf(mx, &E);
  return f <= 0.875f ? E - 9 : E - 8;
}

// Pass 2: Ft (KP x rows, pitch ldt) = FP8(F^T / 2^p_j), colscale[j] = 2^p_j.
__global__ __launch_bounds__(256) void pack_fp8_t_kernel(const float* __restrict__ F,
                                                        int64_t rows, int KP,
                                                        const unsigned* __restrict__ maxbits,
                                                        uint8_t* __restrict__ Ft, int64_t ldt,
                                                        float* __restrict__ colscale) {
  __shared__ float tile[32][33];
  const int64_t r0 = (int64_t)blockIdx.x * 32;
  const int c0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8) {
    const int64_t r = r0 + i;
    const int cc = c0 + tx;
    tile[i][tx] = (r < rows && cc < KP) ? F[r * KP + cc] : 0.f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int cc = c0 + i;
    const int64_t r = r0 + tx;
    if (cc < KP && r < rows)
      Ft[(int64_t)cc * ldt + r] = to_fp8_e4m3_rne(ldexpf(tile[tx][i], -fp8_col_exp(maxbits[cc])));
  }
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int j = threadIdx.x; j < KP; j += blockDim.x)
      colscale[j] = ldexpf(1.f, fp8_col_exp(maxbits[j]));
}

hipError_t pack_bf16_t(const float* F, int64_t rows, int KP, uint16_t* Ft, int64_t ldt,
                       hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  dim3 grid((unsigned)cdiv(rows, 32), (unsigned)cdiv(KP, 32));
  pack_bf16_t_kernel<<<grid, 256, 0, st>>>(F, rows, KP, Ft, ldt);
  return NMF_LAUNCH_CHECK();
}

hipError_t pack_fp8_t(const float* F, int64_t rows, int KP, uint8_t* Ft, int64_t ldt,
                      float* colscale, unsigned* maxbits, hipStream_t st) {
  if (KP < 4 || KP > 128 || KP % 4 != 0) return hipErrorInvalidValue;
  zero_u32_kernel<<<1, 128, 0, st>>>(maxbits, KP);
  if (rows > 0) {
    const int R = 256 / (KP / 4);
    const int64_t want = cdiv(rows, 4 * R), blocks = want < 1024 ? want : 1024;
    colmax_kernel<<<(unsigned)blocks, 256, 0, st>>>(F, rows, KP, maxbits);
    dim3 grid((unsigned)cdiv(rows, 32), (unsigned)cdiv(KP, 32));
    pack_fp8_t_kernel<<<grid, 256, 0, st>>>(F, rows, KP, maxbits, Ft, ldt, colscale);
  }
  return NMF_LAUNCH_CHECK();
}

constexpr int B_MT = 4, B_STAGES = 4, B_WPE = 1;  // launch shape (timing sweep at 131072 x 65536, k = 100)
// FP8 A^T W: eight columns a lane, so that a load takes whole lines of A (a
// wave of four columns a lane reads 64 bytes of a row), and two stages (a
// stage holds twice the bytes). 131072 x 65536 at k = 50: 1807 -> 1320 us, 24000 x
// 16400 176 -> 131. The accumulators are twice as many too: from 96 columns on
// they spill (k = 100: 1990 us with four columns a lane, 2228 with eight), and
// a small A has too few workgroups of 512 columns.
static bool lp_wide(bool tn, int esize, int64_t M, int N, int64_t K) {
  return tn && esize == 1 && N <= 80 && M >= 512 && M * K >= ((int64_t)1 << 28);
}

// One workgroup per CU and round, slabs of at least 1024, at most 2^21 rows of
// them (1 GB at the largest rank). A slab's cost is taken at rank 64 and
// bfloat16. bfloat16, 24000 x 16400 at k = 50, A^T W: 7 slabs for 4, 240 -> 199 us;
// 100000 x 4800 249 -> 180; 20000^2 at k = 100 274 -> 200 and A H^T 295 -> 220 (FP8
// 222 -> 168 and 205 -> 162).
int64_t gemm_lp_splits(bool tn, int esize, int64_t M, int N, int64_t K) {
  const bool wide = lp_wide(tn, esize, M, N, K);
  const int64_t blocks = cdiv(M, 16 * (wide ? 8 : B_MT) * BWAVES);
  int64_t s = 1;
  while (blocks * s < 256 && K / (2 * s) >= 1024 && s < (wide ? 32 : 16)) s *= 2;
  return full_rounds(blocks, s, 256, 256.0 / (double)K, [&](int64_t t) {
    return t == 1 || (K / t >= 1024 && t <= 32 && (t <= s || t * M <= ((int64_t)1 << 21)));
  });
}

bool gemm_lp_reads_a(int64_t M, int64_t ldx) { return M >= 4 && ldx < TN_MAX_LD; }

template <typename TE>
static hipError_t gemm_lp(bool tn, const TE* X, int64_t ldx, const TE* Y, int64_t ldy,
                          const float* colscale, float* D, int64_t ldd, int64_t M, int N,
                          int64_t K, float* part, hipStream_t st) {
  constexpr int VE = 16 / (int)sizeof(TE);
  constexpr int BK = SB / (int)sizeof(TE);
  if (M <= 0) return hipSuccess;
  if (N % 16 != 0 || N < 16 || N > 128 || ldx % VE != 0 || ldy % VE != 0 || (tn && !gemm_lp_reads_a(M, ldx)))
    return hipErrorInvalidValue;
  const bool wide = lp_wide(tn, sizeof(TE), M, N, K);
  const int64_t splits = gemm_lp_splits(tn, sizeof(TE), M, N, K);
  const int64_t kchunk = round_up(cdiv(K, splits), BK);
  const int64_t nsplit = cdiv(K, kchunk);
  float* out = nsplit > 1 ? part : D;
  const int64_t ldo = nsplit > 1 ? N : ldd;
  const int64_t dsplit = (int64_t)M * N;
  dim3 grid((unsigned)cdiv(M, 16 * (wide ? 8 : B_MT) * BWAVES), (unsigned)nsplit);
  const int NT = N / 16;
#define CASE(J)                                                                            \
  case J:                                                                                  \
    if constexpr (sizeof(TE) == 1 && J <= 5)                                               \
      if (wide) {                                                                          \
        gemm_lp_kernel<TE, J, true, 8, 2, B_WPE><<<grid, 64 * BWAVES, 0, st>>>(            \
            X, ldx, Y, ldy, colscale, out, ldo, dsplit, M, K, kchunk);                     \
        break;                                                                             \
      }                                                                                    \
    if (tn)                                                                                \
      gemm_lp_kernel<TE, J, true, B_MT, B_STAGES, B_WPE><<<grid, 64 * BWAVES, 0, st>>>(    \
          X, ldx, Y, ldy, colscale, out, ldo, dsplit, M, K, kchunk);                       \
    else                                                                                   \
      gemm_lp_kernel<TE, J, false, B_MT, B_STAGES, B_WPE><<<grid, 64 * BWAVES, 0, st>>>(   \
          X, ldx, Y, ldy, colscale, out, ldo, dsplit, M, K, kchunk);                       \
    break;
  switch (NT) {
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef CASE
  hipError_t e = NMF_LAUNCH_CHECK();
  if (e != hipSuccess || nsplit == 1) return e;
  return reduce_splits<float>(part, (int)nsplit, dsplit, M, N, ldd, D, N, st);
}

hipError_t gemm_bf16(bool tn, const uint16_t* X, int64_t ldx, const uint16_t* Y, int64_t ldy,
                     float* D, int64_t ldd, int64_t M, int N, int64_t K, float* part,
                     hipStream_t st) {
  return gemm_lp<uint16_t>(tn, X, ldx, Y, ldy, nullptr, D, ldd, M, N, K, part, st);
}

hipError_t gemm_fp8(bool tn, const uint8_t* X, int64_t ldx, const uint8_t* Y, int64_t ldy,
                    const float* colscale, float* D, int64_t ldd, int64_t M, int N, int64_t K,
                    float* part, hipStream_t st) {
  if (!colscale) return hipErrorInvalidValue;
  return gemm_lp<uint8_t>(tn, X, ldx, Y, ldy, colscale, D, ldd, M, N, K, part, st);
}

}  // namespace nmfk
