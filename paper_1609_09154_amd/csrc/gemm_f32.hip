// Float products of Algorithm 1 with the matrix cores' float instruction
// (MFMA 16x16x4 and 4x4x1), for padded ranks up to 64:
//
//   NN:  D (M x N) = X (M x K) Y        X = A, Y = H^T
//   TN:  D (M x N) = X^T Y, X (K x M)   X = A, Y = W; or X = A^T, Y = H^T
//
// Most float products take gemm.hip's bfloat16 splits, which are faster on large
// matrices. These are for small ones of whole waves at low rank (f32_sums in
// api.hip says where), and for the forward pass of the unrolled float HALS
// layer at every size, where what counts is the order of the sums: the layer's gradient
// jumps where an entry of the sweep passes zero (its mask is x > 0), so two
// forward passes that differ in the last bit give gradients that agree to
// 1e-7 on most inputs and to 1e-3 where one entry of a few thousand lies on
// the other side. A layer's results therefore keep the sums that its forward
// pass has always had, bit for bit: the slab counts, the order of K within a
// lane, the guarded order of a ragged wave and the separate tile of a rank
// remainder below are part of what it returns.
//
// A wave owns MW 16-row tiles of the streamed side and all rank tiles, so
// every entry of A is loaded once, by one lane; the rank side is read through
// the L2. What bounds them is the float instruction: 8192 x 4096 at k = 64
// takes 47 us a product (92 TFLOP/s of the 157 that it peaks at) where the
// splits take 32.
//
// Rank remainder (NR = 1): when k exceeds a multiple of 16 by at most 4
// (k = 50 = 3 * 16 + 2), the last four columns are computed with the 4x4x1
// instruction instead of a fourth 16-wide tile. The A operand's register is
// read as sixteen 4-row blocks (block b = lane / 4: lane group b / 4 fixes the
// K index, b % 4 the four rows), each multiplied by the remainder columns of
// its own K index; the four lane groups' blocks are summed at the end with two
// cross-lane adds. Columns past 16 NT + 4 are written as zeros.
#include "common.h"
#include "kernels.h"
#include "pipeline.h"

namespace nmfk {

// 16 independent 4x4 blocks, k = 1: block b = l / 4 takes A_b[i] from lane
// 4b + i and B_b[j] from lane 4b + j; lane 4b + j holds D_b[r][j] in element r.
__device__ __forceinline__ f32x4 mfma4x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// A step's operands: X and Y of the MW and NT tiles, and the remainder columns
// (yr, NR = 1).
template <int NT, int MW> struct FragF32 {
  float x[4][MW];
  float y[4][NT];
  float yr[4];
};

// acc += X Y over the four K values of a lane.
#define F32_COMPUTE(F)                                                          \
  {                                                                             \
    _Pragma("unroll") for (int u = 0; u < 4; ++u)                               \
      _Pragma("unroll") for (int t = 0; t < MW; ++t) {                          \
        _Pragma("unroll") for (int nt = 0; nt < NT; ++nt)                       \
          acc[t][nt] = mfma16(F.x[u][t], F.y[u][nt], acc[t][nt]);               \
        if constexpr (NR) accr[t] = mfma4x4(F.x[u][t], F.yr[u], accr[t]);       \
      }                                                                         \
  }
// The rank side's four K values from K0 + 4 g: one 16-byte load a column from
// its transpose (YT), else four elements.
#define F32_LOAD_Y(DST, COL, K0)                                                \
  {                                                                             \
    if constexpr (YT) {                                                         \
      const V16<float> t_ = load16<float>(Y + (int64_t)(COL) * ldy + (K0) + 4 * g); \
      _Pragma("unroll") for (int u = 0; u < 4; ++u) DST(u) = t_.v[u];           \
    } else {                                                                    \
      _Pragma("unroll") for (int u = 0; u < 4; ++u)                             \
        DST(u) = Y[((K0) + 4 * g + u) * ldy + (COL)];                           \
    }                                                                           \
  }

// The remainder columns of the four lane groups (different K), summed; lanes
// 0..15 then hold rows 4 (lane / 4) + r of column cr.
#define F32_STORE_REM(ROW)                                                      \
  _Pragma("unroll") for (int t = 0; t < MW; ++t)                                \
    _Pragma("unroll") for (int r = 0; r < 4; ++r) {                             \
      float v = accr[t][r];                                                     \
      v += __shfl_xor(v, 16, 64);                                               \
      v += __shfl_xor(v, 32, 64);                                               \
      const int64_t row = ROW(t, 4 * (lane >> 2) + r);                          \
      if (g == 0 && row < M) {                                                  \
        Dp[row * ldd + cr] = v;                                                 \
        for (int z = 16 * NT + 4 + (lane & 3); z < ncols; z += 4) Dp[row * ldd + z] = 0.f; \
      }                                                                         \
    }

template <int NT, int MW, bool VX, bool YT, int STAGES, int WPE, int NR>
__global__ __launch_bounds__(256, WPE) void gemm_nn_f32_kernel(
    const float* __restrict__ X, int64_t ldx, const float* __restrict__ Y, int64_t ldy,
    float* __restrict__ D, int64_t ldd, int64_t dsplit, int64_t M, int64_t K, int64_t kchunk,
    int ncols) {
  constexpr int KSTEP = 16;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int64_t m0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (16 * MW);
  if (m0 >= M) return;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  const float* xr[MW];
#pragma unroll
  for (int t = 0; t < MW; ++t) {
    int64_t row = m0 + 16 * t + c;
    row = row < M ? row : M - 1;
    xr[t] = X + row * ldx;
  }
  f32x4 acc[MW][NT], accr[MW];
  const int cr = 16 * NT + (lane & 3);  // remainder column fed by this lane
#pragma unroll
  for (int t = 0; t < MW; ++t) {
    accr[t] = zero4<float>();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[t][nt] = zero4<float>();
  }
  FragF32<NT, MW> fr[STAGES];

#define NN_LOAD(F, K0)                                                          \
  {                                                                             \
    _Pragma("unroll") for (int t = 0; t < MW; ++t) {                            \
      if constexpr (VX) {                                                       \
        const V16<float> t_ = load16_stream<float>(xr[t] + (K0) + 4 * g);       \
        _Pragma("unroll") for (int u = 0; u < 4; ++u) F.x[u][t] = t_.v[u];      \
      } else {                                                                  \
        _Pragma("unroll") for (int u = 0; u < 4; ++u) F.x[u][t] = xr[t][(K0) + 4 * g + u]; \
      }                                                                         \
    }                                                                           \
    _Pragma("unroll") for (int nt = 0; nt < NT; ++nt) {                         \
      auto y_ = [&](int u) -> float& { return F.y[u][nt]; };                    \
      F32_LOAD_Y(y_, 16 * nt + c, K0)                                           \
    }                                                                           \
    if constexpr (NR) {                                                         \
      auto y_ = [&](int u) -> float& { return F.yr[u]; };                       \
      F32_LOAD_Y(y_, cr, K0)                                                    \
    }                                                                           \
  }
  const int64_t nsteps = (kend - kbeg) / KSTEP;
  NMF_PIPELINE(STAGES, NN_LOAD, F32_COMPUTE, fr, kbeg, nsteps, KSTEP)
#undef NN_LOAD

  const int64_t ktail = kbeg + nsteps * KSTEP;
  if (ktail < kend) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t kk = ktail + 4 * g + u;
      const bool ok = kk < kend;
#pragma unroll
      for (int t = 0; t < MW; ++t) fr[0].x[u][t] = ok ? xr[t][kk] : 0.f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        fr[0].y[u][nt] = ok ? (YT ? Y[(int64_t)(16 * nt + c) * ldy + kk] : Y[kk * ldy + 16 * nt + c])
                            : 0.f;
      if constexpr (NR) fr[0].yr[u] = ok ? (YT ? Y[(int64_t)cr * ldy + kk] : Y[kk * ldy + cr]) : 0.f;
    }
    F32_COMPUTE(fr[0]);
  }

  float* Dp = D + (int64_t)blockIdx.y * dsplit;
#pragma unroll
  for (int t = 0; t < MW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = m0 + 16 * t + acc_row<float>(lane, r);
      if (row < M) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) Dp[row * ldd + 16 * nt + c] = acc[t][nt][r];
      }
    }
  if constexpr (NR) {
#define NN_ROW(T, I) (m0 + 16 * (T) + (I))
    F32_STORE_REM(NN_ROW)
#undef NN_ROW
  }
}

// Column of X that lane column c feeds into M-tile t. VX: tile t takes columns
// m0 + 64 (t / 4) + 4 c + t % 4 (one 16-byte load per lane covers four tiles);
// else m0 + 16 t + c.
template <bool VX> __device__ __forceinline__ int64_t tn_col_f32(int64_t m0, int t, int c) {
  if constexpr (VX) return m0 + 64 * (t / 4) + 4 * c + (t % 4);
  else return m0 + 16 * t + c;
}

// One pipeline step covers 16 rows of X: lane group g supplies rows k0 + 4g + u
// to product u (u = 0..3). A wave whose columns run past M takes all of its
// rows in the guarded loop, four at a time.
template <int NT, int MW, bool VX, bool YT, int STAGES, int WPE, int NR>
__global__ __launch_bounds__(256, WPE) void gemm_tn_f32_kernel(
    const float* __restrict__ X, int64_t ldx, const float* __restrict__ Y, int64_t ldy,
    float* __restrict__ D, int64_t ldd, int64_t dsplit, int64_t M, int64_t K, int64_t kchunk,
    int ncols) {
  constexpr int KSTEP = 16;
  static_assert(MW % 4 == 0, "16-byte loads cover four tiles");
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int64_t m0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (16 * MW);
  if (m0 >= M) return;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  const bool full = m0 + 16 * MW <= M;
  f32x4 acc[MW][NT], accr[MW];
  const int cr = 16 * NT + (lane & 3);  // remainder column fed by this lane
#pragma unroll
  for (int t = 0; t < MW; ++t) {
    accr[t] = zero4<float>();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[t][nt] = zero4<float>();
  }
  FragF32<NT, MW> fr[STAGES];

#define TN_LOAD(F, K0)                                                          \
  {                                                                             \
    _Pragma("unroll") for (int u = 0; u < 4; ++u) {                             \
      const float* xrow = X + ((K0) + 4 * g + u) * ldx;                         \
      if constexpr (VX) {                                                       \
        _Pragma("unroll") for (int q = 0; q < MW / 4; ++q) {                    \
          const V16<float> t_ = load16_stream<float>(xrow + m0 + 64 * q + 4 * c); \
          _Pragma("unroll") for (int v = 0; v < 4; ++v) F.x[u][q * 4 + v] = t_.v[v]; \
        }                                                                       \
      } else {                                                                  \
        _Pragma("unroll") for (int t = 0; t < MW; ++t) F.x[u][t] = xrow[m0 + 16 * t + c]; \
      }                                                                         \
    }                                                                           \
    _Pragma("unroll") for (int nt = 0; nt < NT; ++nt) {                         \
      auto y_ = [&](int u) -> float& { return F.y[u][nt]; };                    \
      F32_LOAD_Y(y_, 16 * nt + c, K0)                                           \
    }                                                                           \
    if constexpr (NR) {                                                         \
      auto y_ = [&](int u) -> float& { return F.yr[u]; };                       \
      F32_LOAD_Y(y_, cr, K0)                                                    \
    }                                                                           \
  }
  const int64_t nsteps = full ? (kend - kbeg) / KSTEP : 0;
  NMF_PIPELINE(STAGES, TN_LOAD, F32_COMPUTE, fr, kbeg, nsteps, KSTEP)
#undef TN_LOAD

  for (int64_t k0 = kbeg + nsteps * KSTEP; k0 < kend; k0 += 4) {
    const int64_t kk = k0 + g;
    const bool okk = kk < kend;
    const int64_t kc = okk ? kk : kbeg;
#pragma unroll
    for (int t = 0; t < MW; ++t) {
      const int64_t col = tn_col_f32<VX>(m0, t, c);
      fr[0].x[0][t] = (okk && col < M) ? X[kc * ldx + col] : 0.f;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      fr[0].y[0][nt] = okk ? (YT ? Y[(int64_t)(16 * nt + c) * ldy + kc] : Y[kc * ldy + 16 * nt + c])
                           : 0.f;
    if constexpr (NR) fr[0].yr[0] = okk ? (YT ? Y[(int64_t)cr * ldy + kc] : Y[kc * ldy + cr]) : 0.f;
#pragma unroll
    for (int t = 0; t < MW; ++t) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[t][nt] = mfma16(fr[0].x[0][t], fr[0].y[0][nt], acc[t][nt]);
      if constexpr (NR) accr[t] = mfma4x4(fr[0].x[0][t], fr[0].yr[0], accr[t]);
    }
  }

  float* Dp = D + (int64_t)blockIdx.y * dsplit;
#pragma unroll
  for (int t = 0; t < MW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = tn_col_f32<VX>(m0, t, acc_row<float>(lane, r));
      if (row < M) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) Dp[row * ldd + 16 * nt + c] = acc[t][nt][r];
      }
    }
  if constexpr (NR) {
#define TN_ROW(T, I) tn_col_f32<VX>(m0, T, I)
    F32_STORE_REM(TN_ROW)
#undef TN_ROW
  }
}
#undef F32_COMPUTE
#undef F32_LOAD_Y
#undef F32_STORE_REM

// Launch shapes, from a timing sweep at 65536^2, k = 50: one wave per SIMD with
// a deep register pipeline, TN then takes 128 columns of A per wave. TN below
// 2^28 entries of A (8192 x 4096 at k = 64) has too few of those waves; two per
// SIMD of 64 columns each took 5% less time per product there.
constexpr int F32_WAVES = 4, F32_NN_MW = 4;
static bool tn_small(int64_t M, int64_t K) { return M * K < ((int64_t)1 << 28); }

// Slabs: about one workgroup per CU, each at least 256 long (64 for a product
// under 2^26 multiply-adds) and, while the slabs stay under 2^28 elements, at
// most 8192: the matrix cores add a slab's products into one float
// accumulator, and over 32768 terms its rounding moved a HALS trajectory by
// 1.1e-5 at its second iteration, against 2.4e-7 with slabs of 8192, which are
// summed in double.
int64_t gemm_f32_splits(GemmKind kind, int64_t M, int64_t N, int64_t K) {
  const int mw = kind == GemmKind::NN ? F32_NN_MW : tn_small(M, K) ? 4 : 8;
  const int64_t wgs = cdiv(M, 16 * mw * F32_WAVES);
  const int64_t minlen = M * N * K < ((int64_t)1 << 26) ? 64 : 256;
  int64_t s = 1;
  while (wgs * s < 256 && K / (2 * s) >= minlen && s < MAX_PRODUCT_SPLITS) s *= 2;
  while (K > s * 8192 && s < MAX_PRODUCT_SPLITS && 2 * s * M * N <= ((int64_t)1 << 28)) s *= 2;
  return s;
}

struct F32Call {
  GemmArgs<float> a;
  bool vx;
  int64_t splits, kchunk;
  float* D;
  int64_t ldd;
};

template <int NT, int NR, bool VX, bool YT>
static void f32_launch(GemmKind kind, const F32Call& p, hipStream_t st) {
  const GemmArgs<float>& a = p.a;
  const int ncols = (int)a.N;
  auto grid = [&](int mw) {
    return dim3((unsigned)cdiv(a.M, 16 * mw * F32_WAVES), (unsigned)p.splits);
  };
  if (kind == GemmKind::NN)
    gemm_nn_f32_kernel<NT, F32_NN_MW, VX, YT, 6, 1, NR><<<grid(F32_NN_MW), 64 * F32_WAVES, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, p.D, p.ldd, a.M * a.N, a.M, a.K, p.kchunk, ncols);
  else if (tn_small(a.M, a.K))
    gemm_tn_f32_kernel<NT, 4, VX, YT, 3, 2, NR><<<grid(4), 64 * F32_WAVES, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, p.D, p.ldd, a.M * a.N, a.M, a.K, p.kchunk, ncols);
  else
    gemm_tn_f32_kernel<NT, 8, VX, YT, 4, 1, NR><<<grid(8), 64 * F32_WAVES, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, p.D, p.ldd, a.M * a.N, a.M, a.K, p.kchunk, ncols);
}

template <int NT, int NR>
static void f32_dispatch(GemmKind kind, const F32Call& p, hipStream_t st) {
  if (p.vx && p.a.yt) f32_launch<NT, NR, true, true>(kind, p, st);
  else if (p.vx) f32_launch<NT, NR, true, false>(kind, p, st);
  else if (p.a.yt) f32_launch<NT, NR, false, true>(kind, p, st);
  else f32_launch<NT, NR, false, false>(kind, p, st);
}

hipError_t gemm_f32(GemmKind kind, const GemmArgs<float>& a, int nvalid, float* part,
                    hipStream_t st, int* nsplit) {
  if (kind == GemmKind::TN_GRAM || a.N < 16 || a.N > 64 || a.N % 16 || nvalid < 1 || nvalid > a.N ||
      a.M < 1 || a.K < 1 || a.ldx < (kind == GemmKind::NN ? a.K : a.M) || a.Dt)
    return hipErrorInvalidValue;
  auto aligned = [](const float* p, int64_t ld) { return (uintptr_t)p % 16 == 0 && ld % 4 == 0; };
  // a transposed Y is only read with 16-byte loads
  if (a.ldy < (a.yt ? a.K : a.N) || (a.yt && !aligned(a.Y, a.ldy))) return hipErrorInvalidValue;
  int64_t splits = gemm_f32_splits(kind, a.M, a.N, a.K);
  const int64_t kchunk = round_up(cdiv(a.K, splits), 16);
  splits = cdiv(a.K, kchunk);
  const bool slabs = splits > 1;
  const F32Call p{a, aligned(a.X, a.ldx), splits, kchunk, slabs ? part : a.D,
                  slabs ? a.N : a.ldd};
  const bool rem = nvalid > 16 && nvalid % 16 >= 1 && nvalid % 16 <= 4;
  switch (rem ? nvalid / 16 + 4 : a.N / 16) {
    case 1: f32_dispatch<1, 0>(kind, p, st); break;
    case 2: f32_dispatch<2, 0>(kind, p, st); break;
    case 3: f32_dispatch<3, 0>(kind, p, st); break;
    case 4: f32_dispatch<4, 0>(kind, p, st); break;
    case 5: f32_dispatch<1, 1>(kind, p, st); break;
    case 6: f32_dispatch<2, 1>(kind, p, st); break;
    case 7: f32_dispatch<3, 1>(kind, p, st); break;
    default: return hipErrorInvalidValue;
  }
  const hipError_t e = NMF_LAUNCH_CHECK();
  if (nsplit) *nsplit = (int)splits;
  if (e != hipSuccess || !slabs || nsplit) return e;
  return reduce_splits<float>(part, (int)splits, a.M * a.N, a.M, (int)a.N, a.ldd, a.D, a.N, st);
}

}  // namespace nmfk
