// Double products of Algorithm 1 and the Grams of both types on the gfx950
// matrix cores (MFMA 16x16x4, fp32 or fp64), for one GPU's whole problem (the
// float products are in gemm.hip):
//
//   NN:  D (M x N) = X (M x K) * Y (K x N)   X K-contiguous, Y N-contiguous
//        used for P = A H^T  (X = A, Y = H^T, K = n)
//   TN:  D (M x N) = X^T * Y, X (K x M), Y (K x N), both row-contiguous
//        used for R = A^T W  (X = A, Y = W, K = m)  and the Grams
//        W^T W, H H^T        (X = Y = W or H^T)
//
// N is the padded rank KP = 16 * NT (KP >= k, zero padded), so each wave
// owns MW 16-row tiles of the streamed side and all NT tiles of the rank
// side: every element of A is loaded into registers exactly once, by one
// lane, and feeds NT MFMAs. The rank-side operand (a few MB) is shared by
// all waves and read through the L2.
//
// The reduction index is a sum, so the K positions each lane supplies can be
// permuted freely as long as both operands agree. NN uses that to give each
// lane a 16-byte run of a row of A (VEC consecutive K values feed VEC
// successive MFMAs); TN uses the same freedom on the M side (VEC consecutive
// columns of a row of A feed VEC different output tiles).
//
// Large reductions can be split (grid.y) into slabs written to a workspace
// and summed in a fixed order by reduce_splits, so results are bitwise
// reproducible run to run.
#include <algorithm>

#include "common.h"
#include "grid.h"
#include "kernels.h"
#include "pipeline.h"

namespace nmfk {

// 16 bytes at any element's alignment (rows of A with an odd pitch).
template <bool STREAM, typename T> __device__ __forceinline__ V16<T> load16u(const T* p) {
  typedef T VU __attribute__((ext_vector_type(Tr<T>::VEC), aligned(sizeof(T))));
  const VU* q = reinterpret_cast<const VU*>(p);
  VU t;
  if constexpr (STREAM) t = __builtin_nontemporal_load(q);
  else t = *q;
  V16<T> r;
#pragma unroll
  for (int v = 0; v < Tr<T>::VEC; ++v) r.v[v] = t[v];
  return r;
}

// ---------------------------------------------------------------------------
// NN kernel. Y is either K x N (YT = false, ldy between K rows) or its
// transpose N x K (YT = true, ldy between N rows), which lets each lane fetch
// its VEC consecutive K values of a Y column with one 16-byte load.
// ---------------------------------------------------------------------------
template <typename T, int NT, int MW> struct FragNN {
  V16<T> x[MW];
  T y[NT][Tr<T>::VEC];
};

template <typename T, int NT, int MW, bool YT, int STAGES, int WPE>
__global__ __launch_bounds__(256, WPE) void gemm_nn_kernel(
    const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y, int64_t ldy,
    T* __restrict__ D, int64_t ldd, int64_t dsplit, int64_t M, int64_t K,
    int64_t kchunk) {
  constexpr int VEC = Tr<T>::VEC;
  constexpr int KSTEP = 4 * VEC;
  typedef typename Tr<T>::acc4 acc4;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int64_t m0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (16 * MW);
  if (m0 >= M) return;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;

  const T* xr[MW];
#pragma unroll
  for (int mt = 0; mt < MW; ++mt) {
    int64_t row = m0 + 16 * mt + c;
    row = row < M ? row : M - 1;
    xr[mt] = X + row * ldx;
  }
  acc4 acc[MW][NT];
#pragma unroll
  for (int mt = 0; mt < MW; ++mt) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = zero4<T>();
  }

  FragNN<T, NT, MW> fr[STAGES];

#define NN_LOAD(F, K0)                                                        \
  {                                                                           \
    const int64_t kk0 = (K0) + VEC * g;                                       \
    _Pragma("unroll") for (int mt = 0; mt < MW; ++mt) {                       \
      F.x[mt] = load16u<false, T>(xr[mt] + kk0);                              \
    }                                                                         \
    _Pragma("unroll") for (int nt = 0; nt < NT; ++nt) {                       \
      if constexpr (YT) {                                                     \
        const V16<T> t_ = load16<T>(Y + (int64_t)(16 * nt + c) * ldy + kk0);  \
        _Pragma("unroll") for (int v = 0; v < VEC; ++v) F.y[nt][v] = t_.v[v]; \
      } else {                                                                \
        _Pragma("unroll") for (int v = 0; v < VEC; ++v)                       \
          F.y[nt][v] = Y[(kk0 + v) * ldy + 16 * nt + c];                      \
      }                                                                       \
    }                                                                         \
  }
#define NN_COMPUTE(F)                                                         \
  {                                                                           \
    _Pragma("unroll") for (int v = 0; v < VEC; ++v)                           \
      _Pragma("unroll") for (int mt = 0; mt < MW; ++mt) {                     \
        _Pragma("unroll") for (int nt = 0; nt < NT; ++nt)                     \
          acc[mt][nt] = mfma16(F.x[mt].v[v], F.y[nt][v], acc[mt][nt]);        \
      }                                                                       \
  }

  const int64_t nsteps = (kend - kbeg) / KSTEP;
  NMF_PIPELINE(STAGES, NN_LOAD, NN_COMPUTE, fr, kbeg, nsteps, KSTEP)

  const int64_t ktail = kbeg + nsteps * KSTEP;
  if (ktail < kend) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const int64_t kk = ktail + VEC * g + v;
      const bool ok = kk < kend;
#pragma unroll
      for (int mt = 0; mt < MW; ++mt) fr[0].x[mt].v[v] = ok ? xr[mt][kk] : T(0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        fr[0].y[nt][v] = ok ? (YT ? Y[(int64_t)(16 * nt + c) * ldy + kk] : Y[kk * ldy + 16 * nt + c])
                            : T(0);
    }
    NN_COMPUTE(fr[0]);
  }
#undef NN_LOAD
#undef NN_COMPUTE

  T* Dp = D + (int64_t)blockIdx.y * dsplit;
#pragma unroll
  for (int mt = 0; mt < MW; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = m0 + 16 * mt + acc_row<T>(lane, r);
      if (row < M) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) Dp[row * ldd + 16 * nt + c] = acc[mt][nt][r];
      }
    }
}

// ---------------------------------------------------------------------------
// TN kernel. One pipeline step covers 16 rows of X: lane group g supplies
// rows k0 + 4g + u to MFMA u (u = 0..3). Y is K x N (YT = false) or N x K
// (YT = true, so the four rows a lane needs are one 16-byte load).
// ---------------------------------------------------------------------------
// Column of X that lane column c feeds into M-tile t. Vector path: tile t
// takes columns m0 + 16*VEC*(t/VEC) + VEC*c + t%VEC (one 16-byte load per
// lane covers VEC tiles); scalar path: m0 + 16 t + c. What would pass the last
// column is moved back to end there, so that every wave runs the same pipelined
// loop, and lanes that then share a column compute and store the same value: a
// run or column of a lane by itself, or (BACK) the whole wave, by its m0. (A
// guarded loop of one memory latency per four rows for such waves took 85 of
// the 93 us of a 3000 x 1700 product at k = 40.)
template <typename T, bool VX, bool BACK>
__device__ __forceinline__ int64_t tn_col(int64_t m0, int t, int c, int64_t M) {
  constexpr int VEC = Tr<T>::VEC;
  if constexpr (VX) {
    const int64_t b = m0 + 16 * VEC * (t / VEC) + VEC * c;
    return (BACK || b < M - VEC ? b : M - VEC) + t % VEC;
  } else {
    const int64_t b = m0 + 16 * t + c;
    return b < M ? b : M - 1;
  }
}

template <typename T, int NT, int MW> struct FragTN {
  T x[4][MW];
  T y[4][NT];
};

// SYM 1 (Grams of up to 64 columns): Y is X and one wave takes all columns, so
// the fragment of X serves as Y too, in the same order of columns on either
// side of the output (the Y side read every row again, a float per lane and
// load). SYM 2: only the tiles on and above the diagonal are computed (the sums
// of the others are the same term by term). 11,708,841 rows at KP = 64: float
// 1.10 ms before, 0.99 with the shared fragment, 0.70 with those tiles only;
// double 1.68, 1.54, 1.14.
template <typename T, int NT, int MW, bool VX, bool YT, int STAGES, int WPE, bool STREAM, int SYM>
__global__ __launch_bounds__(256, WPE) void gemm_tn_kernel(
    const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y, int64_t ldy,
    T* __restrict__ D, int64_t ldd, int64_t dsplit, int64_t M, int64_t K,
    int64_t kchunk) {
  constexpr int VEC = Tr<T>::VEC;
  constexpr int NQ = VX ? MW / VEC : MW;  // loads per row on the X side
  static_assert(!VX || MW % VEC == 0, "vector path needs MW % VEC == 0");
  static_assert(!SYM || (MW == NT && !YT), "a Gram's wave takes all columns");
  typedef typename Tr<T>::acc4 acc4;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  int64_t m0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (16 * MW);
  if (m0 >= M) return;
  // Whole waves move back (M >= 16 MW) where the loads at constant distances
  // that this leaves save the registers of an address each: 64 columns at rank
  // 48, 20000 x 12000 at k = 40 558 -> 428 us. Below, where those fit, each lane by
  // itself is 2 to 5% faster (11200 x 42752 at k = 24: 656 against 691 us).
  constexpr bool BACK = VX && NQ > 1 && NT > 2 && !SYM;
  if (BACK && m0 > M - 16 * MW) m0 = M - 16 * MW;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  int64_t xc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) xc[q] = tn_col<T, VX, BACK>(m0, VX ? q * VEC : q, c, M);

  acc4 acc[MW][NT];
#pragma unroll
  for (int t = 0; t < MW; ++t) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[t][nt] = zero4<T>();
  }

  FragTN<T, NT, MW> fr[STAGES];

#define TN_LOAD(F, K0)                                                        \
  {                                                                           \
    _Pragma("unroll") for (int u = 0; u < 4; ++u) {                           \
      const int64_t kk = (K0) + 4 * g + u;                                    \
      const T* xrow = X + kk * ldx;                                           \
      if constexpr (VX) {                                                     \
        _Pragma("unroll") for (int q = 0; q < NQ; ++q) {                      \
          V16<T> t16 = load16u<STREAM, T>(xrow + xc[q]);                      \
          _Pragma("unroll") for (int v = 0; v < VEC; ++v) F.x[u][q * VEC + v] = t16.v[v]; \
        }                                                                     \
      } else {                                                                \
        _Pragma("unroll") for (int t = 0; t < MW; ++t) F.x[u][t] = xrow[xc[t]];    \
      }                                                                       \
    }                                                                         \
    _Pragma("unroll") for (int nt = 0; nt < NT && !SYM; ++nt) {               \
      if constexpr (YT) {                                                     \
        const T* yrow = Y + (int64_t)(16 * nt + c) * ldy + (K0) + 4 * g;      \
        _Pragma("unroll") for (int h = 0; h < 4 / VEC; ++h) {                 \
          const V16<T> t_ = load16<T>(yrow + h * VEC);                        \
          _Pragma("unroll") for (int v = 0; v < VEC; ++v) F.y[h * VEC + v][nt] = t_.v[v]; \
        }                                                                     \
      } else {                                                                \
        _Pragma("unroll") for (int u = 0; u < 4; ++u)                         \
          F.y[u][nt] = Y[((K0) + 4 * g + u) * ldy + 16 * nt + c];             \
      }                                                                       \
    }                                                                         \
  }
#define TN_COMPUTE(F)                                                         \
  {                                                                           \
    _Pragma("unroll") for (int u = 0; u < 4; ++u)                             \
      _Pragma("unroll") for (int t = 0; t < MW; ++t) {                        \
        _Pragma("unroll") for (int nt = SYM == 2 ? t : 0; nt < NT; ++nt)      \
          acc[t][nt] = mfma16(F.x[u][t], SYM ? F.x[u][nt % MW] : F.y[u][nt],  \
                              acc[t][nt]);                                    \
      }                                                                       \
  }

  constexpr int KSTEP = 16;
  const int64_t nsteps = (kend - kbeg) / KSTEP;
  NMF_PIPELINE(STAGES, TN_LOAD, TN_COMPUTE, fr, kbeg, nsteps, KSTEP)

  // Remainder (fewer than 16 rows), 4 at a time.
  for (int64_t k0 = kbeg + nsteps * KSTEP; k0 < kend; k0 += 4) {
    const int64_t kk = k0 + g;
    const bool okk = kk < kend;
    const int64_t kc = okk ? kk : kbeg;
#pragma unroll
    for (int t = 0; t < MW; ++t) {
      const T x = X[kc * ldx + tn_col<T, VX, BACK>(m0, t, c, M)];
      fr[0].x[0][t] = okk ? x : T(0);
    }
#pragma unroll
    for (int nt = 0; nt < NT && !SYM; ++nt)
      fr[0].y[0][nt] = okk ? (YT ? Y[(int64_t)(16 * nt + c) * ldy + kc] : Y[kc * ldy + 16 * nt + c])
                           : T(0);
#pragma unroll
    for (int t = 0; t < MW; ++t) {
#pragma unroll
      for (int nt = SYM == 2 ? t : 0; nt < NT; ++nt)
        acc[t][nt] = mfma16(fr[0].x[0][t], SYM ? fr[0].x[0][nt % MW] : fr[0].y[0][nt], acc[t][nt]);
    }
  }
#undef TN_LOAD
#undef TN_COMPUTE

  T* Dp = D + (int64_t)blockIdx.y * dsplit;
#pragma unroll
  for (int t = 0; t < MW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rho = acc_row<T>(lane, r);
      const int64_t row = tn_col<T, VX, BACK>(m0, t, rho, M);
#pragma unroll
      for (int nt = SYM == 2 ? t : 0; nt < NT; ++nt) {
        const int64_t col = SYM ? tn_col<T, VX, BACK>(0, nt, c, M) : 16 * nt + c;
        Dp[row * ldd + col] = acc[t][nt][r];
        if (SYM == 2 && nt > t) Dp[col * ldd + row] = acc[t][nt][r];
      }
    }
}

// s += src[p * stride] for p = p0, p0 + step, ... < splits, added in that
// order in double. The loads go out RS_BATCH at a time before any is added,
// so a thread waits for one memory latency per batch rather than per slab.
constexpr int RS_BATCH = 8;
template <typename T>
__device__ __forceinline__ double ordered_sum(const T* __restrict__ src, int p0, int step,
                                              int splits, int64_t stride) {
  double s = 0.0;
  int p = p0;
  for (; p + (RS_BATCH - 1) * step < splits; p += RS_BATCH * step) {
    T v[RS_BATCH];
#pragma unroll
    for (int u = 0; u < RS_BATCH; ++u) v[u] = src[(int64_t)(p + u * step) * stride];
#pragma unroll
    for (int u = 0; u < RS_BATCH; ++u) s += (double)v[u];
  }
  for (; p < splits; p += step) s += (double)src[(int64_t)p * stride];
  return s;
}

// out[i] = sum_s part[s * stride + i] in order s = 0, 1, ... (double sums);
// outt (nullable) receives the transpose, outt[c * rows + r]. The grid is
// capped (70,000,001 rows of 64 pass a dispatch's 2^32 work-items).
template <typename T>
__global__ void reduce_splits_kernel(const T* __restrict__ part, int splits, int64_t stride,
                                     int64_t rows, int cols, int64_t ldo, T* __restrict__ out,
                                     int64_t ldp, T* __restrict__ outt) {
  const int64_t total = rows * cols, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += step) {
    const int64_t r = idx / cols, cc = idx - r * cols;
    const double s = ordered_sum<T>(part + r * ldp + cc, 0, 1, splits, stride);
    out[r * ldo + cc] = (T)s;
    if (outt) outt[cc * rows + r] = (T)s;
  }
}

// Same sums for few outputs and many splits (the k x k Grams): RS_SUB
// threads per output each add every RS_SUB-th slab, then one thread adds the
// RS_SUB partial sums in order. The order is fixed, so results stay bitwise
// reproducible.
constexpr int RS_OUT = 16, RS_SUB = 16;
template <typename T>
__global__ __launch_bounds__(RS_OUT * RS_SUB) void reduce_splits_wide_kernel(
    const T* __restrict__ part, int splits, int64_t stride, int64_t rows, int cols, int64_t ldo,
    T* __restrict__ out, int64_t ldp, T* __restrict__ outt) {
  __shared__ double sh[RS_SUB][RS_OUT];
  const int o = threadIdx.x % RS_OUT, sub = threadIdx.x / RS_OUT;
  const int64_t idx = (int64_t)blockIdx.x * RS_OUT + o;
  const int64_t total = rows * cols;
  const int64_t r = idx / cols, cc = idx - r * cols;
  double s = 0.0;
  if (idx < total) s = ordered_sum<T>(part + r * ldp + cc, sub, RS_SUB, splits, stride);
  sh[sub][o] = s;
  __syncthreads();
  if (sub == 0 && idx < total) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < RS_SUB; ++q) t += sh[q][o];
    out[r * ldo + cc] = (T)t;
    if (outt) outt[cc * rows + r] = (T)t;
  }
}

template <typename T>
hipError_t reduce_splits(const T* part, int splits, int64_t dsplit, int64_t M, int N,
                         int64_t ldd, T* D, int64_t ldp, hipStream_t st, T* Dt) {
  const int64_t total = M * N;
  if (total < 65536 && splits > 16)
    reduce_splits_wide_kernel<T><<<(unsigned)cdiv(total, RS_OUT), RS_OUT * RS_SUB, 0, st>>>(
        part, splits, dsplit, M, N, ldd, D, ldp, Dt);
  else
    reduce_splits_kernel<T><<<capped_grid(cdiv(total, 256)), 256, 0, st>>>(part, splits, dsplit, M,
                                                                            N, ldd, D, ldp, Dt);
  return NMF_LAUNCH_CHECK();
}
template hipError_t reduce_splits<float>(const float*, int, int64_t, int64_t, int, int64_t, float*,
                                         int64_t, hipStream_t, float*);
template hipError_t reduce_splits<double>(const double*, int, int64_t, int64_t, int, int64_t,
                                          double*, int64_t, hipStream_t, double*);

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
// Launch shapes of the double products, two waves per SIMD (TN above rank 80:
// one, for its registers). A wave takes 64 rows (columns) of A where its two
// steps in flight fit the registers (NN to rank 64, TN to rank 48, 20000 x 12000
// at k = 40 7.8 -> 6.1 ms for six iterations; at rank 64 the 64-column TN wave
// spilled and took 2.2 ms for 20000^2, the 32-column one takes 1.17) and the
// grid still fills the chip; smaller products halve that until it does, down to
// 16, at low ranks with a deeper pipeline: their time is the latency of a wave's
// steps (3000 x 1700 at k = 40: 48 workgroups of 64-row waves and 93 us, now
// 17). 20000^2 at k = 64 runs at 44 TFLOP/s of the 73 that a large matrix
// product reaches; its register-only pipeline of two steps is what is left.
constexpr int WAVES = 4;  // waves per workgroup of the product kernels
constexpr int prod_stages(int NT, int mw) { return mw == 1 && NT <= 2 ? 4 : 2; }
constexpr int tn_wpe(int NT) { return NT <= 5 ? 2 : 1; }
static int prod_mw(GemmKind kind, int NT, int64_t M, int64_t K) {
  const int64_t room = std::max<int64_t>(1, std::min<int64_t>(MAX_PRODUCT_SPLITS, K / 128));
  int mw = NT <= (kind == GemmKind::NN ? 4 : 3) ? 4 : 2;
  while (mw > 1 && (cdiv(M, 16 * mw * WAVES) * room < 256 || M < 16 * mw)) mw /= 2;
  return mw;
}

// Slabs of the reduction: of the counts up to MAX_PRODUCT_SPLITS whose slabs are
// at least 128 long (64 in a product under 2^26 multiply-adds, such as a 2000 x
// 1000 matrix at k = 10, where they cost little), none longer than MAX_SPLIT_LEN
// while all hold at most 2^28 elements, the one with the fullest rounds of a
// workgroup per CU after what its slabs cost, 4 N / K of the product's time each
// (it is written by the product and read by the row update, whose few workgroups
// are slower at it; N counts to 48, past which the product is bound by its
// operations: A^T W of 1000 x 20000 at k = 60 72 us, 92 with one slab). A second workgroup per CU brings nothing, since
// one already keeps the CU's share of the memory busy. Runs of six HALS
// iterations with at least 512 workgroups, and now: 7424 x 3648 at k = 24 1010 ->
// 882 us, 8192 x 4096 at k = 8 1000 -> 924, 9000 x 7000 at k = 40 2198 -> 1982,
// 16384 x 8192 at k = 60 4.91 -> 4.49 ms, 20000 x 12000 at k = 24 5.67 -> 4.93;
// half that cost per slab takes 1 to 7% longer on the last. Over 140 runs and
// steps of fourteen sizes and five ranks none is more than 3% slower than before.
constexpr int64_t MAX_SPLIT_LEN = 8192;
static int64_t auto_splits(int64_t wgs, int64_t M, int64_t N, int64_t K) {
  const int64_t minlen = M * N * K < ((int64_t)1 << 26) ? 64 : 128;
  auto room = [&](int64_t t) { return t * M * N <= ((int64_t)1 << 28); };
  int64_t s = 1;
  while (K > s * MAX_SPLIT_LEN && s < MAX_PRODUCT_SPLITS && room(s + 1)) ++s;
  return fullest_rounds(wgs, s, 256, 4.0 * (double)std::min<int64_t>(N, 48) / (double)K, [&](int64_t t) {
    return t <= MAX_PRODUCT_SPLITS && K / t >= minlen && room(t);
  });
}

template <typename T, int NT, int MW>
static void nn_launch(const GemmArgs<T>& a, int64_t splits, int64_t kchunk, T* D, int64_t ldd,
                      int64_t dsplit, hipStream_t st) {
  constexpr int S = prod_stages(NT, MW);
  const dim3 grid((unsigned)cdiv(a.M, 16 * MW * WAVES), (unsigned)splits);
  if (a.yt)
    gemm_nn_kernel<T, NT, MW, true, S, 2><<<grid, 64 * WAVES, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
  else
    gemm_nn_kernel<T, NT, MW, false, S, 2><<<grid, 64 * WAVES, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
}

template <typename T, int NT, int MW, bool VX, bool STREAM>
static void tn_launch(const GemmArgs<T>& a, int waves, int64_t splits, int64_t kchunk, T* D,
                      int64_t ldd, int64_t dsplit, hipStream_t st) {
  constexpr int S = prod_stages(NT, MW);
  const dim3 grid((unsigned)cdiv(a.M, 16 * MW * waves), (unsigned)splits);
  if (a.yt)
    gemm_tn_kernel<T, NT, MW, VX, true, S, tn_wpe(NT), STREAM, 0><<<grid, 64 * waves, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
  else
    gemm_tn_kernel<T, NT, MW, VX, false, S, tn_wpe(NT), STREAM, 0><<<grid, 64 * waves, 0, st>>>(
        a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
}

// Gram slabs compute half the tiles (SYM 2), float ones from GRAM_HALF rows on:
// shorter ones do not repay the scattered stores of the other half (200,000 rows at
// KP = 64, 196 a slab: float 27 us with all tiles, 31 with half, double 45 and 36;
// 1,048,576 rows, 1024 a slab: float 79 and 67).
constexpr int64_t GRAM_HALF = 512;
// Gram: the M side is the padded rank itself, one wave per 16 MW columns; its
// operands are rows of the workspace, always aligned.
template <typename T, int NT>
static void gram_launch(const GemmArgs<T>& a, int64_t splits, int64_t kchunk, T* D, int64_t ldd,
                        int64_t dsplit, hipStream_t st) {
  constexpr int MW = sizeof(T) == 8 && NT > 4 ? 2 : NT <= 4 ? NT : 4;
  const dim3 grid((unsigned)cdiv(a.M, 16 * MW), (unsigned)splits);
  constexpr int WPE = sizeof(T) == 8 ? 1 : 2;
  if (MW == NT && (sizeof(T) == 8 || kchunk >= GRAM_HALF))
    gemm_tn_kernel<T, NT, MW, MW % Tr<T>::VEC == 0, false, 2, WPE, false, MW == NT ? 2 : 0>
        <<<grid, 64, 0, st>>>(a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
  else
    gemm_tn_kernel<T, NT, MW, MW % Tr<T>::VEC == 0, false, 2, WPE, false, MW == NT ? 1 : 0>
        <<<grid, 64, 0, st>>>(a.X, a.ldx, a.Y, a.ldy, D, ldd, dsplit, a.M, a.K, kchunk);
}

// TN streams A past the caches (non-temporal loads) where A, with its transposed
// copy if the other direction reads one, is larger than the 256 MB last-level
// cache, which would keep it for the next product (7424 x 3648 at k = 8, 217 MB
// each of the two: 4% of a run). NN's load
// instructions take half a line of a row each, and the other half has to be
// in the cache when the next asks for it.
template <typename T, int NT>
static void prod_dispatch(GemmKind kind, const GemmArgs<T>& a, int64_t splits, int64_t kchunk,
                          T* D, int64_t ldd, int64_t dsplit, hipStream_t st) {
  const int mw = prod_mw(kind, NT, a.M, a.K);
  if (kind == GemmKind::NN) {
    if constexpr (NT <= 4)
      if (mw == 4) return nn_launch<T, NT, 4>(a, splits, kchunk, D, ldd, dsplit, st);
    if (mw == 2) return nn_launch<T, NT, 2>(a, splits, kchunk, D, ldd, dsplit, st);
    return nn_launch<T, NT, 1>(a, splits, kchunk, D, ldd, dsplit, st);
  }
  const bool stream = a.M * a.K * (int64_t)sizeof(T) > ((int64_t)1 << (a.pair ? 27 : 28));
  if constexpr (NT <= 3) {
    if (mw == 4 && stream)
      return tn_launch<T, NT, 4, true, true>(a, WAVES, splits, kchunk, D, ldd, dsplit, st);
    if (mw == 4)
      return tn_launch<T, NT, 4, true, false>(a, WAVES, splits, kchunk, D, ldd, dsplit, st);
  }
  if (mw == 2 && stream)
    return tn_launch<T, NT, 2, true, true>(a, WAVES, splits, kchunk, D, ldd, dsplit, st);
  if (mw == 2)
    return tn_launch<T, NT, 2, true, false>(a, WAVES, splits, kchunk, D, ldd, dsplit, st);
  return tn_launch<T, NT, 1, false, false>(a, WAVES, splits, kchunk, D, ldd, dsplit, st);
}

template <typename T>
int64_t gemm_auto_splits(GemmKind kind, int64_t M, int64_t N, int64_t K) {
  if (kind == GemmKind::TN_GRAM) return 0;
  if (sizeof(T) == 4) return gemm_split_splits(M, (int)N, K);   // gemm_split's products
  const int64_t wgs = cdiv(M, 16 * prod_mw(kind, (int)(N / 16), M, K) * WAVES);
  return auto_splits(wgs, M, N, K);
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

template <typename T>
hipError_t gemm_run(GemmKind kind, const GemmArgs<T>& a_in, int64_t splits, T* part,
                    hipStream_t st, int* nsplit) {
  constexpr int VEC = Tr<T>::VEC;
  GemmArgs<T> a = a_in;
  const int NT = (int)(a.N / 16);
  if (NT < 1 || NT > 8 || a.N % 16 != 0) return hipErrorInvalidValue;
  if (sizeof(T) == 4 && kind != GemmKind::TN_GRAM) return hipErrorInvalidValue;
  if (splits < 1) splits = kind == GemmKind::TN_GRAM ? 1 : gemm_auto_splits<T>(kind, a.M, a.N, a.K);
  const int64_t unit = kind == GemmKind::NN ? 4 * VEC : 16;
  int64_t kchunk = round_up(cdiv(a.K, splits), unit);
  splits = cdiv(a.K, kchunk);
  if (splits < 1) splits = 1;
  // A transposed Y is only read with 16-byte loads; otherwise use it as given.
  if (a.yt && !(aligned16(a.Y) && a.ldy % VEC == 0)) return hipErrorInvalidValue;
  const bool small_m = kind == GemmKind::TN_GRAM;
  if (small_m) a.yt = false;
  // a transposed copy is written by the reduction, so a Gram that wants one
  // goes through it even unsplit
  if (a.Dt && !small_m) return hipErrorInvalidValue;
  const bool reduce = splits > 1 || a.Dt;
  T* D = reduce ? part : a.D;
  const int64_t ldd = reduce ? a.N : a.ldd;
  const int64_t dsplit = a.M * a.N;
  // a Gram reads its padded rows in 16-byte runs
  if (small_m && (!aligned16(a.X) || a.ldx % Tr<T>::VEC != 0)) return hipErrorInvalidValue;
  switch (NT) {
#define CASE(n)                                                                            \
  case n:                                                                                  \
    if (small_m) gram_launch<T, n>(a, splits, kchunk, D, ldd, dsplit, st);                 \
    else if constexpr (sizeof(T) == 8)                                                     \
      prod_dispatch<T, n>(kind, a, splits, kchunk, D, ldd, dsplit, st);                    \
    break;
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
  }
  const hipError_t e = NMF_LAUNCH_CHECK();
  if (nsplit) *nsplit = (int)splits;
  if (e != hipSuccess || !reduce || nsplit) return e;
  return reduce_splits<T>(part, (int)splits, dsplit, a.M, (int)a.N, a.ldd, a.D, a.N, st, a.Dt);
}

template int64_t gemm_auto_splits<float>(GemmKind, int64_t, int64_t, int64_t);
template int64_t gemm_auto_splits<double>(GemmKind, int64_t, int64_t, int64_t);
template hipError_t gemm_run<float>(GemmKind, const GemmArgs<float>&, int64_t, float*, hipStream_t,
                                    int*);
template hipError_t gemm_run<double>(GemmKind, const GemmArgs<double>&, int64_t, double*,
                                     hipStream_t, int*);

}  // namespace nmfk
