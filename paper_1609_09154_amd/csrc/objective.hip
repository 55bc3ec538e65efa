// Relative error ||A - W H||_F / ||A||_F (Section 6.2), evaluated directly:
// tiles of W H are formed on the matrix cores, the matching entries of A are
// read once, and squared differences are summed in double. Each workgroup
// writes one double; finish_relerr sums them in a fixed order, so the value
// is reproducible run to run. The pass that needs ||A|| too (the first of a
// run) sums the squares of A's entries as it reads them.
#include "common.h"
#include "rowtile.h"
#include "kernels.h"

#include "split_mma.h"

#include <type_traits>

namespace nmfk {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Block-wide sum of one double per thread (blockDim.x multiple of 64, <= 1024).
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double sh[16];
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
  return s;  // valid in thread 0
}

// Residual pass. A wave takes 64 columns of A and a run of its 16-row tiles.
// The 64 rows of Ht stay with the wave for all its tiles, so a tile costs one
// read of its 16 x 64 entries of A (lane (g, c) takes columns 4 c .. 4 c + 3 of
// four rows, so a load instruction covers 256 bytes of each row; tile j of the
// product takes columns 4 c + j to match) and of 16 rows of W, both fetched
// while the tile before is computed. Float: the block's four waves take
// neighbouring columns and the same tiles, so that W's rows come once per
// block (the other waves find them in the L1 cache); double: the same columns,
// whose rows of Ht are in LDS, and the run's tiles in turn.
//
// What bounds it is the read of A, at the occupancy that Ht's planes leave:
// 100003 x 5003 at k = 50 took 1781 us (64 x 256 blocks, element loads after
// the product, and 55 us more to sum their partials, and 755 for ||A||) and
// takes 0.57 ms with ||A|| (3.5 TB/s; rows of an odd length are not 16-byte
// aligned) and 0.48 without. Of that, loads that no branch surrounds gave 830 -> 633 us, and
// the waves side by side 633 -> 561 (4096 x 2048 at k = 32: 14.8 -> 13.8 ->
// 11.5; 30000^2 at k = 64: 1304 -> 985 -> 1009).
// Four entries of a row of A, widened to what the difference is taken in.
template <typename TA> struct A4;
template <> struct A4<float> {
  typedef float V __attribute__((ext_vector_type(4), aligned(4)));
  V v;
  __device__ __forceinline__ void load(const float* p) { v = *reinterpret_cast<const V*>(p); }
  __device__ __forceinline__ double at(int j) const { return (double)v[j]; }
  __device__ __forceinline__ void set(int j, float x) { v[j] = x; }
};
template <> struct A4<double> {
  typedef double V __attribute__((ext_vector_type(2), aligned(8)));
  V v[2];
  __device__ __forceinline__ void load(const double* p) {
    v[0] = *reinterpret_cast<const V*>(p);
    v[1] = *reinterpret_cast<const V*>(p + 2);
  }
  __device__ __forceinline__ double at(int j) const { return v[j >> 1][j & 1]; }
  __device__ __forceinline__ void set(int j, double x) { v[j >> 1][j & 1] = x; }
};
template <> struct A4<uint16_t> {
  uint2 v;
  __device__ __forceinline__ void load(const uint16_t* p) { v = *reinterpret_cast<const uint2*>(p); }
  __device__ __forceinline__ double at(int j) const {
    const unsigned w = j < 2 ? v.x : v.y;
    return (double)__uint_as_float((j & 1) ? w & 0xffff0000u : w << 16);
  }
  __device__ __forceinline__ void set(int j, uint16_t x) {
    unsigned& w = j < 2 ? v.x : v.y;
    w = (j & 1) ? (w & 0xffffu) | (unsigned)x << 16 : (w & 0xffff0000u) | x;
  }
};
template <> struct A4<uint8_t> {
  unsigned v;
  __device__ __forceinline__ void load(const uint8_t* p) { v = *reinterpret_cast<const unsigned*>(p); }
  __device__ __forceinline__ double at(int j) const {
    return (double)fp8_e4m3_bits_to_float((uint8_t)(v >> (8 * j)));
  }
  __device__ __forceinline__ void set(int j, uint8_t x) {
    v = (v & ~(0xffu << (8 * j))) | (unsigned)x << (8 * j);
  }
};

constexpr int RC = 64;       // columns of A per wave
constexpr int RWAVES = 4;    // waves per block

// One tile's entries of A: row row0 + rr(r), columns col .. col + 3. ACC: the
// type of the product (row order of its accumulator). A block whose columns
// run past n (not FULL) loads element by element.
template <bool FULL, typename TACC, typename TA>
__device__ __forceinline__ void load_a_tile(A4<TA> (&av)[4], const TA* __restrict__ A, int64_t lda,
                                            int64_t m, int64_t n, int64_t row0, int64_t col,
                                            int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int64_t row = row0 + acc_row<TACC>(lane, r);
    row = row < m ? row : m - 1;
    const TA* p = A + row * lda;
    if constexpr (FULL) {
      av[r].load(p + col);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) av[r].set(j, p[col + j < n ? col + j : n - 1]);
    }
  }
}

// Adds the squares of the tile's A - scale acc to sr and, NORM, A's to sa
// (scale: a power of two).
template <bool FULL, bool NORM, typename TACC, typename TA, typename ACC>
__device__ __forceinline__ void add_tile(const A4<TA> (&av)[4], const ACC (&acc)[4], double scale,
                                         int64_t m, int64_t n, int64_t row0, int64_t col, int lane,
                                         double& sr, double& sa) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (row0 + acc_row<TACC>(lane, r) >= m) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!FULL && col + j >= n) continue;
      const double a = av[r].at(j), d = fma(-scale, (double)acc[j][r], a);
      sr = fma(d, d, sr);
      if constexpr (NORM) sa = fma(a, a, sa);
    }
  }
}

// Float factors: the product on the bfloat16 cores from exact splits
// (split.h), Ht's planes in registers. KS steps of 32 rank entries.
template <typename TA, int KS, bool NORM>
__global__ __launch_bounds__(64 * RWAVES, KS <= 2 ? 2 : 1) void residual_split_kernel(
    const TA* __restrict__ A, int64_t lda, int64_t m, int64_t n, const float* __restrict__ W,
    const float* __restrict__ Ht, int KP, int64_t rows, double* __restrict__ partial,
    double* __restrict__ npartial) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int64_t c0 = ((int64_t)blockIdx.x * RWAVES + wave) * RC, col = c0 + 4 * c;
  const int64_t rbeg = (int64_t)blockIdx.y * rows;
  // a wave past the last column takes no tile
  const int64_t rend = c0 >= n ? 0 : rbeg + rows < m ? rbeg + rows : m;
  const bool full = c0 + RC <= n;
  // eight entries 32 s + 8 g .. of a factor row; clear8: zero past KP
  auto load8 = [&](float (&x)[8], const float* row, int s) {
    const int k0 = 32 * s + 8 * g < KP ? 32 * s + 8 * g : 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 v = *reinterpret_cast<const float4*>(row + k0 + 4 * h);
      x[4 * h] = v.x; x[4 * h + 1] = v.y; x[4 * h + 2] = v.z; x[4 * h + 3] = v.w;
    }
  };
  auto clear8 = [&](float (&x)[8], int s) {
    if (s < KS - 1) return;
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = 32 * s + 8 * g < KP ? x[u] : 0.f;
  };
  Split8 hp[KS][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float* row = Ht + (col + j < n ? col + j : n - 1) * KP;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float x[8];
      load8(x, row, s);
      clear8(x, s);
      hp[s][j] = split8(x);
    }
  }
  double sr = 0.0, sa = 0.0;
  // PF tiles in flight (one wave per SIMD has the registers for two). Loads of
  // tiles past the run's end are clamped, not skipped: with a branch around a
  // load the compiler cannot count what was issued after it, and waits for
  // all of it.
  constexpr int PF = KS <= 2 ? 1 : 2;
  auto run = [&](auto fullc) {
    constexpr bool FULL = decltype(fullc)::value;
    float wv[PF][KS][8];
    A4<TA> av[PF][4];
    auto load_w = [&](int p, int64_t row0) {
      const int64_t row = row0 + c < m ? row0 + c : m - 1;
#pragma unroll
      for (int s = 0; s < KS; ++s) load8(wv[p][s], W + row * KP, s);
    };
    auto load_a = [&](int p, int64_t row0) {
      load_a_tile<FULL, float>(av[p], A, lda, m, n, row0, col, lane);
    };
    auto tile = [&](int p, int64_t row0) {
      f32x4 acc[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = zero4<float>();
      Split8 ws[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        clear8(wv[p][s], s);
        ws[s] = split8(wv[p][s]);
      }
      load_w(p, row0 + PF * 16);
#pragma unroll
      for (int s = 0; s < KS; ++s) split_mma(ws[s], hp[s], acc);
      // scaled sums that are not finite (as in the products): again with the
      // float instruction
      bool bad = false;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) bad = bad || !(fabsf(acc[j][r]) <= 3.402823466e38f);
      double scale = SPLIT_UNSCALE;
      if (__ballot(bad)) {
        scale = 1.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = zero4<float>();
        const int64_t row = row0 + c < m ? row0 + c : m - 1;
        for (int k0 = 0; k0 < KP; k0 += 4)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[j] = mfma16(W[row * KP + k0 + g],
                            Ht[(col + j < n ? col + j : n - 1) * KP + k0 + g], acc[j]);
      }
      add_tile<FULL, NORM, float>(av[p], acc, scale, row0 < rend ? m : 0, n, row0, col, lane, sr, sa);
      load_a(p, row0 + PF * 16);
    };
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      load_w(p, rbeg + p * 16);
      load_a(p, rbeg + p * 16);
    }
    for (int64_t row0 = rbeg; row0 < rend; row0 += PF * 16) {
#pragma unroll
      for (int p = 0; p < PF; ++p) tile(p, row0 + p * 16);
    }
  };
  if (full) run(std::true_type{});
  else run(std::false_type{});
  const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const double s = block_sum(sr);
  if (threadIdx.x == 0) partial[b] = s;
  if constexpr (NORM) {
    __syncthreads();
    const double t = block_sum(sa);
    if (threadIdx.x == 0) npartial[b] = t;
  }
}

// Double factors: the block's 64 rows of Ht in LDS (row 16 j + c holds column
// 4 c + j); lane group g takes rank entries k0 + 2 g and k0 + 2 g + 1 of two
// successive products.
template <int KP, bool NORM>
__global__ __launch_bounds__(64 * RWAVES, 2) void residual_f64_kernel(
    const double* __restrict__ A, int64_t lda, int64_t m, int64_t n, const double* __restrict__ W,
    const double* __restrict__ Ht, int64_t rows, double* __restrict__ partial,
    double* __restrict__ npartial) {
  constexpr int LD = KP + 2;
  __shared__ __attribute__((aligned(16))) double Hs[RC * LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int64_t c0 = (int64_t)blockIdx.x * RC, col = c0 + 4 * c;
  const int64_t rbeg = (int64_t)blockIdx.y * rows, rend = rbeg + rows < m ? rbeg + rows : m;
  const bool full = c0 + RC <= n;
  for (int e = threadIdx.x; e < RC * (KP / 2); e += 64 * RWAVES) {
    const int q = e / (KP / 2), i = 2 * (e % (KP / 2));
    const int64_t cc = c0 + 4 * (q & 15) + (q >> 4);
    const V16<double> v = load16<double>(Ht + (cc < n ? cc : n - 1) * KP + i);
    Hs[q * LD + i] = v.v[0];
    Hs[q * LD + i + 1] = v.v[1];
  }
  __syncthreads();
  double sr = 0.0, sa = 0.0;
  auto run = [&](auto fullc) {
    constexpr bool FULL = decltype(fullc)::value;
    A4<double> av[4];
    int64_t row0 = rbeg + 16 * wave;
    load_a_tile<FULL, double>(av, A, lda, m, n, row0, col, lane);
    for (; row0 < rend; row0 += 16 * RWAVES) {
      f64x4 acc[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = zero4<double>();
      A4<double> cur[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) cur[r] = av[r];
      load_a_tile<FULL, double>(av, A, lda, m, n, row0 + 16 * RWAVES, col, lane);
      const double* wr = W + (row0 + c < m ? row0 + c : m - 1) * KP + 2 * g;
#pragma unroll 2
      for (int k0 = 0; k0 < KP; k0 += 8) {
        const V16<double> w = load16<double>(wr + k0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const V16<double> h = load16<double>(&Hs[(16 * j + c) * LD + k0 + 2 * g]);
          acc[j] = mfma16(w.v[0], h.v[0], acc[j]);
          acc[j] = mfma16(w.v[1], h.v[1], acc[j]);
        }
      }
      add_tile<FULL, NORM, double>(cur, acc, 1.0, m, n, row0, col, lane, sr, sa);
    }
  };
  if (full) run(std::true_type{});
  else run(std::false_type{});
  const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const double s = block_sum(sr);
  if (threadIdx.x == 0) partial[b] = s;
  if constexpr (NORM) {
    __syncthreads();
    const double t = block_sum(sa);
    if (threadIdx.x == 0) npartial[b] = t;
  }
}

// Columns and rows per block: about 1024 blocks (512 and 2048 measured within
// 5% up to 8192^2; fewer cost 25% at 100003 x 5003), at least 64 rows.
constexpr int RBLOCKS = 1024;
template <typename T> constexpr int residual_cols() { return sizeof(T) == 8 ? RC : RC * RWAVES; }
template <typename T> static int64_t residual_rows(int64_t m, int64_t n) {
  const int64_t want = cdiv(RBLOCKS, cdiv(n, residual_cols<T>()));
  return round_up(cdiv(m, want), 16 * RWAVES);
}

template <typename T> int64_t residual_partials(int64_t m, int64_t n) {
  return cdiv(n, residual_cols<T>()) * cdiv(m, residual_rows<T>(m, n));
}
template int64_t residual_partials<float>(int64_t, int64_t);
template int64_t residual_partials<double>(int64_t, int64_t);

template <typename TA, int KS>
static void residual_split_launch(dim3 grid, const TA* A, int64_t lda, int64_t m, int64_t n,
                                  const float* W, const float* Ht, int KP, int64_t rows,
                                  double* partial, double* npartial, hipStream_t st) {
  if (npartial)
    residual_split_kernel<TA, KS, true><<<grid, 64 * RWAVES, 0, st>>>(A, lda, m, n, W, Ht, KP,
                                                                       rows, partial, npartial);
  else
    residual_split_kernel<TA, KS, false><<<grid, 64 * RWAVES, 0, st>>>(A, lda, m, n, W, Ht, KP,
                                                                        rows, partial, npartial);
}

template <typename T, typename TA>
hipError_t residual_sq(const TA* A, int64_t lda, int64_t m, int64_t n, const T* W, const T* Ht,
                       int KP, double* partial, double* npartial, hipStream_t st) {
  if (KP < 16 || KP > 128 || KP % 16) return hipErrorInvalidValue;
  const int64_t rows = residual_rows<T>(m, n);
  const dim3 grid((unsigned)cdiv(n, residual_cols<T>()), (unsigned)cdiv(m, rows));
  if constexpr (sizeof(T) == 8) {
    switch (KP) {
#define CASE(K)                                                                                   \
  case K:                                                                                         \
    if (npartial)                                                                                 \
      residual_f64_kernel<K, true><<<grid, 64 * RWAVES, 0, st>>>(A, lda, m, n, W, Ht, rows,       \
                                                                  partial, npartial);             \
    else                                                                                          \
      residual_f64_kernel<K, false><<<grid, 64 * RWAVES, 0, st>>>(A, lda, m, n, W, Ht, rows,      \
                                                                   partial, npartial);            \
    break;
      CASE(16) CASE(32) CASE(48) CASE(64) CASE(80) CASE(96) CASE(112) CASE(128)
#undef CASE
    }
  } else {
    switch ((KP + 31) / 32) {
#define CASE(K)                                                                               \
  case K:                                                                                     \
    residual_split_launch<TA, K>(grid, A, lda, m, n, W, Ht, KP, rows, partial, npartial, st); \
    break;
      CASE(1) CASE(2) CASE(3) CASE(4)
#undef CASE
    }
  }
  return NMF_LAUNCH_CHECK();
}

// Projected gradient of 1/2 ||A - W H||_F^2 in one factor (Section 6.2's
// stationarity measure), on the row layout: for each row x with its product
// row p and the Gram G of the other factor, g = x G - p, and the projection
// keeps g_i where x_i > 0 and min(g_i, 0) where x_i = 0. Each block sums the
// squares of its rows in double: TPR threads per row (4; 16 for a double
// 128 x 128 Gram, to stay within LDS), RPT = KP / TPR entries each, with G
// and the block's rows staged in LDS.
template <typename T, int KP> struct PgSplit {
  static constexpr int TPR = (sizeof(T) == 8 && KP == 128) ? 16 : 4;
  static constexpr int ROWS = 256 / TPR;
};
template <typename T, int KP>
__global__ __launch_bounds__(256) void pgrad_sq_kernel(const T* __restrict__ X,
                                                       const T* __restrict__ P,
                                                       const T* __restrict__ G, int64_t rows,
                                                       int k, double* __restrict__ partial) {
  constexpr int PG_TPR = PgSplit<T, KP>::TPR, PG_ROWS = PgSplit<T, KP>::ROWS;
  constexpr int RPT = KP / PG_TPR;
  constexpr int VEC = Tr<T>::VEC;
  constexpr int XLD = KP + VEC;
  __shared__ __attribute__((aligned(16))) T Gs[KP * KP];
  __shared__ __attribute__((aligned(16))) T Xs[PG_ROWS * XLD];
  const int64_t rb = (int64_t)blockIdx.x * PG_ROWS;
  stage_square<T, KP, 256>(Gs, G, nullptr);
  stage_rows<T, KP, PG_ROWS, XLD, 256>(Xs, X, rb, rows);
  __syncthreads();
  const int lr = threadIdx.x / PG_TPR;
  const int64_t r = rb + lr;
  const int i0 = (threadIdx.x % PG_TPR) * RPT;
  const T* xs = &Xs[lr * XLD];
  double local = 0.0;
  if (r < rows) {
    T g[RPT];
#pragma unroll
    for (int ii = 0; ii < RPT; ++ii) g[ii] = T(0);
#pragma unroll 8
    for (int j = 0; j < KP; ++j) {
      const T xj = xs[j];
#pragma unroll
      for (int q = 0; q < RPT / VEC; ++q) {
        const V16<T> v = load16<T>(&Gs[j * KP + i0 + q * VEC]);
#pragma unroll
        for (int w = 0; w < VEC; ++w) g[q * VEC + w] = fma(xj, v.v[w], g[q * VEC + w]);
      }
    }
#pragma unroll
    for (int ii = 0; ii < RPT; ++ii) {
      const int i = i0 + ii;
      if (i < k) {
        const double gi = (double)g[ii] - (double)P[r * KP + i];
        const double pr = xs[i] > T(0) ? gi : (gi < 0.0 ? gi : 0.0);
        local += pr * pr;
      }
    }
  }
  const double s = block_sum(local);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Upper bound on the blocks of any pgrad_sq launch (16 rows per block), and
// the exact count of one launch.
int64_t pgrad_partials(int64_t rows) { return cdiv(rows, 16); }
template <typename T>
int64_t pgrad_blocks(int64_t rows, int KP) {
  return cdiv(rows, (sizeof(T) == 8 && KP == 128) ? 16 : 64);
}
template int64_t pgrad_blocks<float>(int64_t, int);
template int64_t pgrad_blocks<double>(int64_t, int);

template <typename T>
hipError_t pgrad_sq(const T* X, const T* P, const T* G, int64_t rows, int k, int KP,
                    double* partial, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  switch (KP) {
#define CASE(K)                                                                             \
  case K:                                                                                   \
    pgrad_sq_kernel<T, K><<<(unsigned)cdiv(rows, PgSplit<T, K>::ROWS), 256, 0, st>>>(      \
        X, P, G, rows, k, partial);                                                         \
    break;
    CASE(16) CASE(32) CASE(48) CASE(64) CASE(80) CASE(96) CASE(112) CASE(128)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return NMF_LAUNCH_CHECK();
}
template hipError_t pgrad_sq<float>(const float*, const float*, const float*, int64_t, int, int,
                                    double*, hipStream_t);
template hipError_t pgrad_sq<double>(const double*, const double*, const double*, int64_t, int,
                                     int, double*, hipStream_t);

// One block of 1024 threads; thread t sums partial[t], partial[t+1024], ... in
// order, then a fixed tree (and the same for npartial, ||A||^2, where given).
template <typename T>
__global__ __launch_bounds__(1024) void finish_kernel(
    const double* __restrict__ partial, const double* __restrict__ npartial, int64_t np,
    const T* __restrict__ G1, const T* __restrict__ G2, int KP, double* __restrict__ ref_sq,
    double* __restrict__ out) {
  double s = 0.0, q = 0.0;
  for (int64_t i = threadIdx.x; i < np; i += blockDim.x) {
    s += partial[i];
    if (npartial != nullptr) q += npartial[i];
  }
  if (G1 != nullptr)
    for (int e = threadIdx.x; e < KP * KP; e += blockDim.x) s += (double)G1[e] * (double)G2[e];
  const double tot = block_sum(s);
  double nrm = 0.0;
  if (npartial != nullptr) {
    __syncthreads();
    nrm = block_sum(q);
  }
  if (threadIdx.x == 0) {
    if (ref_sq != nullptr) {
      if (npartial != nullptr) *ref_sq = nrm;
      else nrm = *ref_sq;
      const double v = tot > 0.0 ? tot : 0.0;
      *out = sqrt(v / nrm);
    } else {
      *out = tot;
    }
  }
}

template <typename T>
hipError_t finish_relerr(const double* partial, const double* npartial, int64_t np, const T* G1,
                         const T* G2, int KP, double* ref_sq, double* out, hipStream_t st) {
  finish_kernel<T><<<1, 1024, 0, st>>>(partial, npartial, np, G1, G2, KP, ref_sq, out);
  return NMF_LAUNCH_CHECK();
}

// Input scan: NaN, Inf or negative entries raise the flag.
template <typename T>
__global__ void check_dense_kernel(const T* __restrict__ A, int64_t lda, int64_t m, int64_t n,
                                   int* __restrict__ flag) {
  const int64_t r0 = (int64_t)blockIdx.x * 16;
  int bad = 0;
  for (int64_t r = r0; r < r0 + 16 && r < m; ++r)
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
      const double a = to_double(A[r * lda + j]);
      if (!(a >= 0.0) || a == (double)INFINITY) bad = 1;
    }
  if (bad) atomicOr(flag, 1);
}

template <typename T>
hipError_t check_dense(const T* A, int64_t lda, int64_t m, int64_t n, int* flag,
                       hipStream_t st) {
  check_dense_kernel<T><<<(unsigned)cdiv(m, 16), 256, 0, st>>>(A, lda, m, n, flag);
  return NMF_LAUNCH_CHECK();
}

#define INST(T)                                                                               \
  template hipError_t residual_sq<T, T>(const T*, int64_t, int64_t, int64_t, const T*,        \
                                        const T*, int, double*, double*, hipStream_t);        \
  template hipError_t finish_relerr<T>(const double*, const double*, int64_t, const T*,       \
                                       const T*, int, double*, double*, hipStream_t);         \
  template hipError_t check_dense<T>(const T*, int64_t, int64_t, int64_t, int*, hipStream_t);
INST(float)
INST(double)
#undef INST
#define INST_LP(TA)                                                                         \
  template hipError_t residual_sq<float, TA>(const TA*, int64_t, int64_t, int64_t,          \
                                             const float*, const float*, int, double*,       \
                                             double*, hipStream_t);                          \
  template hipError_t check_dense<TA>(const TA*, int64_t, int64_t, int64_t, int*, hipStream_t);
INST_LP(uint16_t)
INST_LP(uint8_t)
#undef INST_LP

}  // namespace nmfk
