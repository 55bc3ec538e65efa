// Float products of Algorithm 1 on the bfloat16 matrix cores, at float
// accuracy:
//
//   NN:  D (M x N) = X (M x K) F      X = A,  F = H^T:  P = A H^T
//   TN:  D (M x N) = X^T F, X (K x M) X = A,  F = W:    R = A^T W
//
// Every float is the exact sum of three bfloat16 values, x = h + m + l: h is
// x rounded to nearest even, m the remainder x - h rounded, l what is left (8
// bits each cover the 24 of a float; both operands are scaled by 2^16 first, so
// that this holds down to the smallest float, see split.h). A product x f is
// taken as
//   h h' + h m' + m h' + m m' + h l' + l h'
// whose dropped terms are below 2^-25 |x f| with either sign, well under the
// rounding of a float sum. The six terms of 32 values of K take six
// v_mfma_f32_16x16x32_bf16 (16 cycles each) where the float instruction
// 16x16x4 needs eight of 32 cycles: 96 cycles against 256.
//
// That moves the bound of the large products from the float matrix cores to
// the read of A: 65536^2 at k = 50 took 3.79 ms a product (113 TFLOP/s, 72% of
// the float peak) and takes 3.2 to 3.5 ms for A H^T and 2.9 to 3.1 for A^T W (5.9
// TB/s; a device copy reaches 4.9), by how far the power limit lets the chip
// clock, with a third of the error (1.3e-6 against 3.6e-6 on the factors after
// ten HALS iterations). Products whose A stays in the caches are bound by the
// splits (seven VALU operations an entry) and the latency of a step: 8192 x
// 4096 at k = 64, 46 us before, 31 now.
//
// A is read in its own layout in both directions (a lane's operand is eight
// values along K of one row or column, and the split packs neighbours along K
// either way), so no transposed copy is made. The factor arrives packed
// (split.h), written by the kernel that updates it; a workgroup's four waves
// share each step's slice through LDS.
#include <algorithm>

#include "common.h"
#include "grid.h"
#include "kernels.h"
#include "split.h"
#include "split_mma.h"

namespace nmfk {

// loads of rows whose pitch is any number of floats: 4-byte alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int SPW = 4;      // waves per workgroup
constexpr int SBK = 32;     // K values per step

template <bool STREAM, typename V> __device__ __forceinline__ V load_a(const V* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}

// A step's 16 MT x 32 (NN) or 32 x 16 MT (TN) piece of X: 8 floats per lane
// and tile.
template <int MT> struct XStep { float v[MT][8]; };

// REM: the last of the NT tiles holds only nrem <= 5 rank columns. Its operand
// then takes the three planes of those columns side by side (column 16 (NT - 1)
// + c % nrem, plane c / nrem in lane column c), so that one product with each
// plane of X gives all of the six terms (and three smaller ones): three
// instructions instead of six, and the planes' sums are added at the end.
template <int NT, bool TR, int MT, int STAGES, int WPE, int FLUSH, bool STREAM, bool REM>
__global__ __launch_bounds__(64 * SPW, WPE) void gemm_split_kernel(
    const float* __restrict__ X, int64_t ldx, const u32x4* __restrict__ Fp,
    const float* __restrict__ F, int64_t ldf, int kv, float* __restrict__ D, int64_t ldd,
    int64_t dsplit, int nout, int nrem, int64_t M, int64_t K, int64_t kchunk) {
  constexpr int NF = REM ? NT - 1 : NT;    // tiles of six terms
  constexpr int NR = 16 * NT;              // factor columns
  constexpr int CH = 12 * NR;              // 16-byte chunks of a step's factor slice
  constexpr int PASS = (CH + 64 * SPW - 1) / (64 * SPW);
  static_assert(MT == 2 || MT == 4, "tiles per wave");
  static_assert(STAGES % 2 == 0, "the unrolled ring also indexes the two LDS buffers");
  // chunk (g, plane, column) at (3 g + plane) NR + column: K values 8 g .. 8 g + 7
  __shared__ u32x4 Fs[2][PASS * 64 * SPW];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int64_t m0 = ((int64_t)blockIdx.x * SPW + wave) * (16 * MT);
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  D += (int64_t)blockIdx.y * dsplit;

  // NN: lane (g, c) reads K values 8 g .. 8 g + 7 of row c of each tile.
  // TN: it reads rows 8 g .. 8 g + 7 of MT neighbouring columns, one for each
  // tile (column MT c + t of tile t); a run that would cross the last column
  // is moved back, so that two lanes may hold (and store) the same column.
  const float* xr[TR ? 1 : MT];
  int64_t col0 = 0;
  if constexpr (TR) {
    col0 = m0 + MT * c;
    col0 = col0 < M - MT ? col0 : M - MT;
    xr[0] = X + 8 * g * ldx + col0;
  } else {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      int64_t row = m0 + 16 * t + c;
      row = row < M ? row : M - 1;
      xr[t] = X + row * ldx + 8 * g;
    }
  }

  f32x4 acc[MT][NT], tot[MT][NT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (FLUSH) tot[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

  // REM: the lane's chunk of the last tile within a lane group's chunks
  int remo = 0;
  if constexpr (REM) remo = c < 3 * nrem ? (c / nrem) * NR + 16 * NF + c % nrem : 16 * NF;

  XStep<MT> xf[STAGES];
  u32x4 yv[PASS];   // factor slice of the next step

  auto load_x = [&](XStep<MT>& f, int64_t k0) {
    if constexpr (TR) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* p = xr[0] + (k0 + u) * ldx;
        if constexpr (MT == 4) {
          const f32x4u v = load_a<STREAM>(reinterpret_cast<const f32x4u*>(p));
#pragma unroll
          for (int t = 0; t < MT; ++t) f.v[t][u] = v[t];
        } else {
          const f32x2u v = load_a<STREAM>(reinterpret_cast<const f32x2u*>(p));
#pragma unroll
          for (int t = 0; t < MT; ++t) f.v[t][u] = v[t];
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4u v =
              load_a<STREAM>(reinterpret_cast<const f32x4u*>(xr[t] + k0 + 4 * h));
#pragma unroll
          for (int e = 0; e < 4; ++e) f.v[t][4 * h + e] = v[e];
        }
    }
  };
  auto load_f = [&](u32x4 (&v)[PASS], int64_t k0) {
    const u32x4* src = Fp + (k0 >> 3) * (3 * NR);
#pragma unroll
    for (int s = 0; s < PASS; ++s) {
      const int e = tid + s * 64 * SPW;
      v[s] = src[e < CH ? e : CH - 1];
    }
  };
  auto store_f = [&](const u32x4 (&v)[PASS], int buf) {
#pragma unroll
    for (int s = 0; s < PASS; ++s) Fs[buf][tid + s * 64 * SPW] = v[s];
  };
  auto compute = [&](const XStep<MT>& f, int buf) {
    Split8 a[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) a[t] = split8(f.v[t]);
    const u32x4* fb = &Fs[buf][3 * NR * g + c];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const u32x4 bh = fb[16 * j], bm = fb[NR + 16 * j], bl = fb[2 * NR + 16 * j];
#define TERM(PA, PB)                                             \
  _Pragma("unroll") for (int t = 0; t < MT; ++t)                 \
      acc[t][j] = mfma_bf16(a[t].PA, PB, acc[t][j]);
      TERM(l, bh) TERM(h, bl) TERM(m, bm) TERM(m, bh) TERM(h, bm) TERM(h, bh)
    }
    if constexpr (REM) {
      constexpr int j = NF;
      const u32x4 br = Fs[buf][3 * NR * g + remo];
      TERM(l, br) TERM(m, br) TERM(h, br)
    }
#undef TERM
  };
  auto flush = [&]() {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          tot[t][j][r] += acc[t][j][r];
          acc[t][j][r] = 0.f;
        }
  };

  const int64_t nfull = (kend - kbeg) / SBK;
  if (nfull > 0) {
    load_f(yv, kbeg);
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nfull) load_x(xf[s], kbeg + s * SBK);
    store_f(yv, 0);
    __syncthreads();
    constexpr int AHEAD = STAGES - 1;
    int64_t s = 0;
    int fl = 0;
    for (; s + STAGES + AHEAD <= nfull; s += STAGES) {
#pragma unroll
      for (int u = 0; u < STAGES; ++u) {
        const int64_t st = s + u;
        load_f(yv, kbeg + (st + 1) * SBK);
        load_x(xf[(u + STAGES - 1) % STAGES], kbeg + (st + STAGES - 1) * SBK);
        __builtin_amdgcn_sched_barrier(0);
        compute(xf[u], u & 1);
        store_f(yv, (u + 1) & 1);
        __syncthreads();
      }
      if constexpr (FLUSH) {
        fl += STAGES;
        if (fl >= FLUSH) {
          fl = 0;
          flush();
        }
      }
    }
    for (; s < nfull; s += STAGES) {
#pragma unroll
      for (int u = 0; u < STAGES; ++u) {
        const int64_t st = s + u;
        if (st < nfull) {
          if (st + 1 < nfull) load_f(yv, kbeg + (st + 1) * SBK);
          const int64_t pre = st + STAGES - 1;
          if (pre < nfull) load_x(xf[(u + STAGES - 1) % STAGES], kbeg + pre * SBK);
          compute(xf[u], u & 1);
          if (st + 1 < nfull) store_f(yv, (u + 1) & 1);
          __syncthreads();
        }
      }
    }
  }
  // K tail (fewer than 32 values): element loads, zero beyond kend
  const int64_t kt = kbeg + nfull * SBK;
  auto load_tail = [&](XStep<MT>& f) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t kk = kt + 8 * g + u;
        const int64_t kc = kk < kend ? kk : kt;
        const float v = TR ? X[kc * ldx + col0 + t] : xr[TR ? 0 : t][kc - 8 * g];
        f.v[t][u] = kk < kend ? v : 0.f;
      }
  };
  if (kt < kend) {
    XStep<MT> f;
    load_tail(f);
    const u32x4* src = Fp + (kt >> 3) * (3 * NR);   // zero past the last row
    for (int e = tid; e < CH; e += 64 * SPW) Fs[0][e] = src[e];
    __syncthreads();
    compute(f, 0);
  }
  if constexpr (FLUSH) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][j][r] += tot[t][j][r];
  }

  if constexpr (REM) {
    // lanes c < nrem: the sums with planes l, m and h of column c
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v = acc[t][NF][r];
        const float vm = __shfl(v, lane + nrem, 64), vl = __shfl(v, lane + 2 * nrem, 64);
        acc[t][NF][r] = c < nrem ? (vl + vm) + v : 0.f;
      }
  }
  // Where the scaled sums are not finite (an entry that is not, or of magnitude
  // 2^111 and up, or a result of 2^96 and up) the wave computes its tiles again
  // with the float instruction, step by step as above. Where all waves do
  // (entries of 1e15 on both sides), 30000^2 at k = 50 takes 2.2 ms (A H^T) and
  // 2.0 (A^T W) where ordinary entries take 0.86 and 0.71 and the float
  // instruction alone took 1.1 and 1.4; four K values at a time, one memory
  // latency each, took 3.4 and 2.7.
  bool redo = false;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        redo = redo || !(fabsf(acc[t][j][r]) <= 3.402823466e38f);
        acc[t][j][r] *= SPLIT_UNSCALE;
      }
  if (__ballot(redo)) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a step's product u takes K values k0 + 8 g + u, as load_x has them; the
    // factor's rows come from the L2, the next step's X is in flight
    auto step = [&](const XStep<MT>& f, int64_t k0) {
      constexpr int UB = NT <= 4 ? 8 : 4;   // rows of the factor in registers
#pragma unroll
      for (int u0 = 0; u0 < 8; u0 += UB) {
        float y[UB][NT];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int64_t kk = k0 + 8 * g + u0 + u, kc = kk < kend ? kk : kbeg;
#pragma unroll
          for (int j = 0; j < NT; ++j) y[u][j] = F[kc * ldf + (16 * j + c < kv ? 16 * j + c : 0)];
        }
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const float v = k0 + 8 * g + u0 + u < kend && 16 * j + c < kv ? y[u][j] : 0.f;
#pragma unroll
            for (int t = 0; t < MT; ++t) acc[t][j] = mfma16(f.v[t][u0 + u], v, acc[t][j]);
          }
      }
    };
    if (nfull > 0) load_x(xf[0], kbeg);
    for (int64_t s = 0; s < nfull; s += 2) {
      if (s + 1 < nfull) load_x(xf[1], kbeg + (s + 1) * SBK);
      step(xf[0], kbeg + s * SBK);
      if (s + 2 < nfull) load_x(xf[0], kbeg + (s + 2) * SBK);
      if (s + 1 < nfull) step(xf[1], kbeg + (s + 1) * SBK);
    }
    if (kt < kend) {
      load_tail(xf[0]);
      step(xf[0], kt);
    }
  }
  // element r of tile (t, j): row 4 g + r of the tile, column c
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = 4 * g + r;
      int64_t row = TR ? m0 + MT * rr : m0 + 16 * t + rr;
      bool in = row < M;
      if constexpr (TR) {
        row = (row < M - MT ? row : M - MT) + t;
        in = m0 < M;
      }
      if (in) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (16 * j + c < nout) D[row * ldd + 16 * j + c] = acc[t][j][r];
      }
    }
}

// The packed planes (split.h) of F (rows x kv, row pitch ldf), zero past kv
// and past the last row. One thread per group of 8 rows and column.
__global__ __launch_bounds__(256) void pack_split_kernel(const float* __restrict__ F, int64_t rows,
                                                         int64_t ldf, int kv, int KP,
                                                         u32x4* __restrict__ Fp) {
  const int64_t total = split_groups(rows) * KP, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
    const int64_t k8 = e / KP;
    const int i = (int)(e - k8 * KP);
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t r = 8 * k8 + u;
      x[u] = r < rows && i < kv ? F[r * ldf + i] : 0.f;
    }
    store_split_chunk(x, k8, KP, i, Fp);
  }
}

hipError_t pack_split(const float* F, int64_t rows, int64_t ldf, int kv, int KP, float* Fp,
                      hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (KP < 16 || KP > 128 || KP % 16 || kv < 1 || kv > KP || ldf < kv) return hipErrorInvalidValue;
  pack_split_kernel<<<capped_grid(cdiv(split_groups(rows) * KP, 256)), 256, 0, st>>>(
      F, rows, ldf, kv, KP, reinterpret_cast<u32x4*>(Fp));
  return NMF_LAUNCH_CHECK();
}

// X^T F for a single column of X (M = 1 of the TN form, whose lanes take at
// least two columns): thread (q, j) adds every Q-th product of output j.
__global__ __launch_bounds__(256) void column_product_kernel(
    const float* __restrict__ X, int64_t ldx, const float* __restrict__ F, int64_t ldf, int kv,
    float* __restrict__ D, int64_t dsplit, int KP, int nout, int64_t K, int64_t kchunk) {
  __shared__ double sh[256];
  const int Q = 256 / KP, j = threadIdx.x % KP, q = threadIdx.x / KP;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
  double s = 0.0;
  if (q < Q && j < kv)
    for (int64_t k = kbeg + q; k < kend; k += Q) s += (double)X[k * ldx] * (double)F[k * ldf + j];
  sh[threadIdx.x] = s;
  __syncthreads();
  if (q == 0 && j < nout) {
    for (int p = 1; p < Q; ++p) s += sh[p * KP + j];
    D[(int64_t)blockIdx.y * dsplit + j] = (float)s;
  }
}

// Launch shapes, from sweeps at k = 64 on MI355X. Two waves per SIMD and one
// step of X in flight ahead of the one being multiplied beat one wave with a
// deeper ring everywhere (65536^2: 3.2 against 3.6 ms). 64 rows (or columns)
// of A per wave halve the LDS reads of the factor per byte of A; their
// accumulators leave no registers for the second sum (FLUSH), so they are taken
// only where every slab stays at 8192 values, as float slabs did, with up to
// 2^28 elements of slabs in all (error 3.1e-7 there, 4.2e-7 with the float
// instruction; the matrix core cuts bits off, so it grows with the length:
// 70 x 2,000,003 of
// nonnegative entries in slabs of 62,501 was off by 2.9e-6, 3.5e-7 now). They pay from 2^27 entries of A at ranks up to 64
// (16384^2: 0.20 against 0.23 ms; 8192 x 4096: 0.037 against 0.032 ms);
// below, and at larger ranks, 32 per wave fill the chip better, and every 8
// steps their sums move to a second set of registers with one rounding, since
// the matrix core's own accumulation cuts bits off (error 5e-8 at any length
// up to 16384).
constexpr int SPLIT_WGS = 512;   // two workgroups per CU
constexpr int64_t WIDE_LEN = 8192, SLAB_ROOM = (int64_t)1 << 28;
static bool split_wide(int64_t M, int NT, int64_t K) {
  return NT <= 4 && M >= 64 && M * K >= ((int64_t)1 << 27) &&
         cdiv(K, WIDE_LEN) * M * 16 * NT <= SLAB_ROOM;
}

// Slabs: no longer than the shape allows (up to MAX_PRODUCT_SPLITS of them, or
// what the wide shape needs). From 2^23 entries of A on, the count with the
// fullest rounds of SPLIT_WGS workgroups (fullest_rounds): 7552 x 3136 at k = 6 364 ->
// 344 us a run of four HALS iterations, 1984 x 61888 968 -> 932, 20000^2 at k = 100
// 4.93 -> 4.58 ms. Below, doubled from one until the grid holds that many, then
// full_rounds: there a product is the latency of its slabs, and with fewer of
// them 2048 x 2000 at k = 6 252 -> 267 us. 20000^2 at k = 128:
// 3 slabs for 4 (471 workgroups for 628 on 512 places), 591 -> 501 us; 9000 x
// 7000 at k = 64: 76 -> 59 us; A^T W of 24000 x 16400 at k = 50: 15 for 8, 366 ->
// 304 us (A H^T, 5 for 8: 355 -> 367); 100003 x 5003 at k = 50: 588 -> 533 us (5 for
// 2) and 490 -> 460 us (25 for 32).
int64_t gemm_split_splits(int64_t M, int KP, int64_t K) {
  const bool wide = split_wide(M, KP / 16, K);
  const int64_t wgs = cdiv(M, (wide ? 64 : 32) * SPW), maxlen = wide ? WIDE_LEN : 16384;
  const int64_t minlen = M * K < ((int64_t)1 << 23) ? 64 : 128;
  auto room = [&](int64_t s) { return s * M * KP <= SLAB_ROOM; };
  const double cost = 2.0 * KP / (double)K;
  int64_t s = 1;
  if (M * K >= ((int64_t)1 << 23)) {
    while (K > s * maxlen && (wide || (s < MAX_PRODUCT_SPLITS && room(s + 1)))) ++s;
    const int64_t most = std::max(s, MAX_PRODUCT_SPLITS);
    return fullest_rounds(wgs, s, SPLIT_WGS, cost, [&](int64_t t) {
      return t <= most && K / t >= minlen && room(t);
    });
  }
  while (wgs * s < SPLIT_WGS && K / (2 * s) >= minlen && s < MAX_PRODUCT_SPLITS) s *= 2;
  while (K > s * maxlen && s < MAX_PRODUCT_SPLITS && room(2 * s)) s *= 2;
  return full_rounds(wgs, s, SPLIT_WGS, cost, [&](int64_t t) {
    return t <= MAX_PRODUCT_SPLITS && (t == 1 || K / t >= minlen) && (t <= s || room(t)) &&
           (K <= t * maxlen || (K > s * maxlen && t >= s));
  });
}

struct SplitCall {
  const float* X; int64_t ldx; const u32x4* Fp; const float* F; int64_t ldf; int kv;
  float* D; int64_t ldd, dsplit; int nout, nrem; int64_t M, K, kchunk, splits;
};

template <int NT, bool TR, int MT, int FLUSH, bool STREAM, bool REM = false>
static void split_launch(const SplitCall& a, hipStream_t st) {
  dim3 grid((unsigned)cdiv(a.M, 16 * MT * SPW), (unsigned)a.splits);
  gemm_split_kernel<NT, TR, MT, 2, 2, FLUSH, STREAM, REM><<<grid, 64 * SPW, 0, st>>>(
      a.X, a.ldx, a.Fp, a.F, a.ldf, a.kv, a.D, a.ldd, a.dsplit, a.nout, a.nrem, a.M, a.K,
      a.kchunk);
}

// STREAM (non-temporal loads of A): only where A is larger than the 256 MB
// last-level cache that would keep it for the next product (8192 x 4096:
// 0.039 against 0.037 ms), and only for TN, whose load instructions take
// whole 128-byte lines; NN's take half a line each, and the other half has to
// be in the cache when the second asks for it (65536^2: 3.7 against 3.3 ms).
template <int NT>
static void split_dispatch(bool tn, const SplitCall& a, hipStream_t st) {
  const bool stream = a.M * a.K > ((int64_t)1 << 26);
  if constexpr (NT <= 4) {
    if (split_wide(a.M, NT, a.K)) {
      if constexpr (NT >= 2) {
        if (a.nrem > 0 && a.nrem <= 5) {
          if (tn) split_launch<NT, true, 4, 0, true, true>(a, st);
          else split_launch<NT, false, 4, 0, false, true>(a, st);
          return;
        }
      }
      if (tn) split_launch<NT, true, 4, 0, true>(a, st);
      else split_launch<NT, false, 4, 0, false>(a, st);
      return;
    }
  }
  if (!tn) split_launch<NT, false, 2, 8, false>(a, st);
  else if (stream) split_launch<NT, true, 2, 8, true>(a, st);
  else split_launch<NT, true, 2, 8, false>(a, st);
}

hipError_t gemm_split(bool tn, const float* X, int64_t ldx, const float* Fp, const float* F,
                      int64_t ldf, int kv, int k, float* D, int64_t ldd, int nout, int64_t M,
                      int KP, int64_t K, float* part, hipStream_t st, int* nsplit) {
  if (KP < 16 || KP > 128 || KP % 16 || kv < 1 || kv > KP || k < 1 || k > kv || nout < 1 || nout > KP || M < 1 || K < 1)
    return hipErrorInvalidValue;
  if (ldx < (tn ? M : K) || ldf < kv || ldd < nout || (uintptr_t)Fp % 16) return hipErrorInvalidValue;
  int64_t splits = gemm_split_splits(M, KP, K);
  const int64_t kchunk = round_up(cdiv(K, splits), SBK);
  splits = cdiv(K, kchunk);
  const bool slabs = splits > 1;
  const SplitCall a{X, ldx, reinterpret_cast<const u32x4*>(Fp), F, ldf, kv, slabs ? part : D,
                    slabs ? KP : ldd, M * KP, slabs ? KP : nout, k > KP - 16 ? k - (KP - 16) : 0, M, K,
                    kchunk, splits};
  if (tn && M == 1) {
    column_product_kernel<<<dim3(1, (unsigned)splits), 256, 0, st>>>(
        X, ldx, F, ldf, kv, a.D, a.dsplit, KP, a.nout, K, kchunk);
  } else {
    switch (KP / 16) {
#define CASE(n) case n: split_dispatch<n>(tn, a, st); break;
      CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
    }
  }
  if (nsplit) *nsplit = (int)splits;
  const hipError_t e = NMF_LAUNCH_CHECK();
  if (e != hipSuccess || !slabs || nsplit) return e;
  return reduce_splits<float>(part, (int)splits, a.dsplit, M, nout, ldd, D, KP, st);
}

}  // namespace nmfk
