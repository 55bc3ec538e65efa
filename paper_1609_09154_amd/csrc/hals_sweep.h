// The HALS sweep (Section 4.2, Eq. (5)) on the row layout, instantiated for one
// element type per source file (hals_f32.hip, hals_f64.hip): its fully unrolled
// loops over the rank take most of the library's compile time.
#pragma once

#include "common.h"
#include "rowtile.h"
#include "kernels.h"

namespace nmfk {

// HALS sweep with a group of TPR lanes per row: lane `sub` of a group owns
// entries sub*R .. sub*R + R - 1 of the row (R = KP / TPR) and the matching
// products. Step i forms (x G)_i from the owners' partial sums (group_sum,
// the same bits on every lane of the group) and the owner of entry i updates
// it. G is staged in LDS with column i contiguous (Gs[i][j] = G[j][i]), so a
// lane reads its R entries of the column with one vector load. Rows past the
// end run on a clamped copy of the last row (every lane must join the group
// sums) and store nothing. TPR (4, 8 or 16 lanes per row) is chosen from the
// number of rows: many rows fill the chip with small groups, which take fewer
// permutation steps per column; few rows need larger groups to fill it.
// With TILE (KP <= 64), after the sweep the LDS that held G takes the
// block's new rows (zero past the end) for the copy the next product reads (Xt,
// nullable) and the block's share of Xn^T Xn (Gslab + blockIdx.x * KP * KP,
// nullable), formed on the matrix cores. The tile shares G's space; only at
// 64 rows per block does its padding need more (17 KB against 16 KB at KP =
// 64), which the form without TILE, for calls that want neither output,
// does not take.
// Xs (nullable) scales the incoming rows first, x_i *= Xs[i] where Xs[i] > 0
// (the normalisation's compensation of H, applied as the sweep reads the rows
// rather than by a pass of its own; the same product, so the same bits).
template <typename T, int KP, int TPR, bool SLABS, bool TILE>
__global__ __launch_bounds__(256) void hals_rows_grp_kernel(const T* X, T* Xn, Split<T> P,
                                                            const T* __restrict__ G,
                                                            int64_t rows, int k,
                                                            T* __restrict__ Xt,
                                                            T* __restrict__ Gslab,
                                                            const T* __restrict__ Xscale,
                                                            FactorCopy copy) {
  constexpr int R = KP / TPR, ROWS = 256 / TPR;
  constexpr int VEC = Tr<T>::VEC;
  constexpr int XLD = KP + VEC;
  constexpr int TS = TILE && KP <= 64 ? ROWS * XLD : 0;
  constexpr int LS = KP * KP > TS ? KP * KP : TS;
  __shared__ __attribute__((aligned(16))) T Ls[LS];
  T* Gs = Ls;
  const int sub = threadIdx.x % TPR;
  const int64_t rb = (int64_t)blockIdx.x * ROWS;
  const int64_t r = rb + threadIdx.x / TPR;
  const int64_t rr = r < rows ? r : rows - 1;
  // G's loads, the row's x and its entries of P (summed from the slabs in
  // slab order in double), all in flight together
  SquareStage<T, KP, 256> gst;
  gst.load(G, nullptr);
  T x[R], p[R];
#pragma unroll
  for (int q = 0; q < R; ++q) x[q] = X[rr * KP + sub * R + q];
  if (Xscale) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const T sc = Xscale[sub * R + q];
      if (sc > T(0)) x[q] = x[q] * sc;
    }
  }
  if constexpr (SLABS) {
    double ps[R];
#pragma unroll
    for (int q = 0; q < R; ++q) ps[q] = 0.0;
    slab_sum<T, R>(P.p + rr * KP + sub * R, P.n, P.stride, ps);
#pragma unroll
    for (int q = 0; q < R; ++q) p[q] = (T)ps[q];
  } else {
    // one slab: the product itself (a sum of one term rounds to itself)
#pragma unroll
    for (int q = 0; q < R; ++q) p[q] = P.p[rr * KP + sub * R + q];
  }
  gst.store_t(Gs);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    if (i < k) {
      const T gii = Gs[i * KP + i];
      if (gii > T(0)) {
        const T* gc = &Gs[i * KP + sub * R];
        T part = T(0);
#pragma unroll
        for (int q = 0; q < R; ++q) part = fma(x[q], gc[q], part);
        const T s = group_sum<TPR>(part);
        if (sub == i / R) {
          const T t = x[i % R] + (p[i % R] - s) / gii;
          x[i % R] = t > T(0) ? t : T(0);
        }
      }
    }
  }
  if (r < rows) {
#pragma unroll
    for (int q = 0; q < R; ++q) Xn[r * KP + sub * R + q] = x[q];
  }
  if constexpr (TILE && KP <= 64) {
    if (Xt == nullptr && Gslab == nullptr) return;  // uniform over the block
    __syncthreads();  // every read of G is done
    const bool in = r < rows;
#pragma unroll
    for (int q = 0; q < R; ++q) Ls[(threadIdx.x / TPR) * XLD + sub * R + q] = in ? x[q] : T(0);
    __syncthreads();
    if (Gslab) block_gram_partial<T, KP, ROWS, XLD>(Ls, Ls, Gslab + (int64_t)blockIdx.x * KP * KP);
    if (Xt) store_rows_copy<T, KP, ROWS, XLD>(Ls, rb, rows, Xt, copy);
  }
}

template <typename T, int KP, bool SLABS, bool TILE>
void launch_hals_grp_t(const T* X, T* Xn, Split<T> P, const T* G, int64_t rows, int k, int tpr,
                       T* Xt, T* Gslab, const T* Xs, FactorCopy copy, hipStream_t st) {
  if (tpr == 4)
    hals_rows_grp_kernel<T, KP, 4, SLABS, TILE><<<(unsigned)cdiv(rows, 64), 256, 0, st>>>(
        X, Xn, P, G, rows, k, Xt, Gslab, Xs, copy);
  else if (tpr == 8)
    hals_rows_grp_kernel<T, KP, 8, SLABS, TILE><<<(unsigned)cdiv(rows, 32), 256, 0, st>>>(
        X, Xn, P, G, rows, k, Xt, Gslab, Xs, copy);
  else
    hals_rows_grp_kernel<T, KP, 16, SLABS, TILE><<<(unsigned)cdiv(rows, 16), 256, 0, st>>>(
        X, Xn, P, G, rows, k, Xt, Gslab, Xs, copy);
}

// One slab (the product as it came) needs no double accumulation: that form
// keeps the small register footprint that lets many blocks share a CU.
template <typename T, int KP>
void launch_hals_grp(const T* X, T* Xn, Split<T> P, const T* G, int64_t rows, int k, int tpr,
                     T* Xt, T* Gslab, const T* Xs, FactorCopy copy, hipStream_t st) {
  if constexpr (KP <= 64) {
    if (Xt || Gslab) {
      if (P.n > 1)
        launch_hals_grp_t<T, KP, true, true>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st);
      else
        launch_hals_grp_t<T, KP, false, true>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st);
      return;
    }
  }
  if (P.n > 1) launch_hals_grp_t<T, KP, true, false>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st);
  else launch_hals_grp_t<T, KP, false, false>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st);
}

template <typename T>
hipError_t hals_rows(const T* X, T* Xn, Split<T> P, const T* G, int64_t rows, int k, int KP,
                     T* Xt, T* Gslab, hipStream_t st, const T* Xs, FactorCopy copy) {
  if (rows <= 0) return hipSuccess;
  if (((Xt || Gslab) && KP > 64) || !P.p || P.n < 1) return hipErrorInvalidValue;
  const int tpr = hals_tpr(rows);
  // every padded rank up to NMF_MAX_K takes the grouped sweep; G (KP x KP)
  // is staged in LDS, at most 64 KB (float) or 128 KB (double) at KP = 128
  switch (KP) {
    case 16: launch_hals_grp<T, 16>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 32: launch_hals_grp<T, 32>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 48: launch_hals_grp<T, 48>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 64: launch_hals_grp<T, 64>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 80: launch_hals_grp<T, 80>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 96: launch_hals_grp<T, 96>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 112: launch_hals_grp<T, 112>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    case 128: launch_hals_grp<T, 128>(X, Xn, P, G, rows, k, tpr, Xt, Gslab, Xs, copy, st); break;
    default: return hipErrorInvalidValue;
  }
  return NMF_LAUNCH_CHECK();
}

}  // namespace nmfk
