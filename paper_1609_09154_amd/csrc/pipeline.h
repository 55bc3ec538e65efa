// The register pipeline of the product kernels that read both operands from
// memory (gemm_f64.hip, gemm_f32.hip).
#pragma once

// ---------------------------------------------------------------------------
// Software pipeline over K steps. LOAD(buf, k0) issues the global loads of
// one step into a register buffer, COMPUTE(buf) runs its MFMAs. With three
// buffers the loads of step s+2 are in flight while step s computes.
// ---------------------------------------------------------------------------
// S-stage ring: buffer j % S holds step j; the loads of step s + S - 1 are
// issued before the MFMAs of step s. The steady-state loop body is unrolled S
// times so every buffer index is a compile-time constant and no branch sits
// between a load and its use.
#define NMF_PIPELINE(S, LOAD, COMPUTE, F, KBEG, NSTEPS, STEPK)                             \
  {                                                                                       \
    const int64_t n_ = (NSTEPS);                                                          \
    if (n_ < (S) - 1) {                                                                   \
      for (int64_t s_ = 0; s_ < n_; ++s_) {                                               \
        LOAD(F[0], (KBEG) + s_ * (STEPK));                                                \
        COMPUTE(F[0]);                                                                    \
      }                                                                                   \
    } else {                                                                              \
      _Pragma("unroll") for (int j_ = 0; j_ < (S) - 1; ++j_)                              \
        LOAD(F[j_], (KBEG) + j_ * (STEPK));                                               \
      int64_t s_ = 0;                                                                     \
      for (; s_ + 2 * (S) - 1 <= n_; s_ += (S)) {                                         \
        _Pragma("unroll") for (int j_ = 0; j_ < (S); ++j_) {                              \
          LOAD(F[(j_ + (S) - 1) % (S)], (KBEG) + (s_ + j_ + (S) - 1) * (STEPK));          \
          COMPUTE(F[j_]);                                                                 \
        }                                                                                 \
      }                                                                                   \
      _Pragma("unroll") for (int j_ = 0; j_ < 2 * (S) - 2; ++j_) {                        \
        if (s_ + j_ < n_) {                                                               \
          if (s_ + j_ + (S) - 1 < n_)                                                     \
            LOAD(F[(j_ + (S) - 1) % (S)], (KBEG) + (s_ + j_ + (S) - 1) * (STEPK));        \
          COMPUTE(F[j_ % (S)]);                                                           \
        }                                                                                 \
      }                                                                                   \
    }                                                                                     \
  }
