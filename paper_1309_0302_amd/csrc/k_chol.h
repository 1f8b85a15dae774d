// Cholesky step of Cholesky QR: G = R^T R, upper R, by one wavefront (lane j
// holds column j of G in registers, broadcasts by readlane).  A column is
// inactive when it lies at or past r_eff, is zero, or is numerically
// dependent on the columns before it: its pivot (the squared norm of its
// component orthogonal to them) is at most tau * G_jj with
// tau = RP * max(u^2, 2^-53), the resolution of a Gram of panel-type data
// accumulated in FP64.  An inactive column gets a zero row in R and
// dinv = 0, so the orthonormalised panel has a zero column, which stays zero
// in every later product.
#pragma once

#include "godec_internal.h"
#include "k_common.h"

namespace godec {

__device__ __forceinline__ double lane_bcast(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Global inputs of wave_chol (the active width and, lane j, column j of the
// accumulated factor), loaded ahead so that their latency overlaps other work.
template <int RP> struct CholIn {
  int reff;
  double b[RP];
};
template <int RP>
__device__ __forceinline__ void chol_prefetch(CholIn<RP>& in, const SmallState* st,
                                              const double* acc, int reset_acc) {
  const int lane = threadIdx.x & 63;
  in.reff = st->r_eff;
#pragma unroll
  for (int l = 0; l < RP; ++l)
    in.b[l] = (acc != nullptr && !reset_acc && lane < RP) ? acc[l * RP + lane] : 0.0;
}

// One wavefront (lanes 0..63); G is RP x RP row-major in LDS, and is
// overwritten with R (LDS scratch for the broadcast reads of R below).  R and
// the reciprocal diagonal go to Rq (RP x RP) and dinv; acc may be null.
template <typename TA, int RP>
__device__ __forceinline__ void wave_chol(double* G, double* Rq, double* dinv, double* acc,
                                          int reset_acc, int normalise, const CholIn<RP>& in) {
  const int lane = threadIdx.x & 63;
  const bool col = lane < RP;
  const int reff = in.reff;
  double g[RP];
#pragma unroll
  for (int i = 0; i < RP; ++i) g[i] = col ? G[i * RP + lane] : 0.0;
  const double g0 = col ? G[lane * RP + lane] : 0.0;
  const double u = sizeof(TA) == 8 ? 0x1p-53 : 0x1p-24;
  const double tau = (double)RP * fmax(u * u, 0x1p-53);
  int act = (col && lane < reff && g0 > 0.0) ? 1 : 0;
  double rcol[RP];   // rcol[k] = R[k][lane]
  double rdiag = 0.0;
#pragma unroll
  for (int k = 0; k < RP; ++k) {
    const double piv = lane_bcast(g[k], k);
    const double g0k = lane_bcast(g0, k);
    const int actk = __builtin_amdgcn_readlane(act, k) && piv > tau * g0k;
    if (lane == k) act = actk;
    // no branch on actk: the updates of a step fill the latency of the next
    // step's reciprocal square root
    const double inv = rsqrt_nr(piv);
    const double rkk = piv * inv;
    double rkj = lane > k ? g[k] * inv : (lane == k ? rkk : 0.0);
    rkj = actk ? rkj : 0.0;
    rdiag = actk && lane == k ? rkk : rdiag;
    rcol[k] = rkj;
#pragma unroll
    for (int i = k + 1; i < RP; ++i) g[i] -= lane_bcast(rkj, i) * rkj;
  }
  if (col) {
#pragma unroll
    for (int k = 0; k < RP; ++k) Rq[k * RP + lane] = rcol[k];
    dinv[lane] = act ? 1.0 / rdiag : 0.0;
  }
  if (acc == nullptr) return;
  // acc <- R acc (or R); lane j owns column j
  double a[RP];
  if (reset_acc) {
#pragma unroll
    for (int i = 0; i < RP; ++i) a[i] = rcol[i];
  } else {
    // R through LDS (G is no longer needed): every lane reads R[i][l] at the
    // same address, a broadcast, instead of a readlane pair per term
    __builtin_amdgcn_wave_barrier();
    if (col) {
#pragma unroll
      for (int i = 0; i < RP; ++i) G[i * RP + lane] = rcol[i];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      double s = 0.0;
#pragma unroll
      for (int l = i; l < RP; ++l) s += G[i * RP + l] * in.b[l];
      a[i] = s;
    }
  }
  // R2 only enters through ratios of its singular values, so it may be
  // rescaled by a power of two; T must keep its scale (B = B' T).
  if (normalise) {
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < RP; ++i) mx = fmax(mx, fabs(a[i]));
    mx = wave_max(mx);
    int e = 0;
    if (mx > 0.0 && isfinite(mx)) frexp(mx, &e);
    const double sc = ldexp(1.0, -e);
#pragma unroll
    for (int i = 0; i < RP; ++i) a[i] *= sc;
  }
  if (col) {
#pragma unroll
    for (int i = 0; i < RP; ++i) acc[i * RP + lane] = a[i];
  }
}

template <typename TA, int RP>
__device__ __forceinline__ void wave_chol(double* G, SmallState* st, double* acc, int reset_acc,
                                          int normalise) {
  CholIn<RP> in;
  chol_prefetch<RP>(in, st, acc, reset_acc);
  wave_chol<TA, RP>(G, st->Rq, st->dinv, acc, reset_acc, normalise, in);
}

// Row x of P R^{-1}: x R = y by forward substitution (R upper triangular, zero
// rows and dinv = 0 on inactive columns).  Right-looking: the updates of a
// step are independent, and a row of R is contiguous; the next row is read
// ahead, and no further one (all of R in registers spills).
template <int RP>
__device__ __forceinline__ void row_rinv(const double (&y)[RP], const double* Rq,
                                         const double* dinv, double (&x)[RP]) {
  double r[2][RP];
#pragma unroll
  for (int c = 0; c < RP; ++c) x[c] = y[c];
#pragma unroll
  for (int l = 0; l < RP; ++l) r[0][l] = l == 0 ? dinv[0] : Rq[l];
#pragma unroll
  for (int c = 0; c < RP; ++c) {
    if (c + 1 < RP) {
#pragma unroll
      for (int l = c + 1; l < RP; ++l)
        r[(c + 1) & 1][l] = l == c + 1 ? dinv[l] : Rq[(c + 1) * RP + l];
    }
    asm volatile("" ::: "memory");
    x[c] *= r[c & 1][c];
#pragma unroll
    for (int l = c + 1; l < RP; ++l) x[l] = fma(-x[c], r[c & 1][l], x[l]);
  }
}

}  // namespace godec
