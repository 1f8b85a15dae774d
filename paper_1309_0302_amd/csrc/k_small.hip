// r x r FP64 work of the low-rank step (one workgroup each).
//
// Paper background (Sec. 3.1.2, Eq. 6-9; Algorithm 1): the power-scheme BRP
// needs the QR factors of Y2 = L~^T Y1 and Y1 = L~ Y2, the inverse of the
// r x r matrix A2^T Y1, a rank check on it, and the (2q+1)-th root of the
// r x r core.  With A2 = Y1 these are, exactly:
//   Y2 = (D^T D)^p A1 = Q2 R2        (R2 tracked through the passes below),
//   A2^T Y1 = R2^T R2                (rank check on the singular values of R2),
//   core = R factor of B = L~ Q2     (so L = U_B S_B^{1/p} V_B^T Q2^T).
// The power chain orthonormalises every pass (Cholesky QR with an FP64
// Gram) and keeps the product of the R factors in FP64, rescaled by exact
// powers of two.  B is handled through K = V diag(s^{(1-p)/p}) V^T from
// the eigen-decomposition of B^T B, so that U_L = B K and V_L = Q2.
#include <algorithm>

#include "godec_internal.h"
#include "k_common.h"
#include "k_chol.h"
#include "k_mmb.h"

namespace godec {

// Work items of one round of the eigen-solver: the 2 x 2 blocks of A on and
// above the diagonal (rounded up to whole wavefronts), then the (row, pair)
// items of V.
template <int RP>
constexpr int jacobi_blocks() { return (RP / 2) * (RP / 2 + 1) / 2; }
template <int RP>
constexpr int jacobi_items() { return (jacobi_blocks<RP>() + 63) / 64 * 64 + RP * (RP / 2); }
// Threads of the core: one per entry of an RP x RP matrix and per item of a
// round, up to 704 (RP = 32: two entries for some).
template <int RP>
constexpr int core_threads() {
  int t = RP * RP > jacobi_items<RP>() ? RP * RP : jacobi_items<RP>();
  t = (t + 63) / 64 * 64;
  if (t < 128) t = 128;   // at least one wave for each matrix
  return t < 704 ? t : 704;
}

// Sum of entry e over nparts partial matrices of `stride` doubles, with
// independent accumulators so the loads overlap.
__device__ __forceinline__ double sum_parts(const double* __restrict__ P, int nparts, int stride,
                                            int e) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int b = 0;
  for (; b + 3 < nparts; b += 4) {
    a0 += P[(int64_t)(b + 0) * stride + e];
    a1 += P[(int64_t)(b + 1) * stride + e];
    a2 += P[(int64_t)(b + 2) * stride + e];
    a3 += P[(int64_t)(b + 3) * stride + e];
  }
  for (; b < nparts; ++b) a0 += P[(int64_t)b * stride + e];
  return (a0 + a1) + (a2 + a3);
}

// ---------------------------------------------------------------------------
// Cholesky QR of a panel in two launches: k_gram_part writes partial Grams,
// k_chol_rinv adds them, factors the sum and applies R^{-1} to the rows.
//
// Bound: latency.  Handing the partials over inside one launch (write-through
// stores, two levels of arrival counters, the last block factors, a second
// launch for R^{-1}) took 19 + 5.7 us at 10000 x 20, of which 6 us the tree
// and 6 us the factorisation in a block that runs its code cold.  The kernel
// boundary does the hand-over, and every block adds the partials and factors
// on its own: 5.6 + 10.9 us; 1503 x 20: 17.3 + 5.7 -> 5.6 + 10.0 us; 25 344 x 4:
// 9.7 + 3.9 -> 4.0 + 4.6 us.
//
// A partial holds the 4 x 4 tiles of G on and above the diagonal (whole
// matrix when RP < 4), added in a fixed order everywhere: G is the same bits
// on every run.
// ---------------------------------------------------------------------------
template <int RP>
struct GramTile {
  static constexpr int T4 = (RP + 3) / 4;          // tiles per side
  static constexpr int RW = 4 * T4;                // padded width
  static constexpr int NT = T4 * (T4 + 1) / 2;     // tiles on and above the diagonal
  static constexpr int ENT = RP >= 4 ? NT * 16 : RP * RP;   // doubles of a partial
};

// Tile t in row-major order of the upper triangle.
template <int T4>
__device__ __forceinline__ void gram_tile(int t, int& ta, int& tb) {
  ta = 0;
  while (t >= T4 - ta) { t -= T4 - ta; ++ta; }
  tb = ta + t;
}

// Block b sums P[i]^T P[i] over its `per` rows (a multiple of kGramRows).
// Each thread owns a 4 x 4 tile (two 16-byte LDS reads per 16 multiply-adds;
// with 2 x 2 tiles the LDS reads bounded the loop) over the rows of its
// group.  With Zpart (FP32 panels only), the panel is first formed here: row
// i, column c of P is the sum over h < nch of Zpart[(h rows + i) zs + c] in
// ascending h (the row-chunk partials of a matrix-core Gram pass), and is
// also stored to P.
template <typename TA, int RP>
__global__ __launch_bounds__(256) void k_gram_part(TA* __restrict__ P, int64_t rows, int64_t per,
                                                   double* __restrict__ Gpart,
                                                   const float* __restrict__ Zpart, int nch) {
  using GT = GramTile<RP>;
  constexpr int T4 = GT::T4, RW = GT::RW, NT = GT::NT, CH = kGramRows;
  constexpr int NG = 256 / NT < CH ? 256 / NT : CH;   // row groups
  constexpr int RS = NT * 16;
  constexpr int PER = (CH * T4 + 255) / 256;          // 4-column pieces per thread
  constexpr size_t kPs = sizeof(TA) * CH * RW, kRed = sizeof(double) * NG * RS;
  __shared__ __align__(16) char buf[kPs > kRed ? kPs : kRed];
  TA* ps = reinterpret_cast<TA*>(buf);
  double* red = reinterpret_cast<double*>(buf);
  const int tid = threadIdx.x;
  const int tile = tid % NT, grp = tid / NT;
  const bool active = grp < NG;
  int ta, tb;
  gram_tile<T4>(tile, ta, tb);
  double acc[4][4] = {};
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int64_t r1 = (r0 + per) < rows ? (r0 + per) : rows;
  for (int64_t i0 = r0; i0 < r1; i0 += CH) {
    const int nr = (r1 - i0) < CH ? (int)(r1 - i0) : CH;
    TA x[PER][4];
#pragma unroll
    for (int j = 0; j < PER; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) x[j][c] = TA(0);
    if (Zpart != nullptr) {
      // four chunk partials of every piece in flight at once
      constexpr int HB = 4;
      const int64_t hstride = rows * RW;   // zpart_stride(RP) == RW
      for (int h0 = 0; h0 < nch; h0 += HB) {
        float4 v[HB][PER];
#pragma unroll
        for (int h = 0; h < HB; ++h)
#pragma unroll
          for (int j = 0; j < PER; ++j) {
            const int q = tid + 256 * j;
            v[h][j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (h0 + h < nch && q < nr * T4)
              v[h][j] = *reinterpret_cast<const float4*>(Zpart + (h0 + h) * hstride + i0 * RW +
                                                         4 * (int64_t)q);
          }
#pragma unroll
        for (int h = 0; h < HB; ++h)
#pragma unroll
          for (int j = 0; j < PER; ++j) {
            if (h0 + h >= nch) continue;
            x[j][0] += v[h][j].x;
            x[j][1] += v[h][j].y;
            x[j][2] += v[h][j].z;
            x[j][3] += v[h][j].w;
          }
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int q = tid + 256 * j;
        if (q >= nr * T4) continue;
        if constexpr (RW == RP) {
#pragma unroll
          for (int c = 0; c < 4; ++c) P[i0 * RP + 4 * (int64_t)q + c] = x[j][c];
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (c < RP) P[(i0 + q) * RP + c] = x[j][c];
            else x[j][c] = TA(0);
          }
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int q = tid + 256 * j;
        if (q >= nr * T4) continue;
        if constexpr (RW == RP) {
          load4(P + i0 * RP + 4 * (int64_t)q, x[j]);
        } else {
#pragma unroll
          for (int c = 0; c < RP; ++c) x[j][c] = P[(i0 + q) * RP + c];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int q = tid + 256 * j;
      if (q < CH * T4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) ps[4 * q + c] = x[j][c];
      }
    }
    __syncthreads();
    if (active) {
      for (int ii = grp; ii < nr; ii += NG) {
        TA u[4], w[4];
        load4(ps + ii * RW + 4 * ta, u);
        load4(ps + ii * RW + 4 * tb, w);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int d = 0; d < 4; ++d) acc[c][d] = fma((double)u[c], (double)w[d], acc[c][d]);
      }
    }
  }
  // the groups' tiles, added over the groups: part p of an entry takes the
  // groups p, p + PARTS, ..., then the parts are added
  __syncthreads();
  if (active) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int d = 0; d < 4; ++d) red[(grp * NT + tile) * 16 + 4 * c + d] = acc[c][d];
  }
  __syncthreads();
  constexpr int PARTS = 256 / RS < 1 ? 1 : (256 / RS < NG ? 256 / RS : NG);
  double* gp = Gpart + (int64_t)blockIdx.x * GT::ENT;
  auto put = [&](int e, double v) {
    if constexpr (RP >= 4) {
      gp[e] = v;
    } else {
      if (e / 4 < RP && e % 4 < RP) gp[e / 4 * RP + e % 4] = v;
    }
  };
  if constexpr (PARTS == 1) {
    for (int e = tid; e < RS; e += 256) {
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < NG; ++g) s += red[g * RS + e];
      put(e, s);
    }
  } else {
    const int e = tid % RS, p = tid / RS;
    double s = 0.0;
    if (p < PARTS) {
#pragma unroll 8
      for (int g = p; g < NG; g += PARTS) s += red[g * RS + e];
    }
    __syncthreads();
    if (p < PARTS) red[p * RS + e] = s;
    __syncthreads();
    if (tid < RS) {
      s = 0.0;
#pragma unroll
      for (int g = 0; g < PARTS; ++g) s += red[g * RS + tid];
      put(tid, s);
    }
  }
}

// G (LDS, stride LD) = the sum of nparts partials of k_gram_part, by NT
// threads (all call it; two barriers): pairs of entries, the partials dealt
// to NT / pairs groups, up to 20 loads in flight per thread (a load of lines that
// other XCDs have just written takes about 2000 cycles).  scratch: NT pairs.
template <int RP, int NT, int LD>
__device__ __forceinline__ void gram_sum(const double* __restrict__ Gpart, int nparts, double* G,
                                         double* scratch) {
  using GT = GramTile<RP>;
  constexpr int VW = GT::ENT % 2 ? 1 : 2;
  constexpr int Q = GT::ENT / VW;
  constexpr int SG = NT / Q > 0 ? NT / Q : 1;
  constexpr int NQ = (Q + NT - 1) / NT;   // pairs per thread (one group only)
  const int tid = threadIdx.x;
  auto put = [&](int e, double v) {
    if constexpr (RP < 4) {
      G[e / RP * LD + e % RP] = v;
    } else {
      int ta, tb;
      gram_tile<GT::T4>(e / 16, ta, tb);
      const int i = 4 * ta + e % 16 / 4, j = 4 * tb + e % 4;
      G[i * LD + j] = v;
      if (ta != tb) G[j * LD + i] = v;
    }
  };
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const int q = NQ > 1 ? tid + u * NT : tid % Q, g = NQ > 1 ? 0 : tid / Q;
    const bool on = NQ > 1 ? q < Q : g < SG;
    double s[VW] = {};
    if (on) {
      const double* p = Gpart + VW * q;
      constexpr int B = RP >= 12 ? 20 : 10;
      for (int h = g; h < nparts; h += B * SG) {
        double v[B][VW];
#pragma unroll
        for (int k = 0; k < B; ++k)
#pragma unroll
          for (int x = 0; x < VW; ++x)
            v[k][x] = h + k * SG < nparts ? p[(int64_t)(h + k * SG) * GT::ENT + x] : 0.0;
#pragma unroll
        for (int k = 0; k < B; ++k)
#pragma unroll
          for (int x = 0; x < VW; ++x) s[x] += v[k][x];
      }
    }
    if constexpr (SG == 1) {
      if (on)
#pragma unroll
        for (int x = 0; x < VW; ++x) put(VW * q + x, s[x]);
    } else {
      if (on)
#pragma unroll
        for (int x = 0; x < VW; ++x) scratch[VW * tid + x] = s[x];
      __syncthreads();
      if (tid < Q) {
#pragma unroll
        for (int x = 0; x < VW; ++x) {
          double v = 0.0;
#pragma unroll 8
          for (int k = 0; k < SG; ++k) v += scratch[VW * (k * Q + tid) + x];
          put(VW * tid + x, v);
        }
      }
    }
  }
  __syncthreads();
}

// Out = P R^{-1} with G = R^T R the sum of the partials (k_chol.h; R upper
// triangular, zero rows and 1/diag = 0 on inactive columns), by forward
// substitution in FP64, one row per thread of waves 1 and 2 (their loads run
// beside wave 0's factorisation); optionally also the transposed panel Zt (32
// x ldz) in bf16 or f32 for the next matrix-core pass, rows >= RP zero, and
// Ot = Out^T (RP x ldz).  With acc, the last block only folds R into it (acc <-
// R acc, or R with reset_acc), rescaled by a power of two when normalise is set.
//
// kRinvRows rows per block: the LDS reads of R bound the substitution, so the
// rows are spread over many CUs (256 rows on four waves: 6000 of the block's
// 30000 cycles at RP = 20), each of which adds and factors the same G.
constexpr int kRinvRows = 128;
template <int RP>
constexpr int rinv_threads() { return RP >= 12 ? 512 : 256; }

template <typename TA, int RP, typename TT>
__global__ __launch_bounds__(rinv_threads<RP>()) void k_chol_rinv(
    const TA* __restrict__ P, int64_t rows, const double* __restrict__ Gpart, int nparts,
    const SmallState* __restrict__ st, double* __restrict__ acc, int reset_acc, int normalise,
    TA* __restrict__ Out, TT* __restrict__ Zt, int64_t ldz, TA* __restrict__ Ot) {
  constexpr int NT = rinv_threads<RP>();
  __shared__ double Gs[RP * RP], rq[RP * RP], di[RP];
  __shared__ double scratch[2 * NT];
  const int tid = threadIdx.x;
  const int nrow = (int)gridDim.x - (acc != nullptr ? 1 : 0);   // blocks with rows
  const bool fold = (int)blockIdx.x == nrow;
  const int lr = tid - 64;
  const bool rowlane = !fold && lr >= 0 && lr < kRinvRows;
  CholIn<RP> cin;
  if (tid < 64) chol_prefetch<RP>(cin, st, fold ? acc : nullptr, reset_acc);
  gram_sum<RP, NT, RP>(Gpart, nparts, Gs, scratch);
  TA p[RP];
  auto load_row = [&](int64_t i) {
    if constexpr (RP % 4 == 0) {
#pragma unroll
      for (int c = 0; c < RP; c += 4) {
        TA v[4];
        load4(P + i * RP + c, v);
#pragma unroll
        for (int d = 0; d < 4; ++d) p[c + d] = v[d];
      }
    } else {
#pragma unroll
      for (int c = 0; c < RP; ++c) p[c] = P[i * RP + c];
    }
  };
  int64_t i = (int64_t)blockIdx.x * kRinvRows + lr;
  if (rowlane && i < rows) load_row(i);
  if (tid < 64) wave_chol<TA, RP>(Gs, rq, di, fold ? acc : nullptr, reset_acc, normalise, cin);
  __syncthreads();
  if (!rowlane) return;
  for (; i < rows; i += (int64_t)nrow * kRinvRows) {
    if (i >= (int64_t)nrow * kRinvRows) load_row(i);
    double y[RP], x[RP];
#pragma unroll
    for (int c = 0; c < RP; ++c) y[c] = (double)p[c];
    row_rinv<RP>(y, rq, di, x);
#pragma unroll
    for (int j = 0; j < RP; ++j) Out[i * RP + j] = (TA)x[j];
    if (Ot != nullptr) {
#pragma unroll
      for (int j = 0; j < RP; ++j) Ot[(int64_t)j * ldz + i] = (TA)x[j];
    }
    if (Zt != nullptr) {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const float v = j < RP ? (float)x[j] : 0.f;
        if constexpr (sizeof(TT) == 2)
          Zt[(int64_t)j * ldz + i] = f32_to_bf16(v);
        else
          Zt[(int64_t)j * ldz + i] = (TT)v;
      }
    }
  }
}

// Rotation threshold of the Jacobi sweeps: an off-diagonal entry below
// 4 u sqrt(|a_pp a_qq|) (u = 2^-53) is already at rounding level.
constexpr double kJacobiTol = 4.0 * 0x1p-53;
// A sweep whose rotations all had |a_pq| <= 2^-34 sqrt(a_pp a_qq) leaves the
// off-diagonal at about the square of that (quadratic convergence of cyclic
// Jacobi), far below kJacobiTol, so the confirming sweep is skipped.
constexpr double kJacobiQuad = 0x1p-34;

// Round-robin pairing (circle method) over N (even) players.
__device__ __forceinline__ void rr_pair(int round, int k, int N, int& a, int& b) {
  auto pos = [&](int i) { return i == 0 ? 0 : 1 + ((i - 1 + round) % (N - 1)); };
  a = pos(k);
  b = pos(N - 1 - k);
}

// The rotations that zero two entries a_pq: c and s, whether each is above
// rounding level, and whether it is large enough that another sweep is
// needed.  With
// d = a_qq - a_pp, h = 2 a_pq, r = hypot(d, h): c^2 = (1 + |d| / r) / 2 and
// s = sgn(d) h / (2 r c).  The matrix is scaled to a largest entry of about
// 1, so squares stay in range; blocks below 2^-500 of it are left alone.
// Step by step for both: each is one chain of dependent FP64 operations, and
// without branches the two interleave (one after the other: 490 cycles).
__device__ __forceinline__ void jacobi_rot2(const double (&app)[2], const double (&aqq)[2],
                                            const double (&apq)[2], double (&c)[2],
                                            double (&s)[2], bool (&did)[2], bool (&big)[2]) {
  double d[2], h[2], x[2], y[2], f[2], e[2], c2[2], z[2], g[2];
#define GODEC_PAIR _Pragma("unroll") for (int u = 0; u < 2; ++u)
  GODEC_PAIR d[u] = aqq[u] - app[u];
  GODEC_PAIR h[u] = 2.0 * apq[u];
  GODEC_PAIR x[u] = h[u] * h[u];
  GODEC_PAIR x[u] = fma(d[u], d[u], x[u]);
  GODEC_PAIR y[u] = __builtin_amdgcn_rsq(x[u]);
  // |a_pq| > tol sqrt(|a_pp a_qq|), compared on squares
  GODEC_PAIR {
    const double prod = fabs(app[u] * aqq[u]), apq2 = apq[u] * apq[u];
    did[u] = apq2 > kJacobiTol * kJacobiTol * prod && fabs(apq[u]) > 0x1p-500;
    big[u] = did[u] && apq2 > kJacobiQuad * kJacobiQuad * prod;
  }
  // y = 1 / sqrt(x): one third-order step from the hardware estimate, whose
  // relative error of at most 2^-23 becomes about 2^-69 before rounding
  GODEC_PAIR x[u] = x[u] * y[u];
  GODEC_PAIR e[u] = fma(-x[u], y[u], 1.0);
  GODEC_PAIR f[u] = fma(0.375, e[u], 0.5);
  GODEC_PAIR e[u] = y[u] * e[u];
  GODEC_PAIR y[u] = fma(e[u], f[u], y[u]);
  GODEC_PAIR d[u] = 0.5 * fabs(d[u]);
  GODEC_PAIR c2[u] = fma(d[u], y[u], 0.5);
  GODEC_PAIR z[u] = __builtin_amdgcn_rsq(c2[u]);
  GODEC_PAIR g[u] = (aqq[u] - app[u] >= 0.0 ? apq[u] : -apq[u]) * y[u];
  GODEC_PAIR x[u] = c2[u] * z[u];
  GODEC_PAIR e[u] = fma(-x[u], z[u], 1.0);
  GODEC_PAIR f[u] = fma(0.375, e[u], 0.5);
  GODEC_PAIR e[u] = z[u] * e[u];
  GODEC_PAIR z[u] = fma(e[u], f[u], z[u]);
  GODEC_PAIR c[u] = did[u] ? c2[u] * z[u] : 1.0;
  GODEC_PAIR s[u] = did[u] ? g[u] * z[u] : 0.0;
#undef GODEC_PAIR
}

// C = op(A) B for RP x RP matrices in LDS (stride RP + 1), op the transpose
// with TA_.  2 x 2 outputs per thread: half the LDS reads of one output per
// thread, which bound the product.  `keep(i, j, v)` stores an entry.
template <int RP, int NT, bool TA_, typename F>
__device__ __forceinline__ void small_mm(const double* A, const double* B, F keep) {
  constexpr int LD = RP + 1;
  constexpr int W = RP % 2 ? 1 : 2;   // outputs per side
  constexpr int S = RP / W;
  for (int e = threadIdx.x; e < S * S; e += NT) {
    const int i0 = e / S * W, j0 = e % S * W;
    double c[W][W] = {};
#pragma unroll
    for (int l = 0; l < RP; ++l) {
      double x[W], y[W];
#pragma unroll
      for (int u = 0; u < W; ++u) {
        x[u] = TA_ ? A[l * LD + i0 + u] : A[(i0 + u) * LD + l];
        y[u] = B[l * LD + j0 + u];
      }
#pragma unroll
      for (int u = 0; u < W; ++u)
#pragma unroll
        for (int v = 0; v < W; ++v) c[u][v] = fma(x[u], y[v], c[u][v]);
    }
#pragma unroll
    for (int u = 0; u < W; ++u)
#pragma unroll
      for (int v = 0; v < W; ++v) keep(i0 + u, j0 + v, c[u][v]);
  }
}

// Two-sided cyclic Jacobi on the symmetric matrix G (LDS, stride RP + 1),
// accumulating V <- V J.  G is zero outside its leading active block and V is
// the identity there, so the sweeps run over the full RP x RP at compile-time
// sizes: a pair that touches the padding has a_pq = 0 and is never rotated.
//
// Bound: latency.  A round is one LDS round trip, the chain of a rotation and
// one barrier.  The matrix is kept in slots, so that the pairs of every round
// are the slots (2k, 2k + 1): an item of A reads its 2 x 2 block and the
// diagonal blocks of its two pairs, computes both rotations itself, and writes
// its entries to the slots of the next round in the other buffer, where they
// are moved by the one permutation that steps the round-robin (circle
// method).  After RP - 1 rounds every index is back in its slot.  Only the
// blocks on and above the diagonal are kept (RP <= 20: one wave).  The other
// waves apply the rotations to V one round later, beside the next round of A.
// The form before (rotations by one wave, handed over through LDS, applied in
// place; two barriers and twice the LDS trips) took about 1 us per round;
// core at RP = 20: 68 to 78 -> 43 us, RP = 8: 32 -> 21 us.
//
// G holds the eigenvalues on its diagonal afterwards; the eigenvectors are
// the columns of the returned buffer (V or V1).  A0, A1, V1: scratch of the
// size of G; cs: 2 RP doubles.
template <int RP, int NT>
__device__ __forceinline__ double* jacobi_eig(double* G, double* V, double* A0, double* A1,
                                              double* V1, double* cs, int* rot) {
  if constexpr (RP == 1) {
    return V;
  } else {
    constexpr int LD = RP + 1;
    constexpr int NP = RP / 2;
    constexpr int NA = jacobi_blocks<RP>();
    constexpr int NAP = (NA + 63) / 64 * 64;
    constexpr int NV = RP * NP;
    constexpr int VT = NT - NAP;               // threads of V
    constexpr int IPT = (NV + VT - 1) / VT;    // items of V per thread
    static_assert(RP % 2 == 0 && VT >= 64, "pairs, and a wave for V");
    const int tid = threadIdx.x;
    // slot of circle position j, and the slot that slot s moves to
    auto slot = [](int j) { return j < NP ? 2 * j : 2 * (RP - 1 - j) + 1; };
    auto step = [&](int s) {
      const int j = (s & 1) ? RP - 1 - (s >> 1) : s >> 1;
      return slot(j == 0 ? 0 : (j == 1 ? RP - 1 : j - 1));
    };
    // addresses of this thread's item of A, the same in every round
    int src = 0, low = 0, d1 = 0, d2 = 0, w[4] = {}, diag = -1;
    if (tid < NA) {
      int k1 = 0, f = tid;
      while (f >= NP - k1) { f -= NP - k1; ++k1; }
      const int k2 = k1 + f;
      diag = k1 == k2 ? k1 : -1;
      src = 2 * k1 * LD + 2 * k2;
      low = k1 == k2 ? src + 1 : src + LD;   // below the diagonal: the entry above it
      d1 = 2 * k1 * (LD + 1);
      d2 = 2 * k2 * (LD + 1);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int i = step(2 * k1 + (x >> 1)), j = step(2 * k2 + (x & 1));
        w[x] = i < j ? i * LD + j : j * LD + i;
      }
    }
    // ... and of V: (row, pair)
    int vs[IPT], vk[IPT], vw[IPT][2];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
      const int f = tid - NAP + u * VT, i = f / NP, k = f % NP;
      vs[u] = f >= 0 && f < NV ? i * LD + 2 * k : -1;
      vk[u] = 2 * k;
      vw[u][0] = i * LD + step(2 * k);
      vw[u][1] = i * LD + step(2 * k + 1);
    }
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, j = e % RP;
      A0[slot(i) * LD + slot(j)] = G[i * LD + j];
      V1[i * LD + slot(j)] = V[i * LD + j];
    }
    if (tid < 2) rot[tid] = 0;
    __syncthreads();
    double *Ac = A0, *An = A1, *Vc = V1, *Vn = V, *cw = cs, *cr = cs + RP;
    auto apply_v = [&](const double* q) {
#pragma unroll
      for (int u = 0; u < IPT; ++u) {
        if (vs[u] < 0) continue;
        const double x = Vc[vs[u]], y = Vc[vs[u] + 1];
        const double c = q[vk[u]], s = q[vk[u] + 1];
        Vn[vw[u][0]] = fma(c, x, -(s * y));
        Vn[vw[u][1]] = fma(s, x, c * y);
      }
    };
    auto swap = [](double*& x, double*& y) { double* z = x; x = y; y = z; };
    for (int sweep = 0; sweep < 40; ++sweep) {
      bool any = false, anybig = false;
      for (int round = 0; round < RP - 1; ++round) {
        if (tid < NAP) {
          if (tid < NA) {
            // A <- J^T A J on the block (row pair k1) x (column pair k2)
            const double app[2] = {Ac[d1], Ac[d2]};
            const double apq[2] = {Ac[d1 + 1], Ac[d2 + 1]};
            const double aqq[2] = {Ac[d1 + LD + 1], Ac[d2 + LD + 1]};
            const double a0 = Ac[src], b0 = Ac[src + 1], g0 = Ac[low], e0 = Ac[src + LD + 1];
            double c[2], s[2];
            bool did[2], big[2];
            jacobi_rot2(app, aqq, apq, c, s, did, big);
            const double a2 = fma(c[1], a0, -(s[1] * b0)), b2 = fma(s[1], a0, c[1] * b0);
            const double g2 = fma(c[1], g0, -(s[1] * e0)), e2 = fma(s[1], g0, c[1] * e0);
            An[w[0]] = fma(c[0], a2, -(s[0] * g2));
            An[w[1]] = fma(c[0], b2, -(s[0] * e2));
            An[w[2]] = fma(s[0], a2, c[0] * g2);
            An[w[3]] = fma(s[0], b2, c[0] * e2);
            if (diag >= 0) {
              cw[2 * diag] = c[0];
              cw[2 * diag + 1] = s[0];
              any |= did[0];
              anybig |= big[0];
            }
          }
        } else if (sweep + round > 0) {
          apply_v(cr);
        }
        if (round == RP - 2) {
          if (any) rot[0] = 1;
          if (anybig) rot[1] = 1;
        }
        __syncthreads();
        swap(Ac, An);
        swap(cw, cr);
        if (sweep + round > 0) swap(Vc, Vn);
      }
      // converged when nothing was rotated, or by little enough
      if (rot[0] == 0 || rot[1] == 0) break;
      __syncthreads();
      // (the next writes of rot come a barrier later, or from this thread)
      if (tid < 2) rot[tid] = 0;
    }
    if (tid >= NAP) apply_v(cr);
    __syncthreads();
    swap(Vc, Vn);
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, j = e % RP;
      if (i == j) G[i * LD + i] = Ac[slot(i) * (LD + 1)];
      Vn[i * LD + j] = Vc[i * LD + slot(j)];
    }
    __syncthreads();
    return Vn;
  }
}

// In-place form for the batched core, whose problems keep their rounding: its
// FP32 results follow the last bits of this solver where small eigenvalues
// are noise.  One wave per problem (48 items a round at RP = 8, no barrier
// between waves; with 384 threads per problem 40 us for 32 problems, now
// 35).  The rotations of a round are computed first, then one pass applies
// them, a thread per 2 x 2 block of A (the column rotation of the block's
// column pair, then the row rotation of its row pair) and a thread per (row,
// pair) of V.
template <int RP, int NT>
__device__ __forceinline__ void jacobi_eig_inplace(double* A, double* V, double* cs, int* rot) {
  constexpr int LD = RP + 1;
  constexpr int N = (RP + 1) & ~1;
  constexpr int NP = N / 2;
  constexpr int NBLK = NP * NP;
  __shared__ int pq[2 * NP];
  auto pos = [](int i, int round) {
    if (i == 0) return 0;
    int x = i - 1 + round;
    if (x >= N - 1) x -= N - 1;
    return 1 + x;
  };
  for (int sweep = 0; sweep < 40; ++sweep) {
    int nrot = 0, nbig = 0;   // wave 0's counts (every pair lives in wave 0)
    for (int round = 0; round < N - 1; ++round) {
      if (threadIdx.x < 64) {
        const int k = threadIdx.x;
        bool did = false, big = false;
        if (k < NP) {
          // circle method: position i plays at 0 (fixed) or 1 + (i - 1 + round) mod (N - 1)
          int p = pos(k, round), q = pos(N - 1 - k, round);
          if (p > q) { const int t = p; p = q; q = t; }
          double c = 1.0, sn = 0.0;
          if (q < RP) {
            const double apq = A[p * LD + q];
            const double app = A[p * LD + p], aqq = A[q * LD + q];
            // |a_pq| > tol sqrt(|a_pp a_qq|), compared on squares
            const double prod = fabs(app * aqq), apq2 = apq * apq;
            if (apq2 > kJacobiTol * kJacobiTol * prod && apq != 0.0) {
              // tan of the rotation t = sgn(d) h / (|d| + r), d = a_qq - a_pp,
              // h = 2 a_pq, r = hypot(d, h); with w = sqrt(2 r (r + |d|)):
              // c = (r + |d|) / w, s = sgn(d) h / w.
              const double d = aqq - app, h = 2.0 * apq;
              const double mx = fmax(fabs(d), fabs(h));
              if (mx > 0x1p-450 && mx < 0x1p450) {
                const double r2 = d * d + h * h;
                const double r = r2 * rsqrt_nr(r2);
                const double iw = rsqrt_nr(2.0 * r * (r + fabs(d)));
                c = (r + fabs(d)) * iw;
                sn = (d >= 0.0 ? h : -h) * iw;
              } else {
                const double th = d / h;
                const double t = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                c = 1.0 / sqrt(t * t + 1.0);
                sn = t * c;
              }
              did = true;
              big = apq2 > kJacobiQuad * kJacobiQuad * prod;
            }
          }
          cs[2 * k + 0] = c;
          cs[2 * k + 1] = sn;
          pq[2 * k + 0] = p;
          pq[2 * k + 1] = q;
        }
        nrot += __popcll(__ballot(did));
        nbig += __popcll(__ballot(big));
      }
      __syncthreads();
      for (int e = threadIdx.x; e < NBLK + RP * NP; e += NT) {
        if (e >= NBLK) {
          // V <- V J
          const int f = e - NBLK;
          const int i = f / NP, k = f % NP;
          const double c = cs[2 * k], sn = cs[2 * k + 1];
          const int p = pq[2 * k], q = pq[2 * k + 1];
          if (q >= RP || sn == 0.0) continue;
          const double vip = V[i * LD + p], viq = V[i * LD + q];
          V[i * LD + p] = c * vip - sn * viq;
          V[i * LD + q] = sn * vip + c * viq;
          continue;
        }
        // A <- J^T A J on the block (row pair k1) x (column pair k2)
        const int k1 = e / NP, k2 = e % NP;
        const double c1 = cs[2 * k1], s1 = cs[2 * k1 + 1];
        const double c2 = cs[2 * k2], s2 = cs[2 * k2 + 1];
        if (s1 == 0.0 && s2 == 0.0) continue;
        const int p1 = pq[2 * k1], q1 = pq[2 * k1 + 1];
        const int p2 = pq[2 * k2], q2 = pq[2 * k2 + 1];
        const bool rq = q1 < RP, cq = q2 < RP;   // the partner may be the padding index
        double a = A[p1 * LD + p2];
        double b = cq ? A[p1 * LD + q2] : 0.0;
        double cc = rq ? A[q1 * LD + p2] : 0.0;
        double d = (rq && cq) ? A[q1 * LD + q2] : 0.0;
        if (s2 != 0.0) {
          const double a2 = c2 * a - s2 * b, b2 = s2 * a + c2 * b;
          const double c3 = c2 * cc - s2 * d, d2 = s2 * cc + c2 * d;
          a = a2; b = b2; cc = c3; d = d2;
        }
        if (s1 != 0.0) {
          const double a2 = c1 * a - s1 * cc, c3 = s1 * a + c1 * cc;
          const double b2 = c1 * b - s1 * d, d2 = s1 * b + c1 * d;
          a = a2; cc = c3; b = b2; d = d2;
        }
        A[p1 * LD + p2] = a;
        if (cq) A[p1 * LD + q2] = b;
        if (rq) A[q1 * LD + p2] = cc;
        if (rq && cq) A[q1 * LD + q2] = d;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) rot[0] = (nrot == 0 || nbig == 0) ? 1 : 0;
    __syncthreads();
    if (rot[0]) break;
    __syncthreads();
  }
}

// One-sided (Hestenes) Jacobi: orthogonalise the columns of M (n x n);
// afterwards the column norms are the singular values.
template <int RP>
__device__ void jacobi_svd_values(double* M, int n, double* out, double* cs, int* rot) {
  constexpr int LD = RP + 1;
  const int N = (n + 1) & ~1;
  const int npairs = N / 2;
  for (int sweep = 0; sweep < 60; ++sweep) {
    if (threadIdx.x == 0) *rot = 0;
    __syncthreads();
    for (int round = 0; round < N - 1; ++round) {
      if (threadIdx.x < npairs) {
        int p, q;
        rr_pair(round, threadIdx.x, N, p, q);
        double c = 1.0, s = 0.0;
        if (p < n && q < n) {
          double al = 0, be = 0, ga = 0;
          for (int i = 0; i < n; ++i) {
            const double x = M[i * LD + p], y = M[i * LD + q];
            al += x * x; be += y * y; ga += x * y;
          }
          if (ga != 0.0 && fabs(ga) > kJacobiTol * sqrt(al * be)) {
            const double ze = (be - al) / (2.0 * ga);
            const double t = (ze >= 0 ? 1.0 : -1.0) / (fabs(ze) + sqrt(1.0 + ze * ze));
            c = 1.0 / sqrt(1.0 + t * t);
            s = c * t;
            atomicAdd(rot, 1);
          }
        }
        cs[4 * threadIdx.x + 0] = c;
        cs[4 * threadIdx.x + 1] = s;
        cs[4 * threadIdx.x + 2] = (double)p;
        cs[4 * threadIdx.x + 3] = (double)q;
      }
      __syncthreads();
      for (int e = threadIdx.x; e < n * npairs; e += blockDim.x) {
        const int i = e / npairs, k = e % npairs;
        const double c = cs[4 * k], s = cs[4 * k + 1];
        const int p = (int)cs[4 * k + 2], q = (int)cs[4 * k + 3];
        if (p >= n || q >= n || s == 0.0) continue;
        const double x = M[i * LD + p], y = M[i * LD + q];
        M[i * LD + p] = c * x - s * y;
        M[i * LD + q] = s * x + c * y;
      }
      __syncthreads();
    }
    if (*rot == 0) break;
    __syncthreads();
  }
  if (threadIdx.x < n) {
    double s = 0;
    for (int i = 0; i < n; ++i) s += M[i * LD + threadIdx.x] * M[i * LD + threadIdx.x];
    out[threadIdx.x] = sqrt(s);
  }
  __syncthreads();
}

// Rank check on R2 (A2^T Y1 = R2^T R2), given in W (LDS, stride RP + 1; may be
// overwritten): the number of leading singular values that count.  H, fk, sv,
// cs, rot: scratch.
template <int RP, int NT>
__device__ __forceinline__ void core_rank(double* W, double* H, double* fk, double* sv, double* cs,
                                          int* rot, int n, double rank_tol, int* keep_out) {
  constexpr int LD = RP + 1;
  __shared__ double red[2];
  __shared__ double redA[NT / 64], redB[NT / 64];
  const int tid = threadIdx.x;
  // Certificate first: s_min(R2) >= 1/||R2^{-1}||_F and s_max <= ||R2||_F.
  // R2^{-1} (upper triangular, active block) by back substitution, one lane
  // per column in registers, into H; a zero diagonal fails the certificate.
  if (tid < 64) {
    const double dg = tid < n ? W[tid * LD + tid] : 1.0;
    if (tid < RP) fk[tid] = tid < n ? 1.0 / dg : 0.0;
    const bool ok = n > 0 && __ballot(!(dg != 0.0)) == 0ull;
    if (tid == 0) {
      red[1] = ok ? 1.0 : 0.0;
      *keep_out = n;
    }
    __builtin_amdgcn_wave_barrier();
    if (tid < RP) {
      double h[RP];
#pragma unroll
      for (int i = 0; i < RP; ++i) h[i] = (i == tid) ? 1.0 : 0.0;
#pragma unroll
      for (int i = RP - 1; i >= 0; --i) {
        h[i] *= fk[i];   // past n: zero
#pragma unroll
        for (int l = 0; l < i; ++l) h[l] -= W[l * LD + i] * h[i];
      }
#pragma unroll
      for (int i = 0; i < RP; ++i) H[i * LD + tid] = h[i];
    }
  }
  __syncthreads();
  {
    double fr = 0.0, fi = 0.0;
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, c = e % RP;
      if (c >= i && c < n) {
        fr += W[i * LD + c] * W[i * LD + c];
        fi += H[i * LD + c] * H[i * LD + c];
      }
    }
    fr = wave_sum(fr);
    fi = wave_sum(fi);
    if ((tid & 63) == 0) { redA[tid >> 6] = fr; redB[tid >> 6] = fi; }
    __syncthreads();
    if (tid == 0) {
      double a = 0, b = 0;
      for (int w = 0; w < NT / 64; ++w) { a += redA[w]; b += redB[w]; }
      const bool ok = red[1] != 0.0 && isfinite(a) && isfinite(b) && (1.0 / b) > rank_tol * a;
      red[0] = ok ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  if (red[0] == 0.0 && n > 0) {
    jacobi_svd_values<RP>(W, n, sv, cs, rot);
    if (tid == 0) {
      double smax = 0.0;
      for (int i = 0; i < n; ++i) smax = fmax(smax, sv[i]);
      int keep = 0;
      for (int i = 0; i < n; ++i)
        if (smax > 0.0 && sv[i] * sv[i] > rank_tol * smax * smax) ++keep;
      *keep_out = keep;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Core of the low-rank step.  Inputs: Gpart of B' = D Y_q (so B = B' T; nparts
// partials, those of k_gram_part or RP x RP matrices),
// st->T, st->R2.  Output: K' = T K in the panel type, such that
// U_L = B' K' and L = U_L Q2^T.
// ---------------------------------------------------------------------------
template <typename TA, int RP, int NT>
__device__ __forceinline__ void core_body(const double* __restrict__ Gpart, int nparts,
                                          int tiled, SmallState* st, int p, double rank_tol,
                                          int t_identity, TA* k_panel) {
  constexpr int LD = RP + 1;
  __shared__ double G[RP * LD];
  __shared__ double H[RP * LD];
  __shared__ double T[RP * LD];
  __shared__ double V[RP * LD];
  __shared__ double W[RP * LD];
  __shared__ double V1[RP * LD];
  __shared__ double cs[4 * 16 + 4];
  __shared__ double ev[RP];
  __shared__ double fk[RP];
  __shared__ double sv[RP];
  __shared__ int order[RP];
  __shared__ int rot[2];
  __shared__ int sh_keep;
  const int tid = threadIdx.x;
  const int n = st->r_eff;             // active leading columns
  __shared__ double scratch[2 * NT];
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    if (!tiled) G[i * LD + j] = sum_parts(Gpart, nparts, RP * RP, e);
    T[i * LD + j] = t_identity ? (i == j ? 1.0 : 0.0) : st->T[e];
    W[i * LD + j] = st->R2[e];
  }
  if (tiled) gram_sum<RP, NT, LD>(Gpart, nparts, G, scratch);
  __syncthreads();

  core_rank<RP, NT>(W, H, fk, sv, cs, rot, n, rank_tol, &sh_keep);

  // ---- A = M^T G' M on the active block, M = T or, with a warm start from
  // the previous iteration's eigenvectors, T V ----
  const int warm = st->v_valid;
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    V[i * LD + j] = warm ? st->V[e] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  const double* M = T;
  if (warm) {
    small_mm<RP, NT, false>(T, V, [&](int i, int j, double v) { V1[i * LD + j] = v; });
    __syncthreads();
    M = V1;
  }
  small_mm<RP, NT, false>(G, M, [&](int i, int j, double v) { H[i * LD + j] = v; });
  __syncthreads();
  small_mm<RP, NT, true>(M, H, [&](int i, int j, double v) {
    W[i * LD + j] = (i < n && j < n) ? v : 0.0;
  });
  __syncthreads();
  // symmetrised, and scaled by a power of two to a largest diagonal of about 1
  double mx = 0.0;
#pragma unroll
  for (int i = 0; i < RP; ++i) mx = fmax(mx, fabs(W[i * LD + i]));
  int sce = 0;
  if (mx > 0.0 && isfinite(mx)) frexp(mx, &sce);
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    G[i * LD + j] = ldexp(0.5 * (W[i * LD + j] + W[j * LD + i]), -sce);
  }
  __syncthreads();
  const double* E = jacobi_eig<RP, NT>(G, V, H, W, V1, cs, rot);
  // sort eigenvalues descending (rank of each by counting; ties by index)
  if (tid < n) {
    const double mine = G[tid * LD + tid];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double o = G[j * LD + j];
      rank += (o > mine || (o == mine && j < tid)) ? 1 : 0;
    }
    order[rank] = tid;
    ev[rank] = ldexp(mine, sce);
  }
  __syncthreads();
  const int keep = sh_keep;
  // K = sum_{i < keep, ev_i > 0} v_i ev_i^{(1-p)/(2p)} v_i^T
  const double ex = (1.0 - (double)p) / (2.0 * (double)p);
  if (tid < RP) {
    const double lam = tid < n ? ev[tid] : 0.0;
    fk[tid] = (tid < keep && lam > 0.0) ? ((p == 1) ? 1.0 : pow(lam, ex)) : 0.0;
    if (tid >= n) order[tid] = tid;
  }
  __syncthreads();
  // E's columns in descending order, and those columns times fk, transposed
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    const double x = E[i * LD + order[j]];
    G[j * LD + i] = x;
    W[j * LD + i] = x * fk[j];   // fk is zero where nothing is kept
    st->V[e] = (j < n && i < n) ? x : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  small_mm<RP, NT, true>(G, W, [&](int i, int j, double v) {
    H[i * LD + j] = (i < n && j < n) ? v : 0.0;
  });
  __syncthreads();
  // K' = T K ; the sorted eigenvectors are the next warm start
  int bad = 0;
  small_mm<RP, NT, false>(T, H, [&](int i, int j, double v) {
    if (!isfinite(v)) bad = 1;
    st->K[i * RP + j] = v;
    k_panel[i * RP + j] = (TA)v;
  });
  if (bad) atomicOr(&st->flags, 1);
  if (tid < RP) {
    st->sigma[tid] = (tid < n && ev[tid] > 0.0) ? sqrt(ev[tid]) : 0.0;
    st->sv_c[tid] = 0.0;
  }
  if (tid == 0) {
    st->r_keep = keep;
    st->v_valid = (keep == n) ? 1 : 0;
    if (keep < n) {
      st->r_eff = keep;
      atomicOr(&st->flags, 2);
    }
  }
}

template <typename TA, int RP>
__global__ __launch_bounds__(core_threads<RP>()) void k_core(const double* __restrict__ Gpart,
                                                        int nparts, int tiled, SmallState* st,
                                                        int p, double rank_tol, int t_identity,
                                                        TA* k_panel) {
  core_body<TA, RP, core_threads<RP>()>(Gpart, nparts, tiled, st, p, rank_tol, t_identity,
                                        k_panel);
}

__global__ void k_small_init(SmallState* st, int r) {
  const int tid = threadIdx.x;
  for (int e = tid; e < kMaxRP * kMaxRP; e += blockDim.x) {
    st->R2[e] = 0.0; st->T[e] = 0.0; st->Rq[e] = 0.0; st->V[e] = 0.0; st->K[e] = 0.0;
  }
  if (tid < kMaxRP) {
    st->sigma[tid] = 0.0; st->sv_c[tid] = 0.0; st->dinv[tid] = 0.0; st->active[tid] = tid < r;
  }
  if (tid == 0) { st->r_eff = r; st->r_keep = r; st->flags = 0; st->v_valid = 0; }
}

#define GODEC_RP_SWITCH(rp, ...)                   \
  switch (rp) {                                    \
    case 1: { constexpr int RP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int RP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int RP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int RP = 8; __VA_ARGS__; } break;   \
    case 12: { constexpr int RP = 12; __VA_ARGS__; } break; \
    case 16: { constexpr int RP = 16; __VA_ARGS__; } break; \
    case 20: { constexpr int RP = 20; __VA_ARGS__; } break; \
    case 24: { constexpr int RP = 24; __VA_ARGS__; } break; \
    case 32: { constexpr int RP = 32; __VA_ARGS__; } break; \
    default: break;                                \
  }

int launch_gram_part(const Launch& L, bool f64, int rp, void* P, int64_t rows, double* Gpart,
                     const float* Zpart, int nch) {
  const int64_t steps = std::max<int64_t>(1, (rows + kGramRows - 1) / kGramRows);
  const int64_t per = (steps + kGramMaxBlocks - 1) / kGramMaxBlocks * kGramRows;
  const int64_t nb = std::max<int64_t>(1, (rows + per - 1) / per);
  GODEC_RP_SWITCH(rp, {
    if (f64)
      hipLaunchKernelGGL((k_gram_part<double, RP>), dim3((unsigned)nb), dim3(256), 0, L.stream,
                         (double*)P, rows, per, Gpart, nullptr, 0);
    else
      hipLaunchKernelGGL((k_gram_part<float, RP>), dim3((unsigned)nb), dim3(256), 0, L.stream,
                         (float*)P, rows, per, Gpart, Zpart, nch);
  });
  return (int)nb;
}

void launch_chol_rinv(const Launch& L, bool f64, int rp, const void* P, int64_t rows,
                      const double* Gpart, int nparts, const SmallState* st, double* acc,
                      int reset_acc, int normalise, void* Out, DType zt_type, void* Zt,
                      int64_t ldz, void* Ot) {
  // two blocks per CU at most: longer panels take several rows per thread
  const int64_t nrow = std::min<int64_t>((rows + kRinvRows - 1) / kRinvRows, 2LL * L.num_cu);
  const dim3 g((unsigned)(nrow + (acc != nullptr ? 1 : 0)));
  GODEC_RP_SWITCH(rp, {
    if (f64)
      hipLaunchKernelGGL((k_chol_rinv<double, RP, double>), g, dim3(rinv_threads<RP>()), 0, L.stream,
                         (const double*)P, rows, Gpart, nparts, st, acc, reset_acc, normalise,
                         (double*)Out, (double*)nullptr, ldz, (double*)Ot);
    else if (Zt != nullptr && zt_type == BF16)
      hipLaunchKernelGGL((k_chol_rinv<float, RP, uint16_t>), g, dim3(rinv_threads<RP>()), 0, L.stream,
                         (const float*)P, rows, Gpart, nparts, st, acc, reset_acc, normalise,
                         (float*)Out, (uint16_t*)Zt, ldz, (float*)Ot);
    else
      hipLaunchKernelGGL((k_chol_rinv<float, RP, float>), g, dim3(rinv_threads<RP>()), 0, L.stream,
                         (const float*)P, rows, Gpart, nparts, st, acc, reset_acc, normalise,
                         (float*)Out, (float*)Zt, ldz, (float*)Ot);
  });
}

void launch_core(const Launch& L, bool f64, int rp, const double* Gpart,
                 int nparts, int tiled, SmallState* st, int p, double rank_tol,
                 int t_identity, void* k_panel) {
  GODEC_RP_SWITCH(rp, {
    if (f64)
      hipLaunchKernelGGL((k_core<double, RP>), dim3(1), dim3(core_threads<RP>()), 0, L.stream, Gpart,
                         nparts, tiled, st, p, rank_tol, t_identity, (double*)k_panel);
    else
      hipLaunchKernelGGL((k_core<float, RP>), dim3(1), dim3(core_threads<RP>()), 0, L.stream, Gpart,
                         nparts, tiled, st, p, rank_tol, t_identity, (float*)k_panel);
  });
}

void launch_small_init(const Launch& L, SmallState* st, int r) {
  hipLaunchKernelGGL(k_small_init, dim3(1), dim3(256), 0, L.stream, st, r);
}

}  // namespace godec

namespace godec {

// ---------------------------------------------------------------------------
// Batched r x r work: one workgroup per problem, 8-column panels.
// ---------------------------------------------------------------------------
constexpr int RB = kBatchRP;

__device__ __forceinline__ float* bpanel_rw(const BProb& b, int which) {
  return which == 0 ? b.P0 : (which == 1 ? b.P1 : b.VL);
}

// out = orth(Z) by one Cholesky QR step with an FP64 Gram, Z = the sum of the
// problem's Gram-pass partials (fixed order) or panel `in`; R folded into
// R2 (acc 0, rescaled by powers of two) or T (acc 1).
__global__ __launch_bounds__(256) void kb_chol(const BProb* __restrict__ probs,
                                               const BItem* __restrict__ items,
                                               const float* __restrict__ zslots, int from_slots,
                                               int in, int out, int acc_sel, int reset) {
  __shared__ float zs[kBatchMaxN * RB];
  __shared__ double gp[4][RB * RB];
  __shared__ double G[RB * RB];
  __shared__ double rq[RB * RB];
  __shared__ double di[RB];
  const BProb& b = probs[blockIdx.x];
  const int tid = threadIdx.x;
  const int n = (int)b.n;
  const int ne = n * RB;
  if (from_slots) {
    for (int e = tid; e < ne; e += 256) {
      float s = 0.f;
      for (int it = 0; it < b.nitems; ++it) s += zslots[items[b.item0 + it].zoff + e];
      zs[e] = s;
    }
  } else {
    const float* P = bpanel_rw(b, in);
    for (int e = tid; e < ne; e += 256) zs[e] = P[e];
  }
  __syncthreads();
  {
    const int e = tid % (RB * RB), h = tid / (RB * RB);
    const int a = e / RB, c = e % RB;
    double s = 0.0;
    for (int j = h; j < n; j += 4) s = fma((double)zs[j * RB + a], (double)zs[j * RB + c], s);
    gp[h][e] = s;
  }
  __syncthreads();
  if (tid < RB * RB) G[tid] = (gp[0][tid] + gp[1][tid]) + (gp[2][tid] + gp[3][tid]);
  __syncthreads();
  if (tid < 64) {
    double* acc = acc_sel == 0 ? b.st->R2 : b.st->T;
    wave_chol<float, RB>(G, b.st, acc, reset, acc_sel == 0 ? 1 : 0);
  }
  __syncthreads();
  if (tid < RB * RB) rq[tid] = b.st->Rq[tid];
  if (tid < RB) di[tid] = b.st->dinv[tid];
  __syncthreads();
  float* O = bpanel_rw(b, out);
  for (int j = tid; j < n; j += 256) {
    double x[RB];
#pragma unroll
    for (int c = 0; c < RB; ++c) {
      double s = (double)zs[j * RB + c];
#pragma unroll
      for (int l = 0; l < c; ++l) s = fma(-x[l], rq[l * RB + c], s);
      x[c] = s * di[c];
    }
#pragma unroll
    for (int c = 0; c < RB; ++c) O[j * RB + c] = (float)x[c];
  }
}

// The same for the batched path (jacobi_eig_inplace).
template <typename TA, int RP, int NT>
__device__ __forceinline__ void core_body_inplace(const double* __restrict__ Gpart, int nparts,
                                                  SmallState* st, int p, double rank_tol,
                                                  int t_identity, TA* k_panel) {
  constexpr int LD = RP + 1;
  __shared__ double G[RP * LD];
  __shared__ double H[RP * LD];
  __shared__ double T[RP * LD];
  __shared__ double V[RP * LD];
  __shared__ double W[RP * LD];
  __shared__ double cs[4 * 16 + 4];
  __shared__ double ev[RP];
  __shared__ double fk[RP];
  __shared__ double sv[RP];
  __shared__ int order[RP];
  __shared__ int rot[2];
  __shared__ int sh_keep;
  const int tid = threadIdx.x;
  const int n = st->r_eff;             // active leading columns
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    G[i * LD + j] = sum_parts(Gpart, nparts, RP * RP, e);
    T[i * LD + j] = t_identity ? (i == j ? 1.0 : 0.0) : st->T[e];
    W[i * LD + j] = st->R2[e];
  }
  __syncthreads();

  core_rank<RP, NT>(W, H, fk, sv, cs, rot, n, rank_tol, &sh_keep);

  // ---- G_B = T^T G' T on the active block ----
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    double s = 0.0;
    for (int l = 0; l <= j; ++l) s += G[i * LD + l] * T[l * LD + j];
    H[i * LD + j] = s;
  }
  __syncthreads();
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    double s = 0.0;
    for (int l = 0; l <= i; ++l) s += T[l * LD + i] * H[l * LD + j];
    W[i * LD + j] = (i < n && j < n) ? s : 0.0;
  }
  __syncthreads();
  // symmetrise and set V (warm start from the previous iteration if valid)
  const int warm = st->v_valid;
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    G[i * LD + j] = 0.5 * (W[i * LD + j] + W[j * LD + i]);
    V[i * LD + j] = warm ? st->V[e] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  if (warm) {
    // A = V^T G V
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, j = e % RP;
      double s = 0.0;
      for (int l = 0; l < n; ++l) s += G[i * LD + l] * V[l * LD + j];
      H[i * LD + j] = s;
    }
    __syncthreads();
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, j = e % RP;
      double s = 0.0;
      for (int l = 0; l < n; ++l) s += V[l * LD + i] * H[l * LD + j];
      W[i * LD + j] = s;
    }
    __syncthreads();
    for (int e = tid; e < RP * RP; e += NT) {
      const int i = e / RP, j = e % RP;
      G[i * LD + j] = 0.5 * (W[i * LD + j] + W[j * LD + i]);
    }
    __syncthreads();
  }
  jacobi_eig_inplace<RP, NT>(G, V, cs, rot);
  // sort eigenvalues descending (rank of each by counting; ties by index)
  if (tid < n) {
    const double mine = G[tid * LD + tid];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double o = G[j * LD + j];
      rank += (o > mine || (o == mine && j < tid)) ? 1 : 0;
    }
    order[rank] = tid;
    ev[rank] = mine;
  }
  __syncthreads();
  const int keep = sh_keep;
  // K = sum_{i < keep, ev_i > 0} v_i ev_i^{(1-p)/(2p)} v_i^T
  const double ex = (1.0 - (double)p) / (2.0 * (double)p);
  if (tid < n) {
    const double lam = ev[tid];
    fk[tid] = (tid < keep && lam > 0.0) ? ((p == 1) ? 1.0 : pow(lam, ex)) : 0.0;
  }
  __syncthreads();
  for (int e = tid; e < RP * RP; e += NT) {
    const int a = e / RP, b = e % RP;
    double s = 0.0;
    if (a < n && b < n) {
      for (int i = 0; i < keep; ++i) {
        if (!(ev[i] > 0.0)) continue;
        s += V[a * LD + order[i]] * fk[i] * V[b * LD + order[i]];
      }
    }
    H[a * LD + b] = s;
  }
  __syncthreads();
  // K' = T K ; store eigenvectors (sorted) for the next warm start
  int bad = 0;
  for (int e = tid; e < RP * RP; e += NT) {
    const int i = e / RP, j = e % RP;
    double s = 0.0;
    for (int l = i; l < RP; ++l) s += T[i * LD + l] * H[l * LD + j];
    if (!isfinite(s)) bad = 1;
    st->K[e] = s;
    k_panel[e] = (TA)s;
    st->V[e] = (j < n && i < n) ? V[i * LD + order[j]] : (i == j ? 1.0 : 0.0);
  }
  if (bad) atomicOr(&st->flags, 1);
  if (tid < RP) {
    st->sigma[tid] = (tid < n && ev[tid] > 0.0) ? sqrt(ev[tid]) : 0.0;
    st->sv_c[tid] = 0.0;
  }
  if (tid == 0) {
    st->r_keep = keep;
    st->v_valid = (keep == n) ? 1 : 0;
    if (keep < n) {
      st->r_eff = keep;
      atomicOr(&st->flags, 2);
    }
  }
}

// Core of the low-rank step per problem: the Gram of B' from the apply
// pass's partials, then the shared FP64 core (rank certificate, Jacobi
// eigen-solver, K' = T K into Kp).
__global__ __launch_bounds__(64) void kb_core(const BProb* __restrict__ probs,
                                              const double* __restrict__ gslots, int p,
                                              int t_identity) {
  const BProb& b = probs[blockIdx.x];
  core_body_inplace<float, RB, 64>(gslots + (int64_t)b.item0 * RB * RB, b.nitems, b.st, p,
                                   b.rank_tol, t_identity, b.Kp);
}

__global__ void kb_small_init(const BProb* __restrict__ probs) {
  const BProb& b = probs[blockIdx.x];
  SmallState* st = b.st;
  const int tid = threadIdx.x;
  for (int e = tid; e < kMaxRP * kMaxRP; e += blockDim.x) {
    st->R2[e] = 0.0; st->T[e] = 0.0; st->Rq[e] = 0.0; st->V[e] = 0.0; st->K[e] = 0.0;
  }
  if (tid < kMaxRP) {
    st->sigma[tid] = 0.0; st->sv_c[tid] = 0.0; st->dinv[tid] = 0.0; st->active[tid] = tid < b.r;
  }
  if (tid == 0) { st->r_eff = b.r; st->r_keep = b.r; st->flags = 0; st->v_valid = 0; }
}

void bl_chol(const Launch& L, const BatchArgs& a, int from_slots, int in, int out, int acc,
             int reset) {
  hipLaunchKernelGGL(kb_chol, dim3((unsigned)a.nprob), dim3(256), 0, L.stream, a.probs, a.items,
                     a.zslots, from_slots, in, out, acc, reset);
}

void bl_core(const Launch& L, const BatchArgs& a, int t_identity) {
  hipLaunchKernelGGL(kb_core, dim3((unsigned)a.nprob), dim3(64), 0, L.stream, a.probs,
                     a.gslots, a.p, t_identity);
}

void bl_small_init(const Launch& L, const BatchArgs& a) {
  hipLaunchKernelGGL(kb_small_init, dim3((unsigned)a.nprob), dim3(256), 0, L.stream, a.probs);
}

}  // namespace godec
