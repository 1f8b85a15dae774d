// The L update of a narrow matrix through A = D^T D.
//
// Algorithm 1's power scheme (Eq. 6-9) applies D^T D to an n x r panel
// p + q times (p = 2q + 1), orthonormalising in between.  With n at most a
// few hundred columns A = D^T D is a small matrix, so it is formed once per
// iteration, in FP64 on the matrix cores, and the passes run on A:
//   kgf_gram, kgf_sum   A = D^T D (32 x 32 tiles over row ranges, then their
//                       sum in range order),
//   kgf_pass (x p + q)  Z = orth(last product), Y = A Z and the partials of
//                       Y^T Y for the next orthonormalisation,
//   kgf_pass (last)     C = Y_q^T A Y_q = B'^T B', the core's Gram matrix,
//   k_core              K' = T K as on the general path,
//   kgf_ul              U_L = D (Y_q K').
// Everything up to Y_q K' is FP64 (the general path rounds each panel to the type
// of X), and D is read twice per iteration instead of 2 (p + q) + 1 times.
//
// Why: on matrices like these the general path is a chain of short launches
// (two panel products, their partial sums, a Gram tree with the Cholesky step
// and the substitution, five launches and 30-45 us per pass), bound by
// latency and not by data.  Here a pass is one launch of n / 16 blocks: every
// thread repeats the r x r work (a few hundred FP64 operations) instead of
// waiting for one block that does it.
#include <hip/hip_ext.h>

#include "godec_internal.h"
#include "k_chol.h"
#include "k_common.h"

namespace godec {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4g __attribute__((ext_vector_type(4)));

constexpr int kGfSlabs = kGfMaxN / 16;  // most blocks of a pass
constexpr int kGfMaxK = kGfMaxN / 32;   // MFMA steps of a wave over its eighth of n

// v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and,
// in register v, C[4 v + l / 16][l % 16].
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Tile (ti, tj), ti >= tj, number t of the lower triangle.
__device__ __forceinline__ void tile_of(int t, int& ti, int& tj) {
  ti = 0;
  while (t > ti) {
    t -= ti + 1;
    ++ti;
  }
  tj = t;
}

// part[s][tile] = (D[:, tile ti])^T D[:, tile tj] over the rows of range s.
// Block: one 32 x 32 tile (the last, partly empty columns cost little at this
// size); its waves take the range's 32-row steps in turn, operands straight
// from memory (16 columns x 4 rows per load) and the next step in flight
// while the current one is multiplied, and their tiles are added in wave
// order.  Bound: the FP64 matrix cores: 25 344 x 200 FP32 takes 47 us, 41
// without the loads of D (35 TFLOP/s; independent products alone reach 40
// with two waves per SIMD).  64 x 64 tiles, more of them past n and above the
// diagonal, took 48; three or four blocks per CU instead of two 44.
template <typename T>
__global__ __launch_bounds__(256) void kgf_gram(const T* __restrict__ D, int64_t ldd,
                                                int64_t mpad, int64_t rows_per,
                                                double* __restrict__ part) {
  constexpr int KS = kGfStep / 4;
  constexpr int EL = kGfTile * kGfTile;
  __shared__ double red[4][EL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int ti, tj;
  tile_of((int)blockIdx.x, ti, tj);
  const int64_t r0 = (int64_t)blockIdx.y * rows_per + kGfStep * wave;
  const int64_t re = (int64_t)(blockIdx.y + 1) * rows_per;
  const int64_t r1 = re < mpad ? re : mpad;
  const int g = lane >> 4, i = lane & 15;
  const T* pa = D + kGfTile * ti + i;
  const T* pb = D + kGfTile * tj + i;
  T a[2][KS], b[2][KS];
  auto load = [&](int64_t r) {
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[h][s] = pa[(r + 4 * s + g) * ldd + 16 * h];
        b[h][s] = pb[(r + 4 * s + g) * ldd + 16 * h];
      }
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (r0 < r1) load(r0);   // wave-uniform
  for (int64_t r = r0; r < r1; r += 4 * kGfStep) {
    double ca[2][KS], cb[2][KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ca[h][s] = (double)a[h][s];
        cb[h][s] = (double)b[h][s];
      }
    if (r + 4 * kGfStep < r1) load(r + 4 * kGfStep);   // uniform
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = mfma64(ca[x][s], cb[y][s], acc[x][y]);
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[wave][(16 * x + 4 * v + g) * kGfTile + 16 * y + i] = acc[x][y][v];
  __syncthreads();
  double* out = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * EL;
  for (int e = threadIdx.x; e < EL; e += 256)
    out[e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

// A (ldA x ldA, symmetric) = the sum of the ranges' tiles in range order.
__global__ __launch_bounds__(256) void kgf_sum(const double* __restrict__ part, int ntile,
                                               int nsplit, int64_t ldA, double* __restrict__ A) {
  constexpr int EL = kGfTile * kGfTile;
  int ti, tj;
  tile_of((int)blockIdx.x, ti, tj);
  const int e = (int)blockIdx.y * 256 + threadIdx.x;
  const double* p = part + (int64_t)blockIdx.x * EL + e;
  const int64_t step = (int64_t)ntile * EL;
  double s = 0.0;
  int q = 0;
  for (; q + 7 < nsplit; q += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; q < nsplit; ++q) s += p[q * step];
  const int64_t r = kGfTile * ti + e / kGfTile, c = kGfTile * tj + e % kGfTile;
  A[r * ldA + c] = s;
  if (ti != tj) A[c * ldA + r] = s;
}

// Cholesky factor of G (RP x RP in LDS) in every thread's own registers, with
// the rule of wave_chol for inactive columns: no lane exchange and no LDS
// round trip, and the rows of the panel are substituted from registers.  R is
// packed by columns (R[l][c], l <= c, at c (c + 1) / 2 + l).
template <typename TA, int RP>
__device__ __forceinline__ void chol_regs(const double* G, int reff,
                                          double (&R)[RP * (RP + 1) / 2], double (&dinv)[RP]) {
  const double u = sizeof(TA) == 8 ? 0x1p-53 : 0x1p-24;
  const double tau = (double)RP * fmax(u * u, 0x1p-53);
#pragma unroll
  for (int c = 0; c < RP; ++c)
#pragma unroll
    for (int l = 0; l <= c; ++l) R[c * (c + 1) / 2 + l] = G[l * RP + c];
#pragma unroll
  for (int k = 0; k < RP; ++k) {
    const double piv = R[k * (k + 1) / 2 + k];
    const double g0 = G[k * RP + k];
    const bool act = k < reff && g0 > 0.0 && piv > tau * g0;
    const double inv = act ? rsqrt_nr(piv) : 0.0;
    dinv[k] = inv;
#pragma unroll
    for (int c = k; c < RP; ++c)
      R[c * (c + 1) / 2 + k] = act ? R[c * (c + 1) / 2 + k] * inv : 0.0;
#pragma unroll
    for (int c = k + 1; c < RP; ++c)
#pragma unroll
      for (int i = k + 1; i <= c; ++i)
        R[c * (c + 1) / 2 + i] =
            fma(-R[i * (i + 1) / 2 + k], R[c * (c + 1) / 2 + k], R[c * (c + 1) / 2 + i]);
  }
}

template <int RP>
__device__ __forceinline__ void row_rinv_regs(const double (&y)[RP],
                                              const double (&R)[RP * (RP + 1) / 2],
                                              const double (&dinv)[RP], double (&x)[RP]) {
#pragma unroll
  for (int c = 0; c < RP; ++c) {
    double s = y[c];
#pragma unroll
    for (int l = 0; l < c; ++l) s = fma(-x[l], R[c * (c + 1) / 2 + l], s);
    x[c] = s * dinv[c];
  }
}

struct GfPass {
  const double* A;       // ldA x ldA
  int64_t ldA;
  int n, np;             // columns, rounded up to 32
  const double* A1;      // start panel n x r (or null)
  int r;
  const void* warm;      // start panel of the type of X, RP columns (or null)
  const double* Y;       // else: the last product (np x RP) and the partials
  const double* G;       //   of its Gram (np / 16 of RP x RP)
  int second;            // a second Cholesky QR round; V_L and V_L^T are written
  SmallState* st;
  double* acc;           // R factors folded into (R2 or T)
  int reset, normalise;
  void* VL;
  void* VLt;
  int64_t ldv;           // row length of V_L^T
  double* Z;             // the orthonormal panel (np x RP), when wanted
  double* Yn;            // A Z (np x RP); null: no product
  double* Gn;            // partials: Y^T Y, or Z^T A Z with bt
  int bt;
};

// acc <- R acc (or R), a thread per entry; rescaled by a power of two when
// normalise is set.  R: RP x RP row-major in LDS, old: scratch of as much.
template <int RP>
__device__ void fold_r(const double* R, double* old, double* acc, int reset, int normalise,
                       double* red) {
  constexpr int E = RP * RP;
  const int tid = threadIdx.x;
  if (tid < E) old[tid] = reset ? 0.0 : acc[tid];
  __syncthreads();
  const int i = tid / RP, j = tid % RP;
  double s = 0.0;
  if (tid < E) {
    if (reset) {
      s = R[tid];
    } else {
      for (int l = i; l < RP; ++l) s = fma(R[i * RP + l], old[l * RP + j], s);
    }
  }
  if (normalise) {
    // only the ratios of R2's singular values matter
    double mx = tid < E ? fabs(s) : 0.0;
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    mx = red[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) mx = fmax(mx, red[w]);
    int e = 0;
    if (mx > 0.0 && isfinite(mx)) frexp(mx, &e);
    s *= ldexp(1.0, -e);
  }
  if (tid < E) acc[tid] = s;
  __syncthreads();
}

// One pass.  Block b < np / 16 owns rows [16 b, 16 b + 16) of the product; the
// panel is kept whole in LDS, a thread per row.  The A operand (16 rows x n,
// by symmetry a column slab: coalesced) is loaded first, so that it arrives
// while the panel is orthonormalised; the eight waves split the contraction.
// One more block folds the R factors into acc, off the others' way.
template <typename TA, int RP>
__global__ __launch_bounds__(512) void kgf_pass(GfPass a) {
  constexpr int E = RP * RP;
  // row groups of the second round's Gram: at most 32, so that no sum has a
  // chain of more than 32 (512 partials in a row, at RP = 1, left | |v| - 1 | at
  // 3e-16 where 1e-16 is reached)
  constexpr int NG = 512 / E < 32 ? 512 / E : 32;
  extern __shared__ double zs[];   // np x RP
  __shared__ double gs[E], rl[E];
  __shared__ double red[8][16][17];
  __shared__ double ys[16][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int np = a.np, nb = np / 16;
  const int slab = (int)blockIdx.x * 16;
  const bool fold = (int)blockIdx.x == nb;
  const int n = a.n;
  const bool product = a.Yn != nullptr && !fold;
  // ---- the A operand of this wave: k in [kw wave, kw (wave + 1)) ----
  const int kw = np / 8, nk = np / 32;
  const int kr = kw * wave + (lane >> 4);
  double av[kGfMaxK];
  if (product) {
    const double* p = a.A + slab + (lane & 15);
#pragma unroll
    for (int k = 0; k < kGfMaxK; ++k)
      if (k < nk) av[k] = p[(int64_t)(kr + 4 * k) * a.ldA];
  }
  const int reff = a.st->r_eff;
  double R[RP * (RP + 1) / 2], dinv[RP];
  // R of the last step (packed, in every thread) into acc
  auto fold_acc = [&](int reset) {
    for (int e = tid; e < E; e += 512) rl[e] = 0.0;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
      for (int c = 0; c < RP; ++c)
#pragma unroll
        for (int l = 0; l <= c; ++l) rl[l * RP + c] = R[c * (c + 1) / 2 + l];
    }
    __syncthreads();
    fold_r<RP>(rl, gs, a.acc, reset, a.normalise, &red[0][0][0]);
  };
  // ---- the panel ----
  double x[RP];   // row tid
  if (a.Y != nullptr) {
    double y[RP];
#pragma unroll
    for (int c = 0; c < RP; ++c) y[c] = tid < np ? a.Y[tid * RP + c] : 0.0;
    for (int e = tid; e < E; e += 512) {
      double v[kGfSlabs];
#pragma unroll
      for (int b = 0; b < kGfSlabs; ++b) v[b] = b < nb ? a.G[b * E + e] : 0.0;
      double s = 0.0;
#pragma unroll
      for (int b = 0; b < kGfSlabs; ++b) s += v[b];
      gs[e] = s;
    }
    __syncthreads();
    chol_regs<TA, RP>(gs, reff, R, dinv);
    row_rinv_regs<RP>(y, R, dinv, x);
    if (fold) {
      __syncthreads();
      fold_acc(a.reset);
    }
  } else {
#pragma unroll
    for (int c = 0; c < RP; ++c) {
      x[c] = 0.0;
      if (tid < n && c < a.r && c < reff)
        x[c] = a.warm != nullptr ? (double)((const TA*)a.warm)[tid * RP + c]
                                 : a.A1[tid * a.r + c];
    }
  }
  if (tid < np) {
#pragma unroll
    for (int c = 0; c < RP; ++c) zs[tid * RP + c] = x[c];
  }
  __syncthreads();
  if (a.second) {
    double* gp = &red[0][0][0];   // NG * E <= 512 partials
    const int e = tid % E, h = tid / E;
    if (h < NG) {
      const int ra = e / RP, rb = e % RP;
      double s = 0.0;
      for (int j = h; j < n; j += NG) s = fma(zs[j * RP + ra], zs[j * RP + rb], s);
      gp[h * E + e] = s;
    }
    __syncthreads();
    if (tid < E) {
      double s = 0.0;
      for (int q = 0; q < NG; ++q) s += gp[q * E + tid];
      gs[tid] = s;
    }
    __syncthreads();
    chol_regs<TA, RP>(gs, reff, R, dinv);
    if (fold) {
      __syncthreads();
      fold_acc(0);
      return;
    }
    double y[RP];
#pragma unroll
    for (int c = 0; c < RP; ++c) y[c] = x[c];
    row_rinv_regs<RP>(y, R, dinv, x);
    if (tid < np) {
#pragma unroll
      for (int c = 0; c < RP; ++c) zs[tid * RP + c] = x[c];
    }
    if (tid >= slab && tid < slab + 16 && tid < n) {
#pragma unroll
      for (int c = 0; c < RP; ++c) {
        ((TA*)a.VL)[tid * RP + c] = (TA)x[c];
        ((TA*)a.VLt)[c * a.ldv + tid] = (TA)x[c];
      }
    }
    __syncthreads();
  }
  if (fold) return;
  const int oi = tid >> 4, oc = tid & 15;   // this thread's entry of the 16 x 16 block
  if (a.Z != nullptr && oi < 16 && oc < RP)
    a.Z[(slab + oi) * RP + oc] = zs[(slab + oi) * RP + oc];
  if (!product) return;
  // ---- Y = A Z over the block's rows ----
  f64x4 c4 = {0.0, 0.0, 0.0, 0.0};
  const int cj = lane & 15;
#pragma unroll
  for (int k = 0; k < kGfMaxK; ++k) {
    if (k < nk) {
      const double b = cj < RP ? zs[(kr + 4 * k) * RP + cj] : 0.0;
      c4 = mfma64(av[k], b, c4);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][4 * v + (lane >> 4)][cj] = c4[v];
  __syncthreads();
  if (oi < 16) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += red[w][oi][oc];
    ys[oi][oc] = s;
    if (oc < RP) a.Yn[(slab + oi) * RP + oc] = s;
  }
  __syncthreads();
  for (int e = tid; e < E; e += 512) {
    const int ra = e / RP, rb = e % RP;
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      s = fma(a.bt ? zs[(slab + i) * RP + ra] : ys[i][ra], ys[i][rb], s);
    a.Gn[(int64_t)blockIdx.x * E + e] = s;
  }
}

// P = Zq K' for U_L = D P, row j of it (K' in LDS; null: P = Zq).
template <int RP>
__device__ __forceinline__ void p_row(const double* __restrict__ Zq, const double* ks, int j,
                                      double (&p)[RP]) {
  double z[RP];
#pragma unroll
  for (int c = 0; c < RP; ++c) z[c] = Zq[j * RP + c];
#pragma unroll
  for (int c = 0; c < RP; ++c) {
    p[c] = z[c];
    if (ks != nullptr) {
      p[c] = 0.0;
#pragma unroll
      for (int l = 0; l < RP; ++l) p[c] = fma(z[l], ks[l * RP + c], p[c]);
    }
  }
}

// U_L = D P, P rounded to the type of X.  FP32: 64 rows per block, a wave
// takes 16 rows over all n columns with v_mfma_f32_16x16x4f32 (a lane reads
// four consecutive columns and feeds them to four products, the same order on
// both operands), P^T in LDS.  Every load of D is issued first.
template <int RP>
__global__ __launch_bounds__(256) void kgf_ul_f32(const float* __restrict__ D, int64_t ldd,
                                                  int64_t m, int np,
                                                  const double* __restrict__ Zq,
                                                  const double* __restrict__ K,
                                                  float* __restrict__ UL) {
  constexpr int LP = kGfMaxN + 4;
  __shared__ __align__(16) float pt[RP * LP];
  __shared__ double ks[RP * RP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * 64 + 16 * wave;
  const int nt = np / 16;
  const float* pd = D + (row0 + i) * ldd + 4 * g;   // D has whole 64-row groups
  float4 d[2 * kGfMaxK];
#pragma unroll
  for (int t = 0; t < 2 * kGfMaxK; ++t)
    if (t < nt) d[t] = *reinterpret_cast<const float4*>(pd + 16 * t);
  if (K != nullptr && tid < RP * RP) ks[tid] = K[tid];
  __syncthreads();
  for (int j = tid; j < np; j += 256) {
    double p[RP];
    p_row<RP>(Zq, K != nullptr ? ks : nullptr, j, p);
#pragma unroll
    for (int c = 0; c < RP; ++c) pt[c * LP + j] = (float)p[c];
  }
  __syncthreads();
  f32x4g acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f32x4g{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2 * kGfMaxK; ++t) {
    if (t < nt) {
      float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < RP) b = *reinterpret_cast<const float4*>(&pt[i * LP + 16 * t + 4 * g]);
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t].x, b.x, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t].y, b.y, acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t].z, b.z, acc[2], 0, 0, 0);
      acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t].w, b.w, acc[3], 0, 0, 0);
    }
  }
  const f32x4g s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  if (i < RP) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = row0 + 4 * g + v;
      if (row < m) UL[row * RP + i] = s[v];
    }
  }
}

// FP64: 16 rows per block, the eight waves split the contraction.
template <int RP>
__global__ __launch_bounds__(512) void kgf_ul_f64(const double* __restrict__ D, int64_t ldd,
                                                  int64_t m, int np,
                                                  const double* __restrict__ Zq,
                                                  const double* __restrict__ K,
                                                  double* __restrict__ UL) {
  extern __shared__ double ps[];   // np x RP
  __shared__ double red[8][16][17];
  __shared__ double ks[RP * RP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * 16;
  const int nk = np / 32;
  const int kr = (np / 8) * wave + (lane >> 4);
  const double* pd = D + (row0 + (lane & 15)) * ldd + kr;
  double d[kGfMaxK];
#pragma unroll
  for (int k = 0; k < kGfMaxK; ++k)
    if (k < nk) d[k] = pd[4 * k];
  if (K != nullptr && tid < RP * RP) ks[tid] = K[tid];
  __syncthreads();
  if (tid < np) {
    double p[RP];
    p_row<RP>(Zq, K != nullptr ? ks : nullptr, tid, p);
#pragma unroll
    for (int c = 0; c < RP; ++c) ps[tid * RP + c] = p[c];
  }
  __syncthreads();
  f64x4 c4 = {0.0, 0.0, 0.0, 0.0};
  const int cj = lane & 15;
#pragma unroll
  for (int k = 0; k < kGfMaxK; ++k)
    if (k < nk) c4 = mfma64(d[k], cj < RP ? ps[(kr + 4 * k) * RP + cj] : 0.0, c4);
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][4 * v + (lane >> 4)][cj] = c4[v];
  __syncthreads();
  const int oi = tid >> 4, oc = tid & 15;
  if (oi < 16 && oc < RP && row0 + oi < m) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += red[w][oi][oc];
    UL[(row0 + oi) * RP + oc] = s;
  }
}

#define GF_RP_SWITCH(rp, ...)                                \
  switch (rp) {                                              \
    case 1: { constexpr int RP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int RP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int RP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int RP = 8; __VA_ARGS__; } break;   \
    case 12: { constexpr int RP = 12; __VA_ARGS__; } break; \
    case 16: { constexpr int RP = 16; __VA_ARGS__; } break; \
    default: break;                                          \
  }

void pass(const Launch& L, bool f64, int rp, const GfPass& a) {
  // the first pass folds nothing
  const unsigned nb = (unsigned)(a.np / 16) + (a.Y != nullptr ? 1u : 0u);
  GF_RP_SWITCH(rp, {
    const size_t lds = sizeof(double) * a.np * RP;
    if (f64)
      hipLaunchKernelGGL((kgf_pass<double, RP>), dim3(nb), dim3(512), lds, L.stream, a);
    else
      hipLaunchKernelGGL((kgf_pass<float, RP>), dim3(nb), dim3(512), lds, L.stream, a);
  });
}

}  // namespace

void launch_gram_form(const Launch& L, const GramForm& g) {
  // A = D^T D
  const int nt = (int)(g.ldA / kGfTile);
  const int ntile = nt * (nt + 1) / 2;
  const dim3 gg((unsigned)ntile, (unsigned)g.nsplit);
  if (g.f64)
    hipExtLaunchKernelGGL(kgf_gram<double>, gg, dim3(256), 0, L.stream, g.ev_gram[0],
                          g.ev_gram[1], 0, (const double*)g.D, g.ldd, g.mpad, g.rows_per, g.part);
  else
    hipExtLaunchKernelGGL(kgf_gram<float>, gg, dim3(256), 0, L.stream, g.ev_gram[0],
                          g.ev_gram[1], 0, (const float*)g.D, g.ldd, g.mpad, g.rows_per, g.part);
  hipLaunchKernelGGL(kgf_sum, dim3((unsigned)ntile, kGfTile * kGfTile / 256), dim3(256), 0,
                     L.stream, (const double*)g.part, ntile, g.nsplit, g.ldA, g.A);
  GfPass a{};
  a.A = g.A; a.ldA = g.ldA;
  a.n = (int)g.n; a.np = (int)((g.n + 31) / 32 * 32);
  a.st = g.st;
  a.VL = g.VL; a.VLt = g.VLt; a.ldv = g.ldv;
  int cur = 0;
  // subspace chain: p products, each orthonormalised by the next pass; R2
  a.A1 = g.A1; a.r = g.r; a.warm = g.warm;
  a.Yn = g.Y[0]; a.Gn = g.G[0];
  pass(L, g.f64, g.rp, a);
  a.acc = g.st->R2; a.normalise = 1;
  a.reset = 1;
  for (int j = 1; j < g.p; ++j) {
    a.Y = g.Y[cur]; a.G = g.G[cur];
    cur ^= 1;
    a.Yn = g.Y[cur]; a.Gn = g.G[cur];
    pass(L, g.f64, g.rp, a);
    a.reset = 0;
  }
  // Q2 by a second round; then the B chain's q products (their R factors
  // into T) and the product whose Gram with Y_q is B'^T B'
  a.second = 1;
  const int more = g.proj ? 0 : g.q + 1;
  for (int j = 0; j < (more > 0 ? more : 1); ++j) {
    a.Y = g.Y[cur]; a.G = g.G[cur];
    cur ^= 1;
    const bool last = j + 1 >= more;
    a.Yn = g.proj ? nullptr : g.Y[cur];
    a.Gn = g.G[cur];
    a.bt = last ? 1 : 0;
    a.Z = last ? g.Zq : nullptr;
    pass(L, g.f64, g.rp, a);
    a.second = 0;
    a.acc = g.st->T; a.normalise = 0;
    a.reset = j == 0 ? 1 : 0;
  }
  if (!g.proj)
    launch_core(L, g.f64, g.rp, g.G[cur], a.np / 16, 0, g.st, g.p, g.rank_tol, g.q == 0 ? 1 : 0, g.Kp);
  const double* K = g.proj ? nullptr : g.st->K;
  GF_RP_SWITCH(g.rp, {
    if (g.f64)
      hipExtLaunchKernelGGL((kgf_ul_f64<RP>), dim3((unsigned)((g.m + 15) / 16)), dim3(512),
                            sizeof(double) * a.np * RP, L.stream, g.ev_ul[0], g.ev_ul[1], 0,
                            (const double*)g.D, g.ldd, g.m, a.np, (const double*)g.Zq, K,
                            (double*)g.UL);
    else
      hipExtLaunchKernelGGL((kgf_ul_f32<RP>), dim3((unsigned)((g.m + 63) / 64)), dim3(256), 0,
                            L.stream, g.ev_ul[0], g.ev_ul[1], 0, (const float*)g.D, g.ldd, g.m,
                            a.np, (const double*)g.Zq, K, (float*)g.UL);
  });
}

}  // namespace godec
