// GoDec matrix completion (Sec. 2): the S update on a fixed support set in
// place of the cardinality constraint, S_t = P_support(X - L_t).  The L
// update and the D update are those of Algorithm 1; these kernels replace
// the radix selection.
#include <hip/hip_runtime.h>

#include "godec_internal.h"
#include "k_common.h"
#include "k_restile.h"

namespace godec {

namespace {

constexpr int kNormBlocks = 2048;   // most blocks (= partial sums) of the pass
constexpr int kTileStride = 68;     // LDS row stride of a 64-column piece: rows 16-byte aligned

template <typename T>
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// *bad = 1 unless the list is strictly ascending within [0, mn).
__global__ __launch_bounds__(256) void kc_check(const int64_t* __restrict__ support,
                                                int64_t nnz, int64_t mn, int* bad) {
  int wrong = 0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * 256) {
    const int64_t id = support[e];
    if (id < 0 || id >= mn || (e > 0 && id <= support[e - 1])) wrong = 1;
  }
  if (wrong) atomicOr(bad, 1);
}

// The list as the pass reads it: for every row i and 64-column word w of it
// the word's membership bits and the list position of its first entry.  One
// thread per word: a lower bound in the ascending list, then the run itself, at
// most 64 entries.  Any list keeps the reads in bounds and the runs short (one
// of equal entries too); what an invalid one leaves here is not used.
__global__ __launch_bounds__(256) void kc_runs(const int64_t* __restrict__ support, int64_t nnz,
                                               int64_t m, int64_t n, int64_t nw,
                                               SupportWord* __restrict__ words) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= m * nw) return;
  const int64_t i = s / nw, w = s % nw;
  const int64_t key = i * n + w * 64;
  const int64_t end = (w + 1) * 64 < n ? key + 64 : (i + 1) * n;
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (support[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  SupportWord o;
  o.start = lo;
  o.bits = 0ull;
  const int64_t last = lo + 64 < nnz ? lo + 64 : nnz;
  for (int64_t e = lo; e < last; ++e) {
    const int64_t id = support[e];
    if (id < key || id >= end) break;
    o.bits |= 1ull << (id - key);
  }
  words[s] = o;
}

// One pass over X for the whole fixed-support step.  Work unit: 16 rows of a
// 256-column block (a wave takes one 64-column word of it), in column-block-
// major order, and block b takes the units [W b / G, W (b + 1) / G) of the W
// units.  A row's membership bits and the start of its run come with one
// 16-byte load, so an entry's place in the list is start + (set bits before
// it): no list read, no LDS and no barrier in the loop.  r = X - (U_L V_L^T)
// goes to s_val (X to s_x, where asked for), and the working copies of D get
// X - S on the words that hold support entries, as whole words (off the
// support D is X already, but full lines are written without a read).
// pall / psel: the block's sums of r^2 off / on the support.
// Bound: HBM: X in, D out, the words and S beside them: 0.87 GB at
// 10000 x 10000, r = 20, 1e7 entries, 246 us (3.5 TB/s; 179 us without the D
// store, 217 without the list).  The list-driven form of this pass (tiles
// staged in LDS, entries looked up per row) and the scattered D update after
// it took 343 + 149 us.
//
// FP32: L in the residual tiles of the selection (the V_L operand of the
// wave's four tiles stays in registers for the column block), handed through
// LDS from the tile layout to a lane per column, so that a row's membership
// bits are one scalar mask and its D segment and its list entries are each
// one coalesced store.
// One 16-row x 64-column piece.  FULL: all of it lies inside the matrix.
// MIXED: the bf16 copy and X at the entries are written (and D if given);
// otherwise D alone.
template <int RP, bool FULL, bool MIXED>
__device__ __forceinline__ void kc_piece(const float* __restrict__ xp, int64_t ldx, int nr,
                                         bool live, const float (&a)[ResK<RP>::KS],
                                         const float (&b)[4][ResK<RP>::KS], float* lt, int lane,
                                         const SupportWord* __restrict__ wr, int64_t nw,
                                         float* __restrict__ s_val, float* __restrict__ s_x,
                                         float* __restrict__ drow, uint16_t* __restrict__ drow16,
                                         int64_t ldd, double& acc, double& accs) {
  constexpr int LW = kTileStride;
  float x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = xp[(FULL || i < nr ? i : nr - 1) * ldx];
  // lane l: the word of row l % 16 (broadcast to the wave by readlane below)
  const int li = lane & 15;
  const SupportWord sw = wr[(FULL || li < nr ? li : nr - 1) * nw];
  __builtin_amdgcn_wave_barrier();   // the last piece's reads of the tile are done
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const f32x4_t L = res_tile<RP>(a, b[t]);
    *reinterpret_cast<f32x4_t*>(&lt[li * LW + 16 * t + res_col(0, lane)]) = L;
  }
  __builtin_amdgcn_wave_barrier();
  const int blo = (int)(sw.bits & 0xffffffffull), bhi = (int)(sw.bits >> 32);
  const int slo = (int)(sw.start & 0xffffffffll), shi = (int)(sw.start >> 32);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (FULL || i < nr) {   // uniform
      const unsigned int mlo = (unsigned int)__builtin_amdgcn_readlane(blo, i);
      const unsigned int mhi = (unsigned int)__builtin_amdgcn_readlane(bhi, i);
      const int64_t s0 = ((int64_t)__builtin_amdgcn_readlane(shi, i) << 32) |
                         (unsigned int)__builtin_amdgcn_readlane(slo, i);
      const unsigned long long bits = ((unsigned long long)mhi << 32) | mlo;
      const float r = x[i] - lt[i * LW + lane];
      const bool on = (bits >> lane) & 1ull;
      const double off = on || !(FULL || live) ? 0.0 : (double)r;
      acc = fma(off, off, acc);
      const float d = on ? x[i] - r : x[i];
      if (on) {
        const unsigned int q = __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
        (s_val + s0)[q] = r;
        if (MIXED) (s_x + s0)[q] = x[i];
        accs = fma((double)r, (double)r, accs);
      }
      if (bits != 0ull && (FULL || live)) {
        if (MIXED) drow16[lane] = f32_to_bf16(d);
        if (!MIXED || drow != nullptr) drow[lane] = d;
      }
    }
    if (MIXED) drow16 += ldd;
    if (!MIXED || drow != nullptr) drow += ldd;
  }
}

template <int RP, bool MIXED>
__global__ __launch_bounds__(256) void kc_pass_f32(
    const float* __restrict__ X, int64_t ldx, const float* __restrict__ UL,
    const float* __restrict__ VLt, int64_t ldv, int64_t m, int64_t n, int64_t nw,
    const SupportWord* __restrict__ words, float* __restrict__ s_val, float* __restrict__ s_x,
    float* __restrict__ D, uint16_t* __restrict__ D16, int64_t ldd, double* __restrict__ pall,
    double* __restrict__ psel) {
  constexpr int KS = ResK<RP>::KS;
  __shared__ __align__(16) float tile[4][16 * kTileStride];
  __shared__ double red[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nrb = (m + 15) / 16;
  const int64_t units = nrb * ((n + 255) / 256);
  const int64_t u0 = units * blockIdx.x / gridDim.x;
  const int64_t u1 = units * (blockIdx.x + 1) / gridDim.x;
  double acc = 0.0, accs = 0.0;   // sums of r^2 off and on the support
  float b[4][KS];
  int64_t cb = u0 / nrb, rb = u0 - cb * nrb;
  bool load_v = true;
  for (int64_t u = u0; u < u1; ++u, ++rb) {
    if (rb == nrb) {
      rb = 0;
      ++cb;
      load_v = true;
    }
    const int64_t r0 = rb * 16;
    const int64_t w = cb * 4 + wave;
    if (w >= nw) continue;   // wave-uniform
    const int64_t cw = w * 64;
    if (load_v) {
#pragma unroll
      for (int t = 0; t < 4; ++t) res_load_vt<RP>(VLt, ldv, n, cw + 16 * t, lane, b[t]);
      load_v = false;
    }
    float a[KS];
    res_load_u<RP>(UL, m, r0, lane, a);
    const int nr = (m - r0) < 16 ? (int)(m - r0) : 16;
    const bool live = cw + lane < n;
    const float* xp = X + r0 * ldx + (live ? cw + lane : n - 1);
    const SupportWord* wr = words + r0 * nw + w;
    float* drow = D ? D + r0 * ldd + cw : nullptr;
    uint16_t* drow16 = MIXED ? D16 + r0 * ldd + cw : nullptr;
    if (nr == 16 && cw + 64 <= n)
      kc_piece<RP, true, MIXED>(xp, ldx, nr, live, a, b, tile[wave], lane, wr, nw, s_val, s_x,
                                drow, drow16, ldd, acc, accs);
    else
      kc_piece<RP, false, MIXED>(xp, ldx, nr, live, a, b, tile[wave], lane, wr, nw, s_val, s_x,
                                 drow, drow16, ldd, acc, accs);
  }
  double tot = block_sum<float>(acc, red);
  if (threadIdx.x == 0) pall[blockIdx.x] = tot;
  __syncthreads();
  tot = block_sum<float>(accs, red);
  if (threadIdx.x == 0) psel[blockIdx.x] = tot;
}

// FP64: a thread owns a column and keeps its row of V_L in registers for the
// column block; a row's word is the same for the whole wave.
template <int RP>
__global__ __launch_bounds__(256) void kc_pass_f64(
    const double* __restrict__ X, int64_t ldx, const double* __restrict__ UL,
    const double* __restrict__ VLt, int64_t ldv, int64_t m, int64_t n, int64_t nw,
    const SupportWord* __restrict__ words, double* __restrict__ s_val, double* __restrict__ s_x,
    double* __restrict__ D, int64_t ldd, double* __restrict__ pall, double* __restrict__ psel) {
  constexpr int G = 4;   // rows whose X loads are in flight together
  __shared__ double red[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nrb = (m + 15) / 16;
  const int64_t units = nrb * ((n + 255) / 256);
  const int64_t u0 = units * blockIdx.x / gridDim.x;
  const int64_t u1 = units * (blockIdx.x + 1) / gridDim.x;
  double acc = 0.0, accs = 0.0;
  double v[RP];
  int64_t have = -1;
  for (int64_t u = u0; u < u1; ++u) {
    const int64_t cb = u / nrb;
    const int64_t i0 = (u - cb * nrb) * 16;
    const int64_t w = cb * 4 + wave;
    if (w >= nw) continue;   // wave-uniform
    const int64_t j = cb * 256 + threadIdx.x;
    const bool live = j < n;
    if (cb != have) {
#pragma unroll
      for (int c = 0; c < RP; ++c) v[c] = live ? VLt[c * ldv + j] : 0.0;
      have = cb;
    }
    const int64_t i1 = (i0 + 16) < m ? (i0 + 16) : m;
    for (int64_t c0 = i0; c0 < i1; c0 += G) {
      double x[G];
#pragma unroll
      for (int g = 0; g < G; ++g) x[g] = (live && c0 + g < i1) ? X[(c0 + g) * ldx + j] : 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int64_t i = c0 + g;
        if (i >= i1) break;   // uniform
        const SupportWord sw = words[i * nw + w];
        const double* ui = UL + i * RP;
        double l = 0.0;
#pragma unroll
        for (int c = 0; c < RP; ++c) l = fma(ui[c], v[c], l);
        const double r = x[g] - l;
        const bool on = (sw.bits >> lane) & 1ull;
        if (on) {
          const int64_t ent = sw.start + __popcll(sw.bits & ((1ull << lane) - 1ull));
          s_val[ent] = r;
          if (s_x) s_x[ent] = x[g];
          accs = fma(r, r, accs);
        } else if (live) {
          acc = fma(r, r, acc);
        }
        if (D != nullptr && sw.bits != 0ull && live) D[i * ldd + j] = on ? x[g] - r : x[g];
      }
    }
  }
  double tot = block_sum<double>(acc, red);
  if (threadIdx.x == 0) pall[blockIdx.x] = tot;
  __syncthreads();
  tot = block_sum<double>(accs, red);
  if (threadIdx.x == 0) psel[blockIdx.x] = tot;
}

// The plan of a fixed-support step: nnz, sum_sel2 = sum of the support
// partials, sum_obs2 = sum of the off-support partials (np of each), sum_r2 =
// both (strided per thread, then a tree in LDS: a fixed order).
__global__ __launch_bounds__(256) void kc_finish(const double* __restrict__ psel,
                                                 const double* __restrict__ pall, int np,
                                                 int64_t nnz, SelPlan* __restrict__ plan) {
  __shared__ double ra[256], rb[256];
  // every partial in flight at once
  constexpr int PER = kNormBlocks / 256;
  double va[PER], vb[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = threadIdx.x + 256 * u;
    va[u] = q < np ? psel[q] : 0.0;
    vb[u] = q < np ? pall[q] : 0.0;
  }
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u) { a += va[u]; b += vb[u]; }
  ra[threadIdx.x] = a;
  rb[threadIdx.x] = b;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      ra[threadIdx.x] += ra[threadIdx.x + h];
      rb[threadIdx.x] += rb[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  plan->nnz = nnz;
  plan->sum_sel2 = ra[0];
  plan->sum_obs2 = rb[0];
  plan->sum_r2 = rb[0] + ra[0];
  plan->threshold = 0.0;
  plan->slow = 0;
  plan->overflow = 0;
  plan->mode = SEL_DONE;
}


}  // namespace

#define GC_RP_SWITCH(rp, ...)                                \
  switch (rp) {                                              \
    case 1: { constexpr int RP = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int RP = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int RP = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int RP = 8; __VA_ARGS__; } break;   \
    case 12: { constexpr int RP = 12; __VA_ARGS__; } break; \
    case 16: { constexpr int RP = 16; __VA_ARGS__; } break; \
    case 20: { constexpr int RP = 20; __VA_ARGS__; } break; \
    case 24: { constexpr int RP = 24; __VA_ARGS__; } break; \
    case 32: { constexpr int RP = 32; __VA_ARGS__; } break; \
    default: break;                                          \
  }

void launch_support_runs(const Launch& L, const int64_t* support, int64_t nnz, int64_t m,
                         int64_t n, SupportWord* words, int* bad) {
  const int64_t nw = (n + 63) / 64;
  const int64_t g = (nnz + 255) / 256, lim = 16LL * L.num_cu;
  if (nnz > 0)
    hipLaunchKernelGGL(kc_check, dim3((unsigned)(g < lim ? g : lim)), dim3(256), 0, L.stream,
                       support, nnz, m * n, bad);
  hipLaunchKernelGGL(kc_runs, dim3((unsigned)((m * nw + 255) / 256)), dim3(256), 0, L.stream,
                     support, nnz, m, n, nw, words);
}

void launch_fixed_support(const Launch& L, bool f64, int rp, const void* X, int64_t ldx,
                          const void* UL, const void* VLt, int64_t ldv, int64_t m, int64_t n,
                          const SupportWord* words, int64_t nnz,
                          void* s_val, void* s_x, void* D, uint16_t* D16, int64_t ldd,
                          SelPlan* plan, double* scratch) {
  const int64_t nw = (n + 63) / 64;
  const int64_t units = (m + 15) / 16 * ((n + 255) / 256);
  // eight blocks per CU, and units enough for each
  const int64_t lim = L.num_cu * 8LL < kNormBlocks ? L.num_cu * 8LL : kNormBlocks;
  const unsigned ga = (unsigned)(units < lim ? units : lim);
  double* psel = scratch;
  double* pall = scratch + kNormBlocks;
  GC_RP_SWITCH(rp, {
    if (f64)
      hipLaunchKernelGGL((kc_pass_f64<RP>), dim3(ga), dim3(256), 0, L.stream, (const double*)X,
                         ldx, (const double*)UL, (const double*)VLt, ldv, m, n, nw, words,
                         (double*)s_val, (double*)s_x, (double*)D, ldd, pall, psel);
    else if (D16 != nullptr)
      hipLaunchKernelGGL((kc_pass_f32<RP, true>), dim3(ga), dim3(256), 0, L.stream,
                         (const float*)X, ldx, (const float*)UL, (const float*)VLt, ldv, m, n,
                         nw, words, (float*)s_val, (float*)s_x, (float*)D, D16, ldd, pall, psel);
    else
      hipLaunchKernelGGL((kc_pass_f32<RP, false>), dim3(ga), dim3(256), 0, L.stream,
                         (const float*)X, ldx, (const float*)UL, (const float*)VLt, ldv, m, n,
                         nw, words, (float*)s_val, (float*)nullptr, (float*)D,
                         (uint16_t*)nullptr, ldd, pall, psel);
  });
  hipLaunchKernelGGL(kc_finish, dim3(1), dim3(256), 0, L.stream, psel, pall, (int)ga, nnz, plan);
}

int64_t fixed_support_scratch_doubles() { return 2 * (int64_t)kNormBlocks; }

}  // namespace godec
