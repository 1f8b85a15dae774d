// FP32 residual tiles on the matrix cores, shared by the selection and the
// fixed-support pass.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace godec {

// ---------------------------------------------------------------------------
// FP32 residual tiles: L = U_L V_L^T over rows [r0, r0 + 16) and columns
// [c0, c0 + 16) (r0, c0 multiples of 16) by one wavefront with
// v_mfma_f32_16x16x4f32 evaluating the transposed tile V_L U_L^T, k-steps of
// four rank columns in ascending order.  Lane l supplies
// V_L[c0 + l%16][4s + l/16] (A operand) and U_L[r0 + l%16][4s + l/16]
// (B operand), zero past m, n or RP, and receives L at row r0 + l%16 and
// columns c0 + res_col(v, l), v < 4: four consecutive columns of one row, so
// that a lane reads its four X entries with one 16-byte load.
// ---------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int RP>
struct ResK { static constexpr int KS = (RP + 3) / 4; };

__device__ __forceinline__ int res_col(int v, int lane) { return 4 * (lane >> 4) + v; }

// The loaders read a clamped in-bounds address on every lane and zero the
// padding afterwards, so no load sits behind a lane-dependent branch (m, n
// and RP are at least 1).
template <int RP>
__device__ __forceinline__ void res_load_u(const float* __restrict__ UL, int64_t m, int64_t r0,
                                           int lane, float (&a)[ResK<RP>::KS]) {
  const int64_t row = r0 + (lane & 15);
  const int64_t rowc = row < m ? row : m - 1;
  const int g = lane >> 4;
#pragma unroll
  for (int s = 0; s < ResK<RP>::KS; ++s) {
    const int k = 4 * s + g;
    const int kc = k < RP ? k : RP - 1;
    const float u = UL[rowc * RP + kc];
    a[s] = (k < RP && row < m) ? u : 0.f;
  }
}

// V operand from V_L^T (RP x ldv).
template <int RP>
__device__ __forceinline__ void res_load_vt(const float* __restrict__ VLt, int64_t ldv,
                                            int64_t n, int64_t c0, int lane,
                                            float (&b)[ResK<RP>::KS]) {
  const int64_t col = c0 + (lane & 15);
  const int64_t colc = col < n ? col : n - 1;
  const int g = lane >> 4;
#pragma unroll
  for (int s = 0; s < ResK<RP>::KS; ++s) {
    const int k = 4 * s + g;
    const int kc = k < RP ? k : RP - 1;
    const float v = VLt[kc * ldv + colc];
    b[s] = (k < RP && col < n) ? v : 0.f;
  }
}

// V operand from V_L (n x RP, row-major): the same values.
template <int RP>
__device__ __forceinline__ void res_load_v(const float* __restrict__ VL, int64_t n, int64_t c0,
                                           int lane, float (&b)[ResK<RP>::KS]) {
  const int64_t col = c0 + (lane & 15);
  const int64_t colc = col < n ? col : n - 1;
  const int g = lane >> 4;
#pragma unroll
  for (int s = 0; s < ResK<RP>::KS; ++s) {
    const int k = 4 * s + g;
    const int kc = k < RP ? k : RP - 1;
    const float v = VL[colc * RP + kc];
    b[s] = (k < RP && col < n) ? v : 0.f;
  }
}

// u: the U_L operand (res_load_u), v: the V_L operand (res_load_vt or
// res_load_v).
template <int RP>
__device__ __forceinline__ f32x4_t res_tile(const float (&u)[ResK<RP>::KS],
                                            const float (&v)[ResK<RP>::KS]) {
  f32x4_t acc = {};
#pragma unroll
  for (int s = 0; s < ResK<RP>::KS; ++s)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[s], u[s], acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ float res_pick(const f32x4_t& L, int v) {
  float out = L[0];
  out = (v == 1) ? L[1] : out;
  out = (v == 2) ? L[2] : out;
  out = (v == 3) ? L[3] : out;
  return out;
}

}  // namespace godec
