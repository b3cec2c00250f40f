// Device helpers shared by the implicit-GEMM kernels.
#pragma once

#include "internal.h"

namespace hapi {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int xcd_remap(int bid, int nb) {
  // Workgroups are dispatched round-robin over the 8 XCDs (block b -> XCD b % 8).
  // Renumber so that consecutive logical tiles run on one XCD and share its L2.
  const int xcd = bid & 7, idx = bid >> 3;
  const int q = nb >> 3, r = nb & 7;
  return (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }

// erf by Abramowitz & Stegun, Handbook of Mathematical Functions, 7.1.26:
// erf(x) = 1 - t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-x^2), t = 1 / (1 + p x)
// for x >= 0 (odd extension), absolute error <= 1.5e-7: branch-free, one
// reciprocal and one exponential, against a piecewise library erf.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float q = fmaf(t, 1.061405429f, -1.453152027f);
  q = fmaf(t, q, 1.421413741f);
  q = fmaf(t, q, -0.284496736f);
  q = fmaf(t, q, 0.254829592f);
  const float y = fmaf(-t * q, __builtin_amdgcn_exp2f(-ax * ax * 1.4426950408889634f), 1.0f);
  return copysignf(y, x);
}

// GELU is the exact (erf) form: v * Phi(v) = 0.5 v (1 + erf(v / sqrt 2)).
__device__ __forceinline__ float epilogue_act(float v, int relu, int gelu) {
  if (relu) v = fmaxf(v, 0.0f);
  if (gelu) v = 0.5f * v * (1.0f + erf_as(v * 0.70710678118654752f));
  return v;
}

// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

constexpr unsigned kOob = 0x80000000u;  // a byte offset outside every buffer range

// Per-row state of the rows a thread gathers for the A tile.
struct RowState {
  int base;  // element offset of the row's image (NHWC / NCHW) or of the row (GEMM)
  int hi0;   // ho * stride - pad  (large negative: row beyond M)
  int wi0;   // wo * stride - pad
};

template <int LD>
__device__ __forceinline__ RowState make_row(const ConvArgs &a, int m) {
  RowState r;
  if (m >= a.M) {
    r.base = 0; r.hi0 = -(1 << 28); r.wi0 = 0;
    return r;
  }
  if (LD == LD_GEMM) {
    r.base = m * (a.lda ? a.lda : a.K); r.hi0 = 0; r.wi0 = 0;
    return r;
  }
  const int hw = a.Ho * a.Wo;
  const int n = m / hw, rem = m - n * hw;
  const int ho = rem / a.Wo, wo = rem - ho * a.Wo;
  r.base = n * a.H * a.W * a.C;
  r.hi0 = ho * a.stride - a.pad;
  r.wi0 = wo * a.stride - a.pad;
  return r;
}

}  // namespace
}  // namespace hapi
