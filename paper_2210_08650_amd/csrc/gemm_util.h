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

// GELU in its exact (erf) form, v Phi(v) = max(v, 0) - |v| Phi(-|v|).  log2 Phi(-a)
// is nearly quadratic: a polynomial of degree 8, fitted to it on [0, 6.5] for the
// least maximum error of a Phi(-a) (weighted least squares, reweighted to the
// minimax), and one exp2.  Past 6.5 the polynomial falls monotonically
// (-35 at 6.5, -3160 at 16) and to -inf where it overflows.  Clamping v from above
// keeps +inf from meeting exp2(-inf) = 0; -inf does, and gives NaN as
// 0.5 v (1 + erf(v / sqrt 2)) does; NaN goes through the polynomial.
// Largest error against float64 over [-40, 40] 2.5e-7 (for v < 0 5.0e-8), rms 3.5e-8;
// erf by Abramowitz & Stegun 7.1.26 with its reciprocal: 4.7e-7 (2.6e-7), 7.1e-8, and
// smaller on no part of the range (in [-4, -3] 9e-4 against 2.3e-5 relative).
// 11 full-rate instructions and an exp2 for 15 and two transcendental ones: ViT-B/16
// b128 3,835 -> 3,759 us, one block at 48 images 242 -> 237 us.
__device__ __forceinline__ float gelu_erf(float v) {
  const float a = fabsf(v);
  float p = fmaf(a, -1.9919600617868127e-06f, 2.9272845495142974e-05f);
  p = fmaf(a, p, -1.3809293159283698e-04f);
  p = fmaf(a, p, -2.5342297158204019e-04f);
  p = fmaf(a, p, 7.2163678705692291e-03f);
  p = fmaf(a, p, -5.2603028714656830e-02f);
  p = fmaf(a, p, -4.5917221903800964e-01f);
  p = fmaf(a, p, -1.1511096954345703e+00f);
  p = fmaf(a, p, -9.9999988079071045e-01f);
  return fmaf(-fabsf(fminf(v, 16.0f)), __builtin_amdgcn_exp2f(p), fmaxf(v, 0.0f));
}

__device__ __forceinline__ float epilogue_act(float v, int relu, int gelu) {
  if (relu) v = fmaxf(v, 0.0f);
  if (gelu) v = gelu_erf(v);
  return v;
}

// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

constexpr unsigned kOob = 0x80000000u;  // a byte offset outside every buffer range

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// A raw buffer of 2^31 - 1 bytes from p on.
__device__ __forceinline__ u32x4_t make_srd(const void *p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  u32x4_t r;
  r[0] = (uint32_t)v;
  r[1] = (uint32_t)(v >> 32) & 0xffffu;
  r[2] = 0x7fffffffu;
  r[3] = 0x00020000u;
  return r;
}

// 16 or 4 bytes per lane from the buffer at voff + soff into LDS at
// lds + 16 * lane or lds + 4 * lane; an offset voff >= 2^31 - 1 reads zeros.  In
// asm because the compiler would otherwise wait for every DMA in flight
// before each LDS read; the kernels place those waits themselves.  No register
// output; m0 is reserved, and nothing else in those kernels uses it.
__device__ __forceinline__ void lds_dma16(u32x4_t srd, uint32_t lds, uint32_t voff, uint32_t soff) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, %3 offen lds"
      :
      : "s"(lds), "v"(voff), "s"(srd), "s"(soff)
      : "memory");
}
__device__ __forceinline__ void lds_dma4(u32x4_t srd, uint32_t lds, uint32_t voff) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dword %1, %2, 0 offen lds"
      :
      : "s"(lds), "v"(voff), "s"(srd)
      : "memory");
}

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
