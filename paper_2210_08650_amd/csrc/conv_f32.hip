// fp32 implicit-GEMM convolutions for gfx950: v_mfma_f32_32x32x2f32, k-tiles of
// 16, reductions cut into slices whose count depends on K only (f32_splits).
#include <type_traits>

#include "gemm_util.h"
#include "internal.h"

namespace hapi {
namespace {

constexpr int kThreads = 256;
constexpr int BKF = kF32Tile;  // k-tile (fp32 elements)
constexpr int LDSF = BKF + 4;  // LDS row pitch in floats (80 B)

template <int LD>
__device__ __forceinline__ float4 load_a_chunk_f32(const ConvArgs &a, const RowState &r, int k0,
                                                   int kh_, int kw_, int c0) {
  const float *x = static_cast<const float *>(a.x);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (LD == LD_GEMM) {
    if (r.hi0 >= 0) v = *reinterpret_cast<const float4 *>(x + r.base + k0);
  } else if (LD == LD_NHWC) {
    const int hi = r.hi0 + kh_, wi = r.wi0 + kw_;
    if ((unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W)
      v = *reinterpret_cast<const float4 *>(x + r.base + (hi * a.W + wi) * a.C + c0);
  } else {  // LD_NCHW element gather, k = (c, u, v)
    if (r.hi0 > -(1 << 27)) {
      float e[4];
      const int khw = a.kh * a.kw;
      int c = k0 / khw, rem = k0 - c * khw;
      int u = rem / a.kw, vv = rem - u * a.kw;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int hi = r.hi0 + u, wi = r.wi0 + vv;
        e[j] = (k0 + j < a.K && (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W)
                   ? x[r.base + (c * a.H + hi) * a.W + wi]
                   : 0.0f;
        if (++vv == a.kw) { vv = 0; if (++u == a.kh) { u = 0; ++c; } }
      }
      v = make_float4(e[0], e[1], e[2], e[3]);
    }
  }
  return v;
}

// Register-staged tiles of 64 x 64, double-buffered, for what the DMA kernel
// below cannot address (f32_dma_fits).
template <int LD>
__global__ __launch_bounds__(kThreads) void conv_f32_kernel(ConvArgs a) {
  constexpr int BM = 64, BN = 64;  // four waves of 32 x 32, one float4 chunk of A and B per thread

  __shared__ __attribute__((aligned(16))) float smem[2 * (BM + BN) * LDSF];

  const int tiles_n = (a.N + BN - 1) / BN;
  const int tile = a.rev ? (int)gridDim.x - 1 - xcd_remap(blockIdx.x, gridDim.x) : xcd_remap(blockIdx.x, gridDim.x);
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;

  const int t = threadIdx.x;
  const int kc = t & 3;   // float4 chunk of the 16-wide k-tile
  const int r0 = t >> 2;  // row

  const RowState rs = make_row<LD>(a, m0 + r0);

  const float *wp = static_cast<const float *>(a.w);
  float4 ra, rb;
  auto load_tile = [&](int kt) {
    const int kbase = kt * BKF;
    int kh_ = 0, kw_ = 0, c0 = 0;
    if (LD == LD_NHWC) {  // C % 16 == 0: the k-tile lies in one tap
      const int tap = kbase / a.C;
      c0 = kbase - tap * a.C + kc * 4;
      kh_ = tap / a.kw;
      kw_ = tap - kh_ * a.kw;
    }
    ra = load_a_chunk_f32<LD>(a, rs, kbase + kc * 4, kh_, kw_, c0);
    const int n = n0 + r0;
    rb = (n < a.N) ? *reinterpret_cast<const float4 *>(wp + (size_t)n * a.Kp + kbase + kc * 4)
                   : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto store_tile = [&](int buf) {
    float *As = smem + buf * (BM + BN) * LDSF + r0 * LDSF + kc * 4;
    *reinterpret_cast<float4 *>(As) = ra;
    *reinterpret_cast<float4 *>(As + BM * LDSF) = rb;
  };

  const int lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lrow = lane & 31, lk = (lane >> 5) * 8;

  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

  // k-tiles [kt0, kt1): slice blockIdx.y of a split reduction, or all of them.
  const int nk_all = a.Kp / BKF;
  const int S = a.splits > 1 ? a.splits : 1;
  const int kt0 = (int)((int64_t)nk_all * blockIdx.y / S), kt1 = (int)((int64_t)nk_all * (blockIdx.y + 1) / S);
  load_tile(kt0);
  store_tile(0);
  __syncthreads();
  for (int kt = kt0; kt < kt1; ++kt) {
    const int cur = (kt - kt0) & 1;
    if (kt + 1 < kt1) load_tile(kt + 1);
    const float *As = smem + cur * (BM + BN) * LDSF + (wm * 32 + lrow) * LDSF + lk;
    const float *Bs = smem + cur * (BM + BN) * LDSF + BM * LDSF + (wn * 32 + lrow) * LDSF + lk;
    // Lane half h feeds k = 8h + s at step s to both operands, so the 8 steps
    // cover the 16 k of the tile exactly once.
    const float4 pa = *reinterpret_cast<const float4 *>(As), qa = *reinterpret_cast<const float4 *>(As + 4);
    const float4 pb = *reinterpret_cast<const float4 *>(Bs), qb = *reinterpret_cast<const float4 *>(Bs + 4);
    const float av[8] = {pa.x, pa.y, pa.z, pa.w, qa.x, qa.y, qa.z, qa.w};
    const float bv[8] = {pb.x, pb.y, pb.z, pb.w, qb.x, qb.y, qb.z, qb.w};
#pragma unroll
    for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], bv[s], acc, 0, 0, 0);
    if (kt + 1 < kt1) store_tile(cur ^ 1);
    __syncthreads();
  }

  const int n = n0 + wn * 32 + lrow;
  if (n >= a.N) return;
  const int mb = m0 + wm * 32 + 4 * (lane >> 5);
  if (S > 1) {  // partial sums of this slice; bias and activation come after the sum
    float *part = a.part + (int64_t)blockIdx.y * a.M * a.N;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mb + 8 * (r >> 2) + (r & 3);
      if (m < a.M) part[(int64_t)m * a.N + n] = acc[r];
    }
    return;
  }
  float *y = static_cast<float *>(a.y);
  const float *res = static_cast<const float *>(a.res);
  const float bias = a.bias ? a.bias[n] : 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = mb + 8 * (r >> 2) + (r & 3);
    if (m >= a.M) continue;
    float v = acc[r] + bias;
    if (res) v += res[(int64_t)m * a.ldr + n];
    y[(int64_t)m * a.ldc + n] = epilogue_act(v, a.relu, a.gelu);
  }
}

// ------------------------------------------------------- LDS-DMA pipeline

// fp32 MFMAs are slow (64 clocks for 4096 FLOP), so the matrix pipe bounds this
// once it never waits: tiles go by DMA into an ST-stage ring, and each half of
// a wave's fragments is read into the registers that the MFMAs just issued
// leave.  AlexNet conv2 at 64 images 122-126 TF/s with two partitions in
// flight (register-staged, double-buffered tiles with partial sums: 95), conv3
// 107 (80), the 11 x 11 / 4 first layer 70 (66); AlexNet b128 1,911 -> 1,574 us,
// b4 154 -> 137 us (fp32 peak 157, a library 8192^3 product 154 TF/s).
//
// Four waves of BM / 2 x BN / 2, ST stages of one 16-wide k-tile.  SEQ: a workgroup
// runs every slice of its tile, one after another, into one sum (total = slice
// 0, + slice 1, ...: what the split reduction adds, bit for bit); otherwise
// slice blockIdx.y goes to the partial sums.
//
// LD_NHWC (1 x 1 included): rows of 64 bytes by 16-byte DMA, chunk c of row r at
// position c ^ ((r >> 2) & 3), so the 16 rows a quarter-wave fragment read touches
// lie in 16 distinct 16-byte slots of 256 bytes.  LD_NCHW: elements by 4-byte
// DMA, each lane its own address (tap offsets from a table in LDS); four rows per
// instruction, 16 bytes of padding after each four for the same spread.
template <int BM, int BN, int ST, int LD, bool SEQ>
__global__ __launch_bounds__(kThreads, 2) void conv_f32_dma_kernel(ConvArgs a) {
  constexpr int TM = BM / 64, TN = BN / 64;
  constexpr bool GATHER = LD == LD_NCHW;
  constexpr int NA = GATHER ? BM / 16 : BM / 64, NB = BN / 64, NQ = NA + NB;  // DMAs per lane per k-tile
  constexpr int kGroup = GATHER ? 272 : 256;                                  // bytes of four A rows
  constexpr int kA = BM / 4 * kGroup, kStage = kA + BN * 64;
  static_assert((ST - 2) * NQ < 64 && TM >= 1 && TN >= 1, "tile");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[ST * kStage];
  __shared__ __attribute__((aligned(16))) int2 taps[GATHER ? kF32Taps : 1];

  const int tiles_n = (a.N + BN - 1) / BN;
  const int tile = a.rev ? (int)gridDim.x - 1 - xcd_remap(blockIdx.x, gridDim.x) : xcd_remap(blockIdx.x, gridDim.x);
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
  const u32x4_t srd_a = make_srd(a.x), srd_b = make_srd(a.w);

  const int nk = a.Kp / BKF;
  const int S = a.splits > 1 ? a.splits : 1;
  const int sl0 = SEQ ? 0 : (int)blockIdx.y, sl1 = SEQ ? S : sl0 + 1;
  const int kt_lo = (int)((int64_t)nk * sl0 / S), kt_hi = (int)((int64_t)nk * sl1 / S);

  if (GATHER) {
    const int khw = a.kh * a.kw;
    for (int k = t; k < a.Kp; k += kThreads) {
      const int c = k / khw, rem = k - c * khw, u = rem / a.kw, v = rem - u * a.kw;
      taps[k] = k < a.K ? make_int2(((c * a.H + u) * a.W + v) * 4, (u << 16) | v) : make_int2(0, 0x40000000);
    }
    __syncthreads();
  }

  // This lane's rows: of DMA i, row 16 g + lane / 4 (g = NA wave + i), or
  // 4 g + lane / 16 of the gather.
  int rbase[NA], rhi[NA], rwi[NA];
  uint32_t boff[NB];
  const int lc = ((lane & 3) ^ ((lane >> 4) & 3)) * 4;
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const RowState r = make_row<LD>(a, m0 + (wave * NA + i) * (GATHER ? 4 : 16) + lane / (GATHER ? 16 : 4));
    rhi[i] = r.hi0;
    rwi[i] = r.wi0;
    // bytes from the buffer's start; the row's first tap may lie in the padding
    const int px = r.hi0 > -(1 << 27) ? r.hi0 * a.W + r.wi0 : 0;
    rbase[i] = (GATHER ? r.base + px : r.base + px * a.C + lc) * 4;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = n0 + (wave * NB + j) * 16 + (lane >> 2);
    boff[j] = n < a.N ? (uint32_t)((n * a.Kp + lc) * 4) : kOob;
  }

  // Load stream: k-tile s_kt next, (tap row, tap column, channel) of its first k.
  int s_kt = kt_lo, s_kh = 0, s_kw = 0, s_c = 0, stage_w = 0;
  if (!GATHER) {
    const int tap = kt_lo * BKF / a.C;
    s_c = kt_lo * BKF - tap * a.C;
    s_kh = tap / a.kw;
    s_kw = tap - s_kh * a.kw;
  }
  auto issue = [&] {
    const uint32_t st = lds0 + stage_w * kStage;
    const bool live = s_kt < kt_hi;
    if constexpr (GATHER) {
      const int2 tp = taps[live ? s_kt * BKF + (lane & 15) : 0];
      const int u = live ? tp.y >> 16 : 0x4000, v = tp.y & 0xffff;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const bool ok = (unsigned)(rhi[i] + u) < (unsigned)a.H && (unsigned)(rwi[i] + v) < (unsigned)a.W;
        lds_dma4(srd_a, st + (wave * NA + i) * kGroup, ok ? (uint32_t)(rbase[i] + tp.x) : kOob);
      }
    } else {
      const int off = live ? ((s_kh * a.W + s_kw) * a.C + s_c) * 4 : 0, kh = live ? s_kh : 0x4000;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const bool ok = (unsigned)(rhi[i] + kh) < (unsigned)a.H && (unsigned)(rwi[i] + s_kw) < (unsigned)a.W;
        lds_dma16(srd_a, st + (wave * NA + i) * 1024, ok ? (uint32_t)(rbase[i] + off) : kOob, 0);
      }
      s_c += BKF;
      if (s_c == a.C) {
        s_c = 0;
        if (++s_kw == a.kw) {
          s_kw = 0;
          ++s_kh;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
      lds_dma16(srd_b, st + kA + (wave * NB + j) * 1024, live ? boff[j] : kOob, (uint32_t)(live ? s_kt * BKF * 4 : 0));
    ++s_kt;
    stage_w = stage_w + 1 == ST ? 0 : stage_w + 1;
  };

  const int wm = wave >> 1, wn = wave & 1;
  const int lrow = lane & 31, lh = lane >> 5;
  // Lane half h feeds k = 8 h + s at step s to both operands, so the 8 steps
  // cover the 16 k of the tile exactly once: two 16-byte chunks per row.
  int aoff[2], boffs[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int c = 2 * lh + e, sc = (c ^ ((lrow >> 2) & 3)) * 16;
    const int ar = wm * TM * 32 + lrow, br = wn * TN * 32 + lrow;
    aoff[e] = GATHER ? (ar >> 2) * kGroup + (ar & 3) * 64 + c * 16 : ar * 64 + sc;
    boffs[e] = kA + br * 64 + sc;
  }

  f32x16_t acc[TM][TN], total[SEQ ? TM : 1][SEQ ? TN : 1];
  float av[TM][8], bv[TN][8];
  int stage_r = 0;  // stage of the k-tile whose fragments are read next
  auto read_frags = [&](auto ec) {
    constexpr int e = decltype(ec)::value;
    const uint8_t *S0 = smem + stage_r * kStage;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float4 p = *reinterpret_cast<const float4 *>(S0 + aoff[e] + i * 8 * kGroup);
      av[i][4 * e] = p.x; av[i][4 * e + 1] = p.y; av[i][4 * e + 2] = p.z; av[i][4 * e + 3] = p.w;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float4 p = *reinterpret_cast<const float4 *>(S0 + boffs[e] + j * 2048);
      bv[j][4 * e] = p.x; bv[j][4 * e + 1] = p.y; bv[j][4 * e + 2] = p.z; bv[j][4 * e + 3] = p.w;
    }
  };
  auto mma = [&](auto ec) {
    constexpr int e = decltype(ec)::value;
#pragma unroll
    for (int s = 4 * e; s < 4 * e + 4; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][s], bv[j][s], acc[i][j], 0, 0, 0);
  };
  // Waits until all but the N youngest k-tiles of this wave have landed, then
  // for every wave: the next k-tile can be read, and the stage before the one
  // being computed is free.
  auto sync = [&](auto young) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(young)::value * NQ) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  using E0 = std::integral_constant<int, 0>;
  using E1 = std::integral_constant<int, 1>;
#pragma unroll
  for (int st = 0; st < ST - 1; ++st) issue();
  sync(std::integral_constant<int, ST - 2>{});
  read_frags(E0{});
  read_frags(E1{});
  stage_r = 1;
  for (int sl = sl0; sl < sl1; ++sl) {
    const int k0 = (int)((int64_t)nk * sl / S), k1 = (int)((int64_t)nk * (sl + 1) / S);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    for (int kt = k0; kt < k1; ++kt) {
      // Each half of the next k-tile's fragments goes into the registers that
      // the MFMAs just issued leave, so no MFMA waits for the LDS.
      sync(std::integral_constant<int, ST - 3>{});
      issue();
      mma(E0{});
      __builtin_amdgcn_sched_barrier(0);
      read_frags(E0{});
      __builtin_amdgcn_sched_barrier(0);
      mma(E1{});
      __builtin_amdgcn_sched_barrier(0);
      read_frags(E1{});
      stage_r = stage_r + 1 == ST ? 0 : stage_r + 1;
    }
    if constexpr (SEQ) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) total[i][j][r] = sl == 0 ? acc[i][j][r] : total[i][j][r] + acc[i][j][r];
    }
  }
  // No DMA may outlive the workgroup's LDS (the last ones read nothing).
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // A lane holds column n = lane % 32 and rows 8 (r / 4) + 4 (lane / 32) + r % 4.
  float *y = static_cast<float *>(a.y);
  float *part = SEQ ? nullptr : a.part + (int64_t)blockIdx.y * a.M * a.N;
  const float *res = static_cast<const float *>(a.res);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn * TN * 32 + j * 32 + lrow;
    if (n >= a.N) continue;
    const float bias = SEQ && a.bias ? a.bias[n] : 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int mb = m0 + wm * TM * 32 + i * 32 + 4 * lh;
      float rv[16];
      if (SEQ && res) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = mb + 8 * (r >> 2) + (r & 3);
          rv[r] = m < a.M ? res[(int64_t)m * a.ldr + n] : 0.0f;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mb + 8 * (r >> 2) + (r & 3);
        if (m >= a.M) continue;
        if constexpr (SEQ) {
          float v = total[i][j][r] + bias;
          if (res) v += rv[r];
          y[(int64_t)m * a.ldc + n] = epilogue_act(v, a.relu, a.gelu);
        } else {
          part[(int64_t)m * a.N + n] = acc[i][j][r];
        }
      }
    }
  }
}

// Sum of the slices in slice order, then bias, residual and activation (the
// unsplit epilogue's order), 4 channels per thread.
__global__ void f32_split_reduce_kernel(ConvArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int ng = a.N / 4;
  if (i >= (int64_t)a.M * ng) return;
  const int64_t m = i / ng;
  const int n = (int)(i - m * ng) * 4;
  const int64_t stride = (int64_t)a.M * a.N;
  float4 v = *reinterpret_cast<const float4 *>(a.part + m * a.N + n);
  for (int sl = 1; sl < a.splits; ++sl) {
    const float4 p = *reinterpret_cast<const float4 *>(a.part + sl * stride + m * a.N + n);
    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
  }
  float o[4] = {v.x, v.y, v.z, v.w};
  const float *res = static_cast<const float *>(a.res);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = o[e] + (a.bias ? a.bias[n + e] : 0.0f);
    if (res) x += res[m * a.ldr + n + e];
    o[e] = epilogue_act(x, a.relu, a.gelu);
  }
  float *y = static_cast<float *>(a.y);
#pragma unroll
  for (int e = 0; e < 4; ++e) y[m * a.ldc + n + e] = o[e];
}

template <int LD>
hipError_t launch_f32_staged(const ConvArgs &a, hipStream_t s) {
  const int tiles = ((a.M + 63) / 64) * ((a.N + 63) / 64);
  const int S = a.splits > 1 ? a.splits : 1;
  if (S > 1 && (!a.part || a.N % 4 != 0 || a.Kp / BKF < S)) return hipErrorInvalidValue;
  hapi_launch(conv_f32_kernel<LD>, dim3(tiles, S), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <int BM, int BN, int ST, int LD, bool SEQ>
hipError_t launch_dma_cfg(const ConvArgs &a, hipStream_t s) {
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hapi_launch((conv_f32_dma_kernel<BM, BN, ST, LD, SEQ>), dim3(tiles, SEQ ? 1 : a.splits), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <int LD>
hipError_t launch_f32_ld(const ConvArgs &a, hipStream_t s) {
  if (!f32_seq(a, (Loader)LD)) {
    if (!a.part || a.N % 4 != 0 || a.Kp / BKF < a.splits) return hipErrorInvalidValue;
    return launch_dma_cfg<64, 64, 5, LD, false>(a, s);
  }
  // 128 x 64 tiles move 3/4 of the operand bytes per FLOP, but a round of them
  // over the CUs is twice as coarse: from four per CU on (AlexNet b100
  // 1,445 -> 1,373 us and b32 514 -> 499 us against from one per CU on, b256
  // 2,904 -> 2,936 us).
  if ((int64_t)((a.M + 127) / 128) * ((a.N + 63) / 64) >= 4 * (int64_t)a.cus) return launch_dma_cfg<128, 64, 4, LD, true>(a, s);
  return launch_dma_cfg<64, 64, 5, LD, true>(a, s);
}

}  // namespace

hipError_t launch_f32_split_reduce(const ConvArgs &a, hipStream_t s) {
  if (a.splits <= 1 || !a.part || a.N % 4 != 0) return hipErrorInvalidValue;
  const int64_t items = (int64_t)a.M * (a.N / 4);
  hapi_launch(f32_split_reduce_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_conv_f32(const ConvArgs &a, Loader ld, hipStream_t s) {
  const bool dma = f32_dma_fits(a, ld);
  switch (ld) {
    case LD_NHWC:
    case LD_GEMM:
      if (dma) return launch_f32_ld<LD_NHWC>(a, s);
      return ld == LD_NHWC ? launch_f32_staged<LD_NHWC>(a, s) : launch_f32_staged<LD_GEMM>(a, s);
    case LD_NCHW:
      if (dma) return launch_f32_ld<LD_NCHW>(a, s);
      return launch_f32_staged<LD_NCHW>(a, s);
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace hapi
