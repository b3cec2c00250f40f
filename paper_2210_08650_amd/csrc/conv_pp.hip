// Implicit-GEMM convolution / linear kernel on 256 x 256 output tiles (bf16,
// gfx950), for layers whose rounds of such tiles fill the chip.
//
// Eight waves, two per SIMD, all load and compute: wave (g, c) owns rows
// 64 g .. + 63 of both 128-row halves of A and columns 32 c .. + 31 of both
// halves of B, a 128 x 64 block in 128 accumulator registers.  Per operand byte
// the tile does 128 FLOP (85 for the 128 x 256 tiles of the persistent
// kernel, whose four producer waves would not fit beside such blocks), and a
// wave reads 0.75 KB of fragments per MFMA.
//
// The two groups g run half a step apart.  A k-tile is two steps, each a memory
// slot (fragments of the next 16 MFMAs out of LDS, four or eight DMAs of a
// later k-tile into it) and a matrix slot (those MFMAs), with a barrier after
// every slot: while one group's waves run their MFMAs, the other's use the LDS
// and the memory pipe of the same SIMDs.  Two stages of 64 KB: each quarter
// of a stage is loaded again as soon as both groups have read it, so a DMA has
// about a k-tile's time to land and the wait never drains the queue.
//
// What bounds it: an 8192 x 4096 x 8192 product on random data, back to back, runs
// at 1.36 PF/s (256 x 128 tiles of the persistent kernel 1.12-1.20, the vendor
// library 1.29-1.57 from run to run).  On a model's layers the rounds of tiles over
// 256 CUs, the stores of a round of tiles at once (they share the loads' counter),
// the residual's loads and GELU cost more: the matrix pipes are busy on 44-48% of
// the cycles in VGG-16's layers at 128 images and 27-32% in ViT-B/16's, with waves
// waiting 27-33% of theirs and no bank conflicts.  Against the kernels those layers
// ran on: ViT-B/16 qkv at 64 images (450 tiles of 12 k-tiles) 62 -> 51 us, fc2
// 81 -> 67 us, ResNet-50's stage-3 shortcut GEMM at 128 images 58 -> 51 us, VGG-16
// conv4_2 at 64 images 262 -> 216 us.  Measured and slower (qkv at 48 us then):
// four slots of 8 MFMAs per k-tile (53 us), reading each fragment into the
// register its predecessor leaves, without groups (52 us), raised wave
// priority around the MFMAs (1-3%), one workgroup per tile instead of the
// persistent loop (50 us).
//
// Each output sums its k-tiles and k-steps in the order of every other bf16
// convolution kernel, so the results have the same bits.
#include <type_traits>

#include "gemm_util.h"
#include "internal.h"

namespace hapi {
namespace {

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int kWaves = 8;
constexpr int kHalf = 128 * BK * 2;      // bytes of half an operand tile (128 rows)
constexpr int kStage = 4 * kHalf;        // A halves 0, 1, then B halves 0, 1
constexpr int kBiasMax = 4096;

// n / d for n < 2^31 by one 64-bit multiply and shift.
struct Magic {
  uint32_t mul;
  int shift;
};
Magic magic_for(int d) {
  int l = 0;
  while (((int64_t)1 << l) < d) ++l;
  const int s = 31 + l;
  return Magic{(uint32_t)((((uint64_t)1 << s) + d - 1) / d), s};
}
__device__ __forceinline__ int mdiv(int n, const Magic &m) { return (int)(((uint64_t)(uint32_t)n * m.mul) >> m.shift); }

struct PPArgs {
  ConvArgs a;
  Magic hw, w;  // divisors of the GEMM row: pixels (or pooling windows) per image and per row
};

// EK: epilogue of bias and ReLU (0), GELU (1), ReLU and 2 x 2 max pooling (2),
// residual and ReLU (3).
template <int LD, int KW, int EK>
__global__ __launch_bounds__(kWaves * 64, 1) void conv_bf16_pp_kernel(PPArgs pa) {
  const ConvArgs &a = pa.a;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * kStage];
  __shared__ __attribute__((aligned(16))) float bias_s[kBiasMax];

  const int tiles_n = (a.N + BN - 1) / BN;
  const int tiles = ((a.M + BM - 1) / BM) * tiles_n;
  const int G = gridDim.x;
  const int wg = xcd_remap(blockIdx.x, G);
  const int t_lo = (int)((int64_t)tiles * wg / G), t_hi = (int)((int64_t)tiles * (wg + 1) / G);
  const int nk = a.Kp / BK;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 2, wn = wave & 3;  // group = wm
  const int lrow = lane & 31, lh = lane >> 5;

  for (int c = t; c < a.N; c += kWaves * 64) bias_s[c] = a.bias ? a.bias[c] : 0.0f;
  __syncthreads();

  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
  const u32x4_t srd_a = make_srd(a.x), srd_b = make_srd(a.w);
  const u32x4_t srd_a2 = make_srd(LD == LD_CAT ? a.x2 : a.x);

  // ---- load stream: the operand half-tiles of k-tile after k-tile, tile after tile
  const int kc0 = ((lane & 7) ^ ((lane >> 4) & 7)) * 8, kc1 = ((lane & 7) ^ ((4 + (lane >> 4)) & 7)) * 8;
  int aoff[4], boff[4], a2off[LD == LD_CAT ? 4 : 1];
  uint32_t amask[4];
  int s_ti = t_lo, s_kt = 0, s_tap = 0, s_cb = 0, s_tapoff = 0;
  const int cpt = (LD == LD_NHWC || LD == LD_CAT) ? a.C / BK : nk;
  const int nk1 = LD == LD_CAT ? a.K1 / BK : nk;
  auto stream_tile = [&] {
    const bool live = s_ti < t_hi;
    const int tile = a.rev ? t_lo + t_hi - 1 - s_ti : s_ti;
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (i >> 1) * 128 + (wave * 2 + (i & 1)) * 8 + (lane >> 3);
      const int kc = (i & 1) ? kc1 : kc0;
      const int m = m0 + r;
      const bool valid = live && m < a.M;
      if (LD == LD_GEMM) {
        aoff[i] = valid ? (int)(((int64_t)m * (a.lda ? a.lda : a.K) + kc) * 2) : (int)kOob;
        amask[i] = 0;
      } else {
        const int mm = valid ? m : 0;
        int n, ho, wo;
        if (EK == 2) {
          const int win = mm >> 2;
          n = mdiv(win, pa.hw);
          const int rem = win - n * ((a.Ho >> 1) * (a.Wo >> 1)), hp = mdiv(rem, pa.w);
          ho = 2 * hp + ((mm >> 1) & 1);
          wo = 2 * (rem - hp * (a.Wo >> 1)) + (mm & 1);
        } else {
          n = mdiv(mm, pa.hw);
          const int rem = mm - n * (a.Ho * a.Wo);
          ho = mdiv(rem, pa.w);
          wo = rem - ho * a.Wo;
        }
        const int hi0 = ho * a.stride - a.pad, wi0 = wo * a.stride - a.pad;
        aoff[i] = (((n * a.H + hi0) * a.W + wi0) * a.C + kc) * 2;
        uint32_t mask = 0;
#pragma unroll
        for (int tap = 0; tap < KW * KW; ++tap)
          mask |= ((unsigned)(hi0 + tap / KW) < (unsigned)a.H && (unsigned)(wi0 + tap % KW) < (unsigned)a.W) ? 1u << tap
                                                                                                             : 0u;
        amask[i] = valid ? mask : 0u;
        if (LD == LD_CAT)
          a2off[LD == LD_CAT ? i : 0] =
              valid ? (((n * a.H2 + ho * a.s2) * a.W2 + wo * a.s2) * a.C2 + kc) * 2 : (int)kOob;
      }
      const int nn = n0 + r;
      boff[i] = live && nn < a.N ? (nn * a.Kp + kc) * 2 : (int)kOob;
    }
    s_kt = s_tap = s_cb = s_tapoff = 0;
  };
  // After the four half-tiles of a k-tile: the next one.
  auto stream_next = [&] {
    if (++s_kt == nk) {
      ++s_ti;
      stream_tile();
      return;
    }
    if (LD == LD_NHWC || LD == LD_CAT) {
      if (++s_cb == cpt) {
        s_cb = 0;
        ++s_tap;
        s_tapoff = ((s_tap / KW) * a.W + s_tap % KW) * a.C * 2;
      }
    }
  };
  auto issue_a = [&](uint32_t stage, int h) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t dst = lds0 + stage + h * kHalf + (wave * 2 + i) * 1024;
      const int x = 2 * h + i;
      if (LD == LD_GEMM) {
        lds_dma16(srd_a, dst, (uint32_t)aoff[x], (uint32_t)(s_kt * BK * 2));
      } else if (LD == LD_CAT && s_kt >= nk1) {
        lds_dma16(srd_a2, dst, (uint32_t)a2off[LD == LD_CAT ? x : 0], (uint32_t)((s_kt - nk1) * BK * 2));
      } else {
        const uint32_t v = (amask[x] >> s_tap) & 1u ? (uint32_t)(aoff[x] + s_tapoff) : kOob;
        lds_dma16(srd_a, dst, v, (uint32_t)(s_cb * BK * 2));
      }
    }
  };
  auto issue_b = [&](uint32_t stage, int h) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      lds_dma16(srd_b, lds0 + stage + (2 + h) * kHalf + (wave * 2 + i) * 1024, (uint32_t)boff[2 * h + i],
            (uint32_t)(s_kt * BK * 2));
  };

  // ---- fragments
  const int sw = (lrow >> 1) & 7;
  int xo[4];  // swizzled chunk of k-step ks
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) xo[ks] = ((2 * ks + lh) ^ sw) * 16;
  const int arow = (wm * 64 + lrow) * 128, brow = 2 * kHalf + (wn * 32 + lrow) * 128;
  bf16x8_t af[2][4], b0[4], b1[4];
  auto read_a = [&](uint32_t stage, int h) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        af[i][ks] = *reinterpret_cast<const bf16x8_t *>(smem + stage + h * kHalf + arow + i * 4096 + xo[ks]);
  };
  auto read_b = [&](uint32_t stage, int h, bf16x8_t(&b)[4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      b[ks] = *reinterpret_cast<const bf16x8_t *>(smem + stage + h * kHalf + brow + xo[ks]);
  };

  f32x16_t acc[4][2];
  int slack = 0;  // phases whose wait has the previous tile's stores among the younger operations
  // End of a memory slot: this wave's fragments are in registers, and its part
  // of the half-tiles that the next memory slot reads has landed (N younger
  // DMAs may be in flight).
  auto mem_end = [&](auto young) {
    constexpr int N = decltype(young)::value;
    if (slack > 0) {
      --slack;
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N + 16) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  using C8 = std::integral_constant<int, 8>;
  auto bar = [&] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mma = [&](int h) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        acc[2 * h + i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0[ks], af[i][ks], acc[2 * h + i][0], 0, 0, 0);
        acc[2 * h + i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1[ks], af[i][ks], acc[2 * h + i][1], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- prologue: two k-tiles (but for A half 1 of the second) in flight
  stream_tile();
  issue_a(0, 0);
  issue_b(0, 0);
  issue_b(0, 1);
  issue_a(0, 1);
  stream_next();
  issue_a(kStage, 0);
  issue_b(kStage, 0);
  issue_b(kStage, 1);
  uint32_t st = 0;  // stage of the k-tile being computed
  mem_end(C8{});
  if (wm == 1) bar();  // the second group runs one slot behind

  const __amdgpu_buffer_rsrc_t ysrd = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrd =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.res ? a.res : a.x), 0, 0x7fffffff, 0x00020000);

  for (int ti = t_lo; ti < t_hi; ++ti) {
    const int tile = a.rev ? t_lo + t_hi - 1 - ti : ti;
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    for (int kt = 0; kt < nk; ++kt) {
      read_a(st, 0);
      read_b(st, 0, b0);
      read_b(st, 1, b1);
      issue_a(st ^ kStage, 1);
      stream_next();
      mem_end(C8{});
      mma(0);
      bar();
      issue_a(st, 0);
      issue_b(st, 0);
      issue_b(st, 1);
      read_a(st, 1);
      mem_end(C8{});
      mma(1);
      if (kt + 1 < nk) bar();
      st ^= kStage;
    }
    if (wm == 0) bar();
    // No DMA may outlive the workgroup's LDS (the last ones read nothing).
    if (ti + 1 == t_hi) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // acc[i][j][4 g + e] = C[row 32 (i % 2) + lane % 32 of the wave's rows in
    // A half i / 2][column 8 g + 4 lh + e of its columns in B half j].
    u32x4_t rr[4][2][2];
    if constexpr (EK == 3) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + (i >> 1) * 128 + wm * 64 + (i & 1) * 32 + lrow;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const int n = n0 + j * 128 + wn * 32 + 16 * p + 8 * lh;
            const uint32_t v = m < a.M && n < a.N ? (uint32_t)((m * a.ldr + n) * 2) : kOob;
            rr[i][j][p] = __builtin_amdgcn_raw_buffer_load_b128(rsrd, v, 0, 0);
          }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + (i >> 1) * 128 + wm * 64 + (i & 1) * 32 + lrow;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const auto s2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][j][8 * p + e]),
                                                             __float_as_uint(acc[i][j][8 * p + 4 + e]), false, false);
            v[e] = __uint_as_float(s2[0]);
            v[4 + e] = __uint_as_float(s2[1]);
          }
          const int n = n0 + j * 128 + wn * 32 + 16 * p + 8 * lh;
          const int nb = n < a.N ? n : 0;
          const float4 c0 = *reinterpret_cast<const float4 *>(bias_s + nb);
          const float4 c1 = *reinterpret_cast<const float4 *>(bias_s + nb + 4);
          v[0] += c0.x; v[1] += c0.y; v[2] += c0.z; v[3] += c0.w;
          v[4] += c1.x; v[5] += c1.y; v[6] += c1.z; v[7] += c1.w;
          if constexpr (EK == 3) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[2 * e] += bf2f((uint16_t)(rr[i][j][p][e] & 0xffff));
              v[2 * e + 1] += bf2f((uint16_t)(rr[i][j][p][e] >> 16));
            }
          }
          u32x4_t o;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            o[e] = f2bf2(epilogue_act(v[2 * e], a.relu, EK == 1), epilogue_act(v[2 * e + 1], a.relu, EK == 1));
          bool ok = m < a.M && n < a.N;
          int row = m;
          if (EK == 2) {
            // rows 4 w .. 4 w + 3 (window w) are lanes l, l ^ 1, l ^ 2, l ^ 3
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              o[e] = bf16x2_max(o[e], (uint32_t)__shfl_xor((int)o[e], 1, 64));
              o[e] = bf16x2_max(o[e], (uint32_t)__shfl_xor((int)o[e], 2, 64));
            }
            ok = ok && (lrow & 3) == 0;
            row = m >> 2;
          }
          // Always issued (16 per tile): the waits of the next phases count them.
          __builtin_amdgcn_raw_buffer_store_b128(o, ysrd, ok ? (uint32_t)((row * a.ldc + n) * 2) : kOob, 0, 0);
        }
    }
    slack = 2;
    if (wm == 1) bar();
  }
  if (wm == 0) bar();
}

template <int LD, int KW, int EK>
hipError_t launch(const PPArgs &pa, hipStream_t s) {
  const ConvArgs &a = pa.a;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const int cus = a.cus > 0 ? a.cus : cu_count();
  hapi_launch((conv_bf16_pp_kernel<LD, KW, EK>), dim3(tiles < cus ? tiles : cus), dim3(kWaves * 64), 0, s, pa);
  return hipGetLastError();
}

template <int LD, int KW>
hipError_t launch_ek(const PPArgs &pa, hipStream_t s) {
  if (pa.a.pool) {
    if constexpr (LD == LD_NHWC && KW == 3) return launch<LD, KW, 2>(pa, s);
    return hipErrorNotSupported;
  }
  if (pa.a.gelu) {
    if constexpr (LD == LD_GEMM) return launch<LD, KW, 1>(pa, s);
    return hipErrorNotSupported;
  }
  if (pa.a.res) {
    if constexpr (LD == LD_GEMM || (LD == LD_NHWC && KW == 3)) return launch<LD, KW, 3>(pa, s);
    return hipErrorNotSupported;
  }
  return launch<LD, KW, 0>(pa, s);
}

}  // namespace

bool conv_pp_supported(const ConvArgs &a, Loader ld) {
  const int64_t lim = (int64_t)1 << 31;
  if (a.Kp < 2 * BK || a.K % BK || a.N > kBiasMax || a.N % 8 || a.ldc % 8 || a.ldr % 8 || a.out_hw || a.pre_scale ||
      (a.res && (a.pool || a.gelu)))
    return false;
  if ((int64_t)a.N * a.Kp * 2 >= lim || (int64_t)a.M * a.ldc * 2 >= lim || (int64_t)a.M * a.ldr * 2 >= lim) return false;
  if (ld == LD_GEMM) return !a.pool && (int64_t)a.M * (a.lda ? a.lda : a.K) * 2 < lim;
  if (ld != LD_NHWC && ld != LD_CAT) return false;
  if (a.gelu || a.C % BK || a.kh != a.kw || (a.kh != 1 && a.kh != 3)) return false;
  if (a.res && (ld == LD_CAT || a.kh == 1)) return false;  // residuals of 3 x 3 and plain 1 x 1 layers only
  if ((int64_t)a.n_img * a.H * a.W * a.C * 2 >= lim) return false;
  return ld == LD_NHWC ? !a.pool || a.kh == 3 : a.C2 % BK == 0 && (int64_t)a.n_img * a.H2 * a.W2 * a.C2 * 2 < lim;
}

hipError_t launch_conv_pp(const ConvArgs &a, Loader ld, hipStream_t s) {
  if (!conv_pp_supported(a, ld)) return hipErrorNotSupported;
  PPArgs pa;
  pa.a = a;
  const bool win = a.pool != 0;
  pa.hw = magic_for(win ? (a.Ho / 2) * (a.Wo / 2) : a.Ho * a.Wo);
  pa.w = magic_for(win ? a.Wo / 2 : a.Wo);
  if (ld == LD_GEMM) return launch_ek<LD_GEMM, 1>(pa, s);
  if (ld == LD_NHWC) return a.kh == 3 ? launch_ek<LD_NHWC, 3>(pa, s) : launch_ek<LD_NHWC, 1>(pa, s);
  return a.kh == 3 ? launch_ek<LD_CAT, 3>(pa, s) : launch_ek<LD_CAT, 1>(pa, s);
}

}  // namespace hapi
