// Group-wise GEMM on BF6 operands for products with few output tiles: the
// layer of w4a4g_f6_gemm_kernel (f6.hip) bit for bit, where its 128 x 128
// tiles would leave most CUs idle.  launch_w4a4g_f6_gemm picks it by
// f6_narrow_group_waves.
//
// What bounds such a product.  A block of the tiled kernel walks all of K at
// 0.8 us (G = 128) or 1.3 us (G = 64) per 128 codes, and 33 x 12288 -> 4096
// gives 32 of them.  The group sum S is a chain of fp32 additions in k order
// that may not be reordered, but its terms t = fl32(fl32(acc_g * s_x) * s_w)
// are independent.  So a block takes a tile of 32 x 32 outputs and splits K
// into rounds of one 128-code unit per wave: every wave computes its unit's
// terms and writes them to LDS, and after one barrier each thread adds its
// outputs' terms to its sums, in k order.  That runs under the next round's
// MFMAs; operands come straight from memory into registers two rounds ahead,
// group scales three (loaded before the operands of their round, so that
// waiting for them does not wait for those).  A round costs 0.64 us (four
// waves) or 1.0 us (eight) at G = 128, 1.05 and 1.6 us at G = 64: the chain
// MFMA -> scaling -> LDS -> barrier -> LDS, and with several blocks per CU
// the LDS traffic of the terms (8 bytes per term).  Eight waves are taken
// where every tile can have its own CU.  Measured back to back, tiled ->
// narrow: 33 x 12288 -> 4096 G = 128 77.9 -> 16.9 us, G = 64 129.4 -> 23.5 us;
// 33 x 4096 -> 12288 G = 128 27.5 -> 13.2 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "f6_common.h"
#include "gemm_common.h"
#include "jq_internal.h"

namespace jq {

namespace {

using namespace gemm_detail;
using namespace f6_detail;

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kLgkm0 = 0xC07F;  // s_waitcnt lgkmcnt(0), the loads in flight left alone

// W waves per block, WPS waves per SIMD at least.
template <int G, int W, int WPS, Epilogue EPI, bool HAS_BIAS>
__global__ __launch_bounds__(64 * W, WPS) void f6_narrow_group_kernel(
    const uint8_t* __restrict__ xf6, const float* __restrict__ sx, int M, int mbands,
    const uint8_t* __restrict__ wf6, const float* __restrict__ sw, int N, int nbands, int ksteps, int KG,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n) {
  constexpr int kGps = 128 / G;                       // groups of a unit
  constexpr int kRg = W * kGps;                       // groups of a round
  constexpr int kScLoads = 64 * kRg / (64 * W);       // scale entries per thread and round (64 rows x kRg)
  constexpr int kVo = 1024 / (64 * W);                // outputs per thread
  typedef float vout __attribute__((ext_vector_type(kVo)));
  // A round's terms [group][32 rows][eight 16-byte chunks of columns], and
  // its scales [group][32 rows of x, 32 rows of w]; two rounds of each.
  __shared__ v4f red[2][kRg * 256];
  __shared__ float scs[2][kRg * 64];
  TileCoord tc;
  if (!tile_of_block(blockIdx.x, tiles_m, tiles_n, &tc)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = 32 * tc.tm, n0 = 32 * tc.tn;
  const int T = ksteps / 2;  // units of 128 codes
  const uint32_t band_bytes = static_cast<uint32_t>(ksteps) * kFragBytes;

  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(xf6), 0, static_cast<int>(mbands * band_bytes), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(wf6), 0, static_cast<int>(nbands * band_bytes), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(sx), 0, static_cast<int>(4u * static_cast<uint32_t>(M) * KG), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rsw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(sw), 0, static_cast<int>(4u * static_cast<uint32_t>(N) * KG), kBufferFlags);
  // Rows past M, columns past N and units past K read as zero (outside the
  // buffers, without touching memory).
  const bool live = m0 + (lane & 31) < M;
  const uint32_t xbase = static_cast<uint32_t>(tc.tm) * band_bytes;
  const uint32_t xo16 = live ? xbase + 16 * lane : kOutside;
  const uint32_t xo8 = live ? xbase + 1024 + 8 * lane : kOutside;
  const uint32_t wo = static_cast<uint32_t>(tc.tn) * band_bytes + 16 * lane;
  // Scale entry e of a round is group e % kRg of row e / kRg (32 rows of x,
  // then 32 of w): the neighbouring groups of a row are neighbours in memory.
  uint32_t sox[kScLoads], sow[kScLoads];
  int sg[kScLoads], sdst[kScLoads];
  bool s_is_w[kScLoads];
#pragma unroll
  for (int j = 0; j < kScLoads; ++j) {
    const int e = tid + 64 * W * j;
    const int r = e / kRg;
    sg[j] = e % kRg;
    s_is_w[j] = r >= 32;
    const int row = s_is_w[j] ? n0 + r - 32 : m0 + r;
    const uint32_t o = 4u * (static_cast<uint32_t>(row) * KG + sg[j]);
    sox[j] = !s_is_w[j] && row < M ? o : kOutside;
    sow[j] = s_is_w[j] && row < N ? o : kOutside;
    sdst[j] = sg[j] * 64 + r;
  }
  float sreg[2][kScLoads];
  auto load_scales = [&](int round, int k) __attribute__((always_inline)) {
    const int so = 4 * kRg * round;
#pragma unroll
    for (int j = 0; j < kScLoads; ++j) {
      const bool in = round * kRg + sg[j] < KG;
      const uint32_t a = __builtin_amdgcn_raw_buffer_load_b32(rsx, in ? sox[j] : kOutside, so, 0);
      const uint32_t b = __builtin_amdgcn_raw_buffer_load_b32(rsw, in ? sow[j] : kOutside, so, 0);
      sreg[k][j] = __uint_as_float(s_is_w[j] ? b : a);
    }
  };
  auto store_scales = [&](int buf, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kScLoads; ++j) scs[buf][sdst[j]] = sreg[k][j];
  };

  v4i32 w[2][3], x16[2][2];
  v2i32 x8[2][2];
  auto issue = [&](auto D_, int i) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
    const int u = wave + W * i;
    const bool in = u < T;
    const int so = in ? u * 2 * kFragBytes : 0;
#pragma unroll
    for (int p = 0; p < 3; ++p)
      w[d][p] = __builtin_bit_cast(
          v4i32, __builtin_amdgcn_raw_buffer_load_b128(rw, in ? wo + 1024 * p : kOutside, so, 0));
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      x16[d][s] = __builtin_bit_cast(
          v4i32, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? xo16 + kFragBytes * s : kOutside, so, 0));
      x8[d][s] = __builtin_bit_cast(
          v2i32, __builtin_amdgcn_raw_buffer_load_b64(rx, in ? xo8 + kFragBytes * s : kOutside, so, 0));
    }
  };

  // A lane's results of a 32x32 MFMA are column m = lane & 31 and rows
  // n = 8j + 4 (lane >> 5) + r of y^T: chunk 2j + (lane >> 5) of row m, at
  // slot chunk ^ (m & 7).  Thread tid sums outputs kVo oc .. of row om.
  const int h = lane >> 5, ml = lane & 31;
  constexpr int kCpr = 32 / kVo;
  const int oc = tid % kCpr, om = tid / kCpr;
  const int oslot = (om * 8 + ((oc * kVo / 4) ^ (om & 7))) * 4 + oc * kVo % 4;
  vout S{};
  // Add round i's terms in k order; groups past K do not exist.
  auto sum = [&](int i) __attribute__((always_inline)) {
    const float* p = reinterpret_cast<const float*>(red[i & 1]) + oslot;
#pragma unroll
    for (int g = 0; g < kRg; ++g) {
      const vout t = *reinterpret_cast<const vout*>(p + 1024 * g);
      if (kRg * i + g < KG) S += t;
    }
  };
  auto round = [&](auto D_, int i) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
    const v8i x0{x16[d][0].x, x16[d][0].y, x16[d][0].z, x16[d][0].w, x8[d][0].x, x8[d][0].y, 0, 0};
    const v8i x1{x16[d][1].x, x16[d][1].y, x16[d][1].z, x16[d][1].w, x8[d][1].x, x8[d][1].y, 0, 0};
    const v8i w0 = __builtin_shufflevector(w[d][0], w[d][1], 0, 1, 2, 3, 4, 5, -1, -1);
    const v8i w1 = __builtin_shufflevector(w[d][1], w[d][2], 2, 3, 4, 5, 6, 7, -1, -1);
    v16f a[kGps];
    a[0] = mfma_bf6(w0, x0, v16f{});
    if constexpr (G == 64)
      a[1] = mfma_bf6(w1, x1, v16f{});
    else
      a[0] = mfma_bf6(w1, x1, a[0]);
    __builtin_amdgcn_sched_barrier(0);
    store_scales((i + 1) & 1, (d + 1) & 1);
    __builtin_amdgcn_sched_barrier(0);
    load_scales(i + 3, (d + 1) & 1);
    issue(D_, i + 2);
    __builtin_amdgcn_sched_barrier(0);
    if (i > 0) sum(i - 1);
#pragma unroll
    for (int gl = 0; gl < kGps; ++gl) {
      const int g = kGps * wave + gl;
      const float* s = scs[i & 1] + 64 * g;
      const float sxv = s[ml];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const v4f sv = *reinterpret_cast<const v4f*>(s + 32 + 8 * j + 4 * h);
        v4f t;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = a[gl][4 * j + r] * sxv;
          t[r] = v * sv[r];
        }
        red[i & 1][(32 * g + ml) * 8 + ((2 * j + h) ^ (ml & 7))] = t;
      }
    }
    // One barrier per round: the terms and the next round's scales are in
    // LDS.  Buffer i & 1 is written again in round i + 2, after the barrier
    // of round i + 1, which every wave reaches only after its sum(i).
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  const int iters = (T + W - 1) / W;
  const std::integral_constant<int, 0> c0{};
  const std::integral_constant<int, 1> c1{};
  load_scales(0, 0);
  load_scales(1, 1);
  __builtin_amdgcn_sched_barrier(0);
  issue(c0, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue(c1, 1);
  __builtin_amdgcn_sched_barrier(0);
  store_scales(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_scales(2, 0);
  __syncthreads();
  for (int i = 0; i < iters; i += 2) {
    round(c0, i);
    if (i + 1 < iters) round(c1, i + 1);
  }
  sum(iters - 1);

  const int row = m0 + om, n = n0 + kVo * oc;
  if (row >= M || n >= N) return;
  const int64_t at = static_cast<int64_t>(row) * N + n;
  if constexpr (EPI == Epilogue::kF32) {
    float* o = static_cast<float*>(out) + at;
#pragma unroll
    for (int r = 0; r < kVo; ++r)
      if (n + r < N) o[r] = S[r];
  } else {
    uint16_t y[kVo];
#pragma unroll
    for (int r = 0; r < kVo; ++r) {
      float v = S[r];
      if (HAS_BIAS) v = v + __uint_as_float(static_cast<uint32_t>(bias[min(n + r, N - 1)]) << 16);
      y[r] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
    }
    uint16_t* o = static_cast<uint16_t*>(out) + at;
    if (N % 2 == 0) {  // pairs: 4-byte aligned, and n + r + 1 < N where n + r < N
#pragma unroll
      for (int r = 0; r < kVo; r += 2)
        if (n + r < N) *reinterpret_cast<uint32_t*>(o + r) = y[r] | (static_cast<uint32_t>(y[r + 1]) << 16);
    } else {
#pragma unroll
      for (int r = 0; r < kVo; ++r)
        if (n + r < N) o[r] = y[r];
    }
  }
}

}  // namespace

// Waves per block (4 or 8) of the narrow kernel for an M x K by K x N
// product, or 0 where the tiled kernel is estimated faster.  n and n_tiled
// are the tiles of the CU that has most.  In ns: a narrow round costs what
// the head of this file says for a block alone, and 390 (G = 128) or 660
// (G = 64, two blocks at a time) per block where that is more; the tiled
// kernel 800 or 1330 per 128 codes for a block alone on its CU, 1180 or 1720
// for two.  Measured over M 1..2048, K 256..12288, N 256..12288; a call
// changes over only where the estimate says at least 8% less.
int f6_narrow_group_waves(int64_t M, int64_t N, int64_t K, int G, int64_t cus) {
  const int64_t units = (K + 127) / 128;
  const int64_t n = ((M + 31) / 32 * ((N + 31) / 32) + cus - 1) / cus;
  const int64_t n_tiled = ((M + 127) / 128 * ((N + 127) / 128) + cus - 1) / cus;
  if (n_tiled > 4) return 0;
  const bool g64 = G == 64;
  const int64_t tiled = 2500 + units * (n_tiled / 2 * (g64 ? 1720 : 1180) + n_tiled % 2 * (g64 ? 1330 : 800));
  const int64_t r4 = g64 ? std::max<int64_t>(1050, (n + 1) / 2 * 1320) : std::max<int64_t>(640, 390 * n);
  const int64_t t4 = 3200 + (units + 3) / 4 * r4;
  const int64_t t8 = 3500 + (units + 7) / 8 * (g64 ? 1600 : 1000);
  if (n == 1 && t8 < t4 && t8 < tiled * 92 / 100) return 8;
  return t4 < tiled * 92 / 100 ? 4 : 0;
}

hipError_t launch_f6_narrow_group(int waves, Epilogue epi, const uint8_t* xf6, const float* sx, int64_t M, int64_t K,
                                  int G, const uint8_t* wf6, const float* sw, int64_t N, const uint16_t* bias,
                                  void* out, hipStream_t st) {
  const int ksteps = static_cast<int>(f6_ksteps(K));
  const int mbands = static_cast<int>((M + 31) / 32), nbands = static_cast<int>((N + 31) / 32);
  const unsigned blocks =
      static_cast<unsigned>((static_cast<int64_t>(mbands) * nbands + kNumXcd - 1) / kNumXcd * kNumXcd);
  const int Mi = static_cast<int>(M), Ni = static_cast<int>(N), KG = static_cast<int>(K / G);
#define JQ_NG(GG, W, WPS, E, B)                                                                                    \
  hipLaunchKernelGGL((f6_narrow_group_kernel<GG, W, WPS, E, B>), dim3(blocks), dim3(64 * W), 0, st, xf6, sx, Mi,   \
                     mbands, wf6, sw, Ni, nbands, ksteps, KG, bias, out, mbands, nbands)
#define JQ_NG_EPI(GG, W, WPS)                                               \
  if (epi == Epilogue::kF32) JQ_NG(GG, W, WPS, Epilogue::kF32, false);      \
  else if (bias != nullptr) JQ_NG(GG, W, WPS, Epilogue::kBf16, true);       \
  else JQ_NG(GG, W, WPS, Epilogue::kBf16, false);
  if (G == 64) {
    if (waves == 8) {
      JQ_NG_EPI(64, 8, 2)
    } else {
      JQ_NG_EPI(64, 4, 2)
    }
  } else {
    if (waves == 8) {
      JQ_NG_EPI(128, 8, 4)
    } else {
      JQ_NG_EPI(128, 4, 3)
    }
  }
#undef JQ_NG_EPI
#undef JQ_NG
  return hipGetLastError();
}

}  // namespace jq
