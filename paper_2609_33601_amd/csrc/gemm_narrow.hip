// Packed-int4 (and packed-ternary) GEMM for products with few output tiles:
// the layer of w4a4_gemm_kernel (gemm.hip) bit for bit, where its 128 x 256
// tiles would leave most CUs idle.  launch_w4a4_gemm picks it by
// gemm_narrow_tile.
//
// What bounds such a product.  A block of the tiled kernel walks all of K
// alone at 0.9 us per 128 codes (the latency of its loads and two barriers a
// stage), and 64 x 12288 -> 3072 gives 12 of them.  Here a block takes a tile
// of 32 or 64 rows x 32 .. 96 columns and its four waves split K: wave w
// takes the units w, w + 4, ... of the whole tile (128 codes; 256 with
// ternary weights, 64 bytes of a weight row either way), loads them straight
// into registers two units ahead and widens both operands itself, with no
// LDS or barrier in the loop.  The int32 partial sums meet once, in LDS.
// The operands are row-major, so a load instruction spans 16 rows of 64
// bytes, and a CU takes in 42 KB/us (the 6-bit engine's consecutive
// fragments reach 115): that rate times the bytes of the CU with the most
// tiles is the time.  128-byte row pieces per unit and four units ahead were
// no faster.  Measured back to back, tiled -> narrow: 64 x 4096 -> 12288
// 34.9 -> 11.6 us, 64 x 12288 -> 3072 89.3 -> 13.4 us, 512 x 12288 -> 3072
// 93.0 -> 33.3 us; ternary 64 x 12288 -> 3072 96.6 -> 11.4 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "jq_internal.h"

namespace jq {

namespace {

using namespace gemm_detail;

typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kW = 4;  // waves of a block, splitting K

// MB x NB sub-tiles of 32 rows x 32 columns per block, each 2 x 2 MFMA tiles
// of 16 x 16; WPS waves per SIMD at least; P sub-tiles meet in LDS per pass.
template <WeightFormat WF, int MB, int NB, int WPS, int P, Epilogue EPI, bool HAS_BIAS>
__global__ __launch_bounds__(64 * kW, WPS) void gemm_narrow_kernel(
    const uint8_t* __restrict__ qx, const float* __restrict__ sx, int M, int K,
    const uint8_t* __restrict__ qw, const float* __restrict__ sw, int N,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n) {
  constexpr bool kTern = WF == WeightFormat::kTernary;
  constexpr int kXL = kTern ? 2 : 1;       // 16-byte activation loads per row and unit
  constexpr int kShift = kTern ? 10 : 8;   // operands enter as 16 * code (ternary weights 64 * code)
  constexpr int kFM = 2 * MB, kFN = 2 * NB;
  // [wave][sub-tile of the pass][32 rows][eight 16-byte chunks of columns]
  __shared__ v4i red[kW * P * 256];
  TileCoord tc;
  if (!tile_of_block(blockIdx.x, tiles_m, tiles_n, &tc)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = 32 * MB * tc.tm, n0 = 32 * NB * tc.tn;
  const int li = lane & 15, lg = lane >> 4;
  const uint32_t xrow = K / 2, wrow = kTern ? K / 4 : K / 2;  // packed row bytes
  const int T = static_cast<int>((wrow + 63) / 64);           // units: 64 bytes of a weight row

  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(qx), 0, static_cast<int>(static_cast<int64_t>(M) * xrow), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(qw), 0, static_cast<int>(static_cast<int64_t>(N) * wrow), kBufferFlags);
  // Lane group lg takes 16 bytes of each weight row of a unit, and the codes
  // they stand for of each activation row.  Rows past M or N and codes past
  // K read as zero (outside the buffers, without touching memory).
  uint32_t xo[kFM], wo[kFN];
#pragma unroll
  for (int f = 0; f < kFM; ++f) {
    const int r = m0 + 16 * f + li;
    xo[f] = r < M ? static_cast<uint32_t>(r) * xrow + 16 * kXL * lg : kOutsideOperand;
  }
#pragma unroll
  for (int f = 0; f < kFN; ++f) {
    const int r = n0 + 16 * f + li;
    wo[f] = r < N ? static_cast<uint32_t>(r) * wrow + 16 * lg : kOutsideOperand;
  }
  v4u w[2][kFN], x[2][kFM][kXL];
  auto issue = [&](auto D_, int i) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
    const int u = wave + kW * i;
    // K % 64 == 0: a lane's codes of a unit lie inside the row, or all past it
    const bool in = u < T && static_cast<uint32_t>(64 * u + 16 * lg) < wrow;
    const int so = u < T ? 64 * u : 0;
#pragma unroll
    for (int f = 0; f < kFN; ++f)
      w[d][f] = __builtin_bit_cast(
          v4u, __builtin_amdgcn_raw_buffer_load_b128(rw, in ? wo[f] : kOutsideOperand, so, 0));
#pragma unroll
    for (int f = 0; f < kFM; ++f)
#pragma unroll
      for (int p = 0; p < kXL; ++p)
        x[d][f][p] = __builtin_bit_cast(
            v4u, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? xo[f] + 16 * p : kOutsideOperand, so * kXL, 0));
  };
  v4i acc[kFN][kFM];
#pragma unroll
  for (int a = 0; a < kFN; ++a)
#pragma unroll
    for (int b = 0; b < kFM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
  auto compute = [&](auto D_) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
#pragma unroll
    for (int s = 0; s < 2 * kXL; ++s) {  // 16 codes per lane each
      v4i bx[kFM];
#pragma unroll
      for (int f = 0; f < kFM; ++f) {
        const v4u v = x[d][f][s / 2];
        const uint32_t p0 = (s & 1) ? v.z : v.x, p1 = (s & 1) ? v.w : v.y;
        bx[f] = kTern ? unpack8_tern_order(p0, p1) : unpack8(p0, p1);
      }
#pragma unroll
      for (int a = 0; a < kFN; ++a) {
        const v4u v = w[d][a];
        v4i aw;
        if constexpr (kTern) aw = unpack_tern(v[s]);
        else aw = s ? unpack8(v.z, v.w) : unpack8(v.x, v.y);
#pragma unroll
        for (int b = 0; b < kFM; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aw, bx[b], acc[a][b], 0, 0, 0);
      }
    }
  };
  // The scheduling barriers keep each unit's loads behind the MFMAs of the
  // unit before it, so that every wait leaves the newer unit in flight.
  const int iters = (T + kW - 1) / kW;
  const std::integral_constant<int, 0> c0{};
  const std::integral_constant<int, 1> c1{};
  issue(c0, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue(c1, 1);
  for (int i = 0; i < iters; i += 2) {
    __builtin_amdgcn_sched_barrier(0);
    compute(c0);
    __builtin_amdgcn_sched_barrier(0);
    issue(c0, i + 2);
    __builtin_amdgcn_sched_barrier(0);
    compute(c1);
    __builtin_amdgcn_sched_barrier(0);
    issue(c1, i + 3);
  }

  // Sum over the waves, P sub-tiles per pass.  A lane's results of MFMA tile
  // (a, b) are rows n = 16a + 4 lg + r of column m = 16b + li of y^T: chunk
  // 4a + lg of row m, at slot chunk ^ (m & 7), which spreads the eight lanes
  // of a 16-byte LDS access over all banks both ways.
  constexpr int kSubs = MB * NB;
#pragma unroll
  for (int p0 = 0; p0 < kSubs; p0 += P) {
    if (p0 > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < P; ++q) {
      if (p0 + q >= kSubs) break;
      const int sm = (p0 + q) / NB, sn = (p0 + q) % NB;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int m = 16 * b + li;
          red[((wave * P + q) * 32 + m) * 8 + ((4 * a + lg) ^ (m & 7))] = acc[2 * sn + a][2 * sm + b];
        }
    }
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < P * 256; e0 += 64 * kW) {
      const int e = e0 + tid;
      const int c = e & 7, q = (e >> 3) % P, m = (e >> 3) / P;
      if (p0 + q >= kSubs) continue;
      const int row = m0 + 32 * ((p0 + q) / NB) + m, n = n0 + 32 * ((p0 + q) % NB) + 4 * c;
      if (row >= M || n >= N) continue;
      const int slot = (q * 32 + m) * 8 + (c ^ (m & 7));
      v4i s = red[slot];
#pragma unroll
      for (int k = 1; k < kW; ++k) s += red[k * P * 256 + slot];
      const int64_t at = static_cast<int64_t>(row) * N + n;
      if constexpr (EPI == Epilogue::kInt32) {
        int32_t* p = static_cast<int32_t*>(out) + at;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < N) p[r] = s[r] >> kShift;
      } else {
        const float sxv = sx[row];
        uint16_t y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int nn = min(n + r, N - 1);
          float v = static_cast<float>(s[r] >> kShift);
          v = v * sxv;
          v = v * sw[nn];
          if (HAS_BIAS) v = v + __uint_as_float(static_cast<uint32_t>(bias[nn]) << 16);
          y[r] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
        }
        uint16_t* p = static_cast<uint16_t*>(out) + at;
        if (N % 4 == 0) {
          *reinterpret_cast<uint2*>(p) =
              make_uint2(y[0] | (static_cast<uint32_t>(y[1]) << 16), y[2] | (static_cast<uint32_t>(y[3]) << 16));
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n + r < N) p[r] = y[r];
        }
      }
    }
  }
}

// The tiles, with their blocks per CU and the time in ns a block spends
// outside its loop (900 more with ternary weights).
struct NarrowTile {
  int mb, nb, per_cu, fixed;
};
constexpr NarrowTile kTiles[] = {{1, 1, 4, 3600}, {2, 2, 2, 4700}, {2, 3, 2, 6300}};

}  // namespace

// Which tile, if any, an M x K by K x N product takes instead of the tiled
// kernel: 0 for none, else 1 + index into kTiles.  Estimates in ns from what
// the CU with the most tiles does (n of them): narrow, its bytes at 42 per
// ns and `fixed` per round of per_cu blocks; tiled, 6650 + 890 (950 ternary)
// per 128 codes for a block alone on its CU, 1550 for two, and never with
// more.  Fitted to 286 measured shapes (M 1..2048, K 256..12288, N
// 256..12288); a call changes over only where the estimate says at least 10%
// less; *ns is the estimate of the tile.
int gemm_narrow_tile(int64_t M, int64_t N, int64_t K, WeightFormat wf, int64_t cus, int64_t* ns) {
  const bool tern = wf == WeightFormat::kTernary;
  const int64_t units = (K + 127) / 128, mb = (M + 31) / 32, nb = (N + 31) / 32;
  const int64_t tiled_n = ((M + 127) / 128 * ((N + 255) / 256) + cus - 1) / cus;
  if (tiled_n > 2) return 0;
  const int64_t tiled = 6650 + units * (tiled_n == 2 ? 1550 : tern ? 950 : 890);
  int best = 0;
  int64_t best_ns = tiled * 90 / 100;
  int i = 0;
  for (const NarrowTile& t : kTiles) {
    ++i;
    const int64_t n = ((mb + t.mb - 1) / t.mb * ((nb + t.nb - 1) / t.nb) + cus - 1) / cus;
    const int64_t bytes = 2048 * t.mb + (tern ? 1024 : 2048) * t.nb;  // of a tile, per 128 codes
    const int64_t t_ns = n * units * bytes / 42 + (n + t.per_cu - 1) / t.per_cu * (t.fixed + (tern ? 900 : 0));
    if (t_ns < best_ns) best = i, best_ns = t_ns;
  }
  *ns = best_ns;
  return best;
}

void gemm_narrow_shape(int tile, int* rows, int* cols) {
  *rows = 32 * kTiles[tile - 1].mb;
  *cols = 32 * kTiles[tile - 1].nb;
}

hipError_t launch_gemm_narrow(int tile, Epilogue epi, const uint8_t* qx, const float* sx, int64_t M, int64_t K,
                              const uint8_t* qw, const float* sw, int64_t N, const uint16_t* bias, void* out,
                              hipStream_t st, WeightFormat wf) {
  const NarrowTile& t = kTiles[tile - 1];
  const int tiles_m = static_cast<int>((M + 32 * t.mb - 1) / (32 * t.mb));
  const int tiles_n = static_cast<int>((N + 32 * t.nb - 1) / (32 * t.nb));
  const unsigned blocks =
      static_cast<unsigned>((static_cast<int64_t>(tiles_m) * tiles_n + kNumXcd - 1) / kNumXcd * kNumXcd);
  const int Mi = static_cast<int>(M), Ki = static_cast<int>(K), Ni = static_cast<int>(N);
#define JQ_N(W, MB, NB, WPS, P, E, B)                                                                             \
  hipLaunchKernelGGL((gemm_narrow_kernel<W, MB, NB, WPS, P, E, B>), dim3(blocks), dim3(64 * kW), 0, st, qx, sx,   \
                     Mi, Ki, qw, sw, Ni, bias, out, tiles_m, tiles_n)
#define JQ_N_EPI(W, MB, NB, WPS, P)                                                  \
  if (epi == Epilogue::kInt32) JQ_N(W, MB, NB, WPS, P, Epilogue::kInt32, false);     \
  else if (bias != nullptr) JQ_N(W, MB, NB, WPS, P, Epilogue::kBf16, true);          \
  else JQ_N(W, MB, NB, WPS, P, Epilogue::kBf16, false);
#define JQ_N_TILE(W)                   \
  switch (tile) {                      \
    case 1: JQ_N_EPI(W, 1, 1, 4, 1) break; \
    case 2: JQ_N_EPI(W, 2, 2, 2, 2) break; \
    default: JQ_N_EPI(W, 2, 3, 2, 2) break; \
  }
  if (wf == WeightFormat::kTernary) {
    JQ_N_TILE(WeightFormat::kTernary)
  } else {
    JQ_N_TILE(WeightFormat::kInt4)
  }
#undef JQ_N_TILE
#undef JQ_N_EPI
#undef JQ_N
  return hipGetLastError();
}

}  // namespace jq
