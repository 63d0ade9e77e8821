// BF6 GEMM for products with few output tiles: a decoding block of a
// diffusion LLM (1 .. 128 tokens), a text stream of some hundred tokens, a
// narrow weight.  The same operands, exact sums and epilogue as the tiled
// kernel of f6.hip (see there for the layouts), and the same results bit for
// bit; launch_w4a4_f6_gemm picks it by f6_narrow_tile.
//
// What bounds such a product.  The tiled kernel gives a tile of 128 to 256
// rows x 256 columns to a block, so 64 x 12288 -> 4096 keeps 16 of 256 CUs
// busy, each walking all of K alone at one stage of 128 codes per 0.45 us
// (the latency of its loads, whatever M).  Here the tile is 32 or 64 rows x
// 32 .. 96 columns and the four waves of a block split K: wave w takes the
// 128-code units w, w + 4, ... of the whole tile, with no barrier and no LDS
// in the loop.  Partial sums are integers below 2^22 in fp32, so they add up
// exactly in any order.  They meet once, in LDS, where each thread sums four
// neighbouring outputs over the waves, applies the epilogue and stores them.
// A unit's fragments are whole consecutive 1 KiB lines in both layouts, read
// straight into registers two units ahead; two to four blocks share a CU.
// What is left is the rate at which a CU pulls operands from L2: 115 KB/us
// per CU (29 TB/s for the chip) over all tiles and shapes measured, i.e. the
// bytes of the CU that holds the most tiles.  Measured back to back on an
// MI355X, tiled -> narrow: 64 x 4096 -> 4096 15.4 -> 5.0 us, 64 x 12288 ->
// 4096 46.9 -> 9.7 us, 256 x 12288 -> 3072 46.6 -> 17.2 us, 512 x 12288 ->
// 3072 46.9 -> 21.6 us.

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

constexpr int kW = 4;  // waves of a block, splitting K
constexpr int kD = 2;  // units a wave loads ahead

// MB x NB bands of 32 activation rows x 32 columns per block; WPS waves (and
// so blocks) per SIMD; P output tiles of 32x32 meet in LDS per pass.
template <int MB, int NB, int WPS, int P, Epilogue EPI, bool HAS_BIAS>
__global__ __launch_bounds__(64 * kW, WPS) void f6_narrow_kernel(
    const uint8_t* __restrict__ xf6, const float* __restrict__ sx, int M, int mbands,
    const uint8_t* __restrict__ wf6, const float* __restrict__ sw, int N, int nbands, int ksteps,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n) {
  // [wave][output tile of the pass][32 rows][eight 16-byte chunks of columns]
  __shared__ v4f red[kW * P * 256];
  TileCoord tc;
  if (!tile_of_block(blockIdx.x, tiles_m, tiles_n, &tc)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mb0 = tc.tm * MB, nb0 = tc.tn * NB;
  const int T = ksteps / 2;  // units of 128 codes
  const uint32_t band_bytes = static_cast<uint32_t>(ksteps) * kFragBytes;

  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(xf6), 0, static_cast<int>(mbands * band_bytes), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(wf6), 0, static_cast<int>(nbands * band_bytes), kBufferFlags);
  // Per-lane offsets of a unit's parts.  Rows past M, bands past the operands
  // and units past K get an offset outside the buffer: they read as zero
  // without touching memory, so one row costs the loads of one row and the
  // loop needs no branch.
  uint32_t xo16[MB], xo8[MB], wo[NB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const bool live = 32 * (mb0 + b) + (lane & 31) < M;
    const uint32_t base = static_cast<uint32_t>(mb0 + b) * band_bytes;
    xo16[b] = live ? base + 16 * lane : kOutside;
    xo8[b] = live ? base + 1024 + 8 * lane : kOutside;
  }
#pragma unroll
  for (int f = 0; f < NB; ++f)
    wo[f] = nb0 + f < nbands ? static_cast<uint32_t>(nb0 + f) * band_bytes + 16 * lane : kOutside;

  v4i32 w[kD][NB][3];                       // weight layout: three 16-byte parts per band and unit
  v4i32 x16[kD][MB][2];                     // activation layout: 16 + 8 bytes per band and k-step
  v2i32 x8[kD][MB][2];
  auto issue = [&](auto D_, int i) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
    const int u = wave + kW * i;
    const bool in = u < T;
    const int so = in ? u * 2 * kFragBytes : 0;
#pragma unroll
    for (int f = 0; f < NB; ++f) {
      const uint32_t o = in ? wo[f] : kOutside;
#pragma unroll
      for (int p = 0; p < 3; ++p)
        w[d][f][p] = __builtin_bit_cast(v4i32, __builtin_amdgcn_raw_buffer_load_b128(rw, o + 1024 * p, so, 0));
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const uint32_t o16 = in ? xo16[b] : kOutside, o8 = in ? xo8[b] : kOutside;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        x16[d][b][s] =
            __builtin_bit_cast(v4i32, __builtin_amdgcn_raw_buffer_load_b128(rx, o16 + kFragBytes * s, so, 0));
        x8[d][b][s] = __builtin_bit_cast(v2i32, __builtin_amdgcn_raw_buffer_load_b64(rx, o8 + kFragBytes * s, so, 0));
      }
    }
  };

  v16f acc[NB][MB];
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[f][b] = v16f{};
  auto compute = [&](auto D_) __attribute__((always_inline)) {
    constexpr int d = decltype(D_)::value;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      v8i xb[MB];
#pragma unroll
      for (int b = 0; b < MB; ++b)
        xb[b] = v8i{x16[d][b][s].x, x16[d][b][s].y, x16[d][b][s].z, x16[d][b][s].w, x8[d][b][s].x, x8[d][b][s].y, 0, 0};
#pragma unroll
      for (int f = 0; f < NB; ++f) {
        const v8i a = s == 0 ? __builtin_shufflevector(w[d][f][0], w[d][f][1], 0, 1, 2, 3, 4, 5, -1, -1)
                             : __builtin_shufflevector(w[d][f][1], w[d][f][2], 2, 3, 4, 5, 6, 7, -1, -1);
#pragma unroll
        for (int b = 0; b < MB; ++b)
          acc[f][b] = mfma_bf6(a, xb[b], acc[f][b]);
      }
    }
  };
  // The scheduling barriers keep the loads of each unit behind the MFMAs of
  // the unit before it, in the prologue as in the loop, so that every wait
  // leaves the newer unit in flight.
  const int iters = (T + kW - 1) / kW;
  const std::integral_constant<int, 0> c0{};
  const std::integral_constant<int, 1> c1{};
  static_assert(kD == 2, "the loop is unrolled by two");
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

  // Sum over the waves, P output tiles per pass.  A lane's accumulators of a
  // tile are column m = lane & 31 and rows n = 8j + 4 (lane >> 5) + r of y^T:
  // chunk 2j + (lane >> 5) of row m, at slot chunk ^ (m & 7), which spreads
  // the eight lanes of a 16-byte LDS access over all banks both ways.
  constexpr int kTiles = MB * NB;
  const int h = lane >> 5, ml = lane & 31;
#pragma unroll
  for (int p0 = 0; p0 < kTiles; p0 += P) {
    if (p0 > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < P; ++q) {
      if (p0 + q >= kTiles) break;
      const v16f& a = acc[(p0 + q) % NB][(p0 + q) / NB];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        red[((wave * P + q) * 32 + ml) * 8 + ((2 * j + h) ^ (ml & 7))] =
            v4f{a[4 * j], a[4 * j + 1], a[4 * j + 2], a[4 * j + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < P * 256; e0 += 64 * kW) {
      const int e = e0 + tid;
      const int c = e & 7, q = (e >> 3) % P, m = (e >> 3) / P;
      if (p0 + q >= kTiles) continue;
      const int row = 32 * (mb0 + (p0 + q) / NB) + m, n = 32 * (nb0 + (p0 + q) % NB) + 4 * c;
      if (row >= M || n >= N) continue;
      const int slot = (q * 32 + m) * 8 + (c ^ (m & 7));
      v4f s = red[slot];
#pragma unroll
      for (int k = 1; k < kW; ++k) s += red[k * P * 256 + slot];
      const int64_t at = static_cast<int64_t>(row) * N + n;
      if constexpr (EPI == Epilogue::kInt32) {
        int32_t* p = static_cast<int32_t*>(out) + at;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < N) p[r] = static_cast<int32_t>(s[r]);
      } else {
        const float sxv = sx[row];
        uint16_t y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int nn = min(n + r, N - 1);
          float v = s[r] * sxv;
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
// outside its loop (launch, first loads, the sum over the waves, the stores).
struct NarrowTile {
  int mb, nb, per_cu, fixed;
};
constexpr NarrowTile kTiles[] = {{1, 1, 4, 3500}, {1, 2, 4, 4600}, {2, 2, 2, 4900}, {2, 3, 2, 6800}};

}  // namespace

// Which tile, if any, an M x K by K x N product takes instead of the tiled
// kernel: 0 for none, else 1 + index into kTiles.  The tiled kernel's time is
// f6_tile_bands' estimate; the narrow one's, in ns, follows from what the CU
// with the most tiles does (n = ceil(tiles / CUs)): its bytes at 115 per ns,
// plus `fixed` per round of per_cu blocks.  Fitted to 165 shapes (M 1..2048, K
// 256..12288, N 256..12288).  A call takes a narrow tile only where the
// estimate says at least 12% less, so that shapes near the line, and every
// large one, go to the tiled kernel: over 219 shapes (M 64..9216) the choice
// among all tiles of both kernels is within 0.9% of the best on average.
int f6_narrow_tile(int64_t M, int64_t N, int64_t K, int64_t cus) {
  const int64_t units = (K + 127) / 128, mb = (M + 31) / 32, nb = (N + 31) / 32;
  int64_t tiled = 0;
  f6_tile_bands(M, N, K, cus, &tiled);
  int best = 0;
  int64_t best_ns = tiled * 88 / 100;
  int i = 0;
  for (const NarrowTile& t : kTiles) {
    ++i;
    const int64_t n = ((mb + t.mb - 1) / t.mb * ((nb + t.nb - 1) / t.nb) + cus - 1) / cus;
    const int64_t ns = n * units * (t.mb + t.nb) * 2 * kFragBytes / 115 + (n + t.per_cu - 1) / t.per_cu * t.fixed;
    if (ns < best_ns) best = i, best_ns = ns;
  }
  return best;
}

void f6_narrow_shape(int tile, int* rows, int* cols) {
  *rows = 32 * kTiles[tile - 1].mb;
  *cols = 32 * kTiles[tile - 1].nb;
}

hipError_t launch_f6_narrow(int tile, Epilogue epi, const uint8_t* xf6, const float* sx, int64_t M, int64_t K,
                            const uint8_t* wf6, const float* sw, int64_t N, const uint16_t* bias, void* out,
                            hipStream_t st) {
  const NarrowTile& t = kTiles[tile - 1];
  const int ksteps = static_cast<int>(f6_ksteps(K));
  const int mbands = static_cast<int>((M + 31) / 32), nbands = static_cast<int>((N + 31) / 32);
  const int tiles_m = (mbands + t.mb - 1) / t.mb, tiles_n = (nbands + t.nb - 1) / t.nb;
  const unsigned blocks =
      static_cast<unsigned>((static_cast<int64_t>(tiles_m) * tiles_n + kNumXcd - 1) / kNumXcd * kNumXcd);
  const int Mi = static_cast<int>(M), Ni = static_cast<int>(N);
#define JQ_N(MB, NB, WPS, P, E, B)                                                                                 \
  hipLaunchKernelGGL((f6_narrow_kernel<MB, NB, WPS, P, E, B>), dim3(blocks), dim3(64 * kW), 0, st, xf6, sx, Mi,    \
                     mbands, wf6, sw, Ni, nbands, ksteps, bias, out, tiles_m, tiles_n)
#define JQ_N_EPI(MB, NB, WPS, P)                                                   \
  if (epi == Epilogue::kInt32) JQ_N(MB, NB, WPS, P, Epilogue::kInt32, false);      \
  else if (bias != nullptr) JQ_N(MB, NB, WPS, P, Epilogue::kBf16, true);           \
  else JQ_N(MB, NB, WPS, P, Epilogue::kBf16, false);
  switch (tile) {
    case 1: JQ_N_EPI(1, 1, 4, 1) break;
    case 2: JQ_N_EPI(1, 2, 4, 2) break;
    case 3: JQ_N_EPI(2, 2, 2, 2) break;
    default: JQ_N_EPI(2, 3, 2, 2) break;
  }
#undef JQ_N_EPI
#undef JQ_N
  return hipGetLastError();
}

}  // namespace jq
