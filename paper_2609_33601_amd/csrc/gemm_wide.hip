// Packed int4 (or ternary) weights x packed int4 activations on gfx950's 6-bit
// matrix cores, for products with many output tiles and long K: the same exact
// sums, epilogue and results, bit for bit, as the int8 kernel of gemm.hip;
// launch_w4a4_gemm picks it by gemm_wide_bands.
//
// Why 6 bits.  v_mfma_f32_32x32x64_f8f6f4 runs at twice the rate of the int8
// instructions, but its operands have to be made from packed codes inside the
// kernel.  E2M3 makes that cheap: its values 0 .. 15/8 are linear in their
// bits (subnormals, then the first binade), so a 4-bit number n, zero-extended
// to 6 bits, is n / 8.  Codes enter as n = code + 8 (the flipped sign bit of
// the packed nibble; ternary codes as code + 2), and spreading 16 nibbles at
// 4-bit pitch to 6-bit pitch takes eight vector instructions: the order of the
// codes within the 16 is free as long as both operands use the same one, and
// at 6-bit pitch every second field can stay in place while the others move by
// two bits.
//   P = sum n_x n_w / 64,  acc = 64 P - oW sum c_x - oX sum c_w - oX oW K'
// with oX = 8, oW = 8 (ternary 2) and K' the padded K.  All of these are
// integers below 2^24 (n_x n_w <= 225, K <= 65536, and 64 P only grows), so
// fp32 holds every partial sum exactly.  The sums of the codes are taken as
// they are converted (v_dot8_i32_i4 on the packed dword; bit counts for
// ternary codes).
//
// Structure.  Persistent blocks of four waves, one per CU and SIMD, on tiles of
// 32 NFM x 256 outputs (NFM = 6, 7, 8).  A step is 256 codes of K, 128 bytes of
// a row (64 of a ternary weight's), so that loads take whole lines.
//   * Activations: every thread loads one 16-byte chunk of each band of 32 rows
//     (eight threads to a row), two steps ahead; it spreads the chunk and
//     stores it to LDS as MFMA fragments, one step ahead, in one of two slots.
//   * Weights: wave w owns columns 64 w .. 64 w + 63; each lane loads its part
//     of a row one step ahead and spreads it one k-step ahead.
//   * The conversions go between the MFMAs, one (16 codes) after each pair or
//     two of MFMAs; one barrier per step, before its last k-step, makes the
//     next step's slot readable.
// Rows past M or N and chunks past the end of K get an offset outside the
// buffers (whatever the step's part of the address, which the range check
// leaves out) and read as zero; zero codes add nothing to acc whatever they meet.
//
// What bounds it.  Per step of a 256 x 256 tile a SIMD has 64 MFMAs (2048
// clocks) and about 600 other instructions to issue at 4.5 clocks each, one
// wave doing both.  Measured, int8 kernel -> this one: 4608 x 12288 -> 3072
// 122 -> 96 us (ternary weights 126 -> 103), 4608 x 3072 -> 9216 99 -> 87 (103
// -> 95), 3000 x 4096 -> 12288 126 -> 100.  Steps of 128 codes, whose loads take
// half lines, were 10% slower; with conversions to BF6 by v_cvt (59 issue slots
// per 32 codes instead of 16) it was no faster than int8.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "gemm_common.h"
#include "jq_internal.h"

namespace jq {

namespace {

using namespace gemm_detail;

typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v3i __attribute__((ext_vector_type(3)));
typedef unsigned v4u32 __attribute__((ext_vector_type(4)));
typedef unsigned v2u32 __attribute__((ext_vector_type(2)));

constexpr int kBN = 256;        // tile columns
constexpr int kWaves = 4;
constexpr int kStep = 256;      // codes of K per step
constexpr int kFrag = 1536;     // one 32-row x 64-code fragment
constexpr int kLgkm0 = 0xC07F;  // lgkmcnt(0), other counters untouched

// Every sum of products of offset codes (at most 15 * 15) is exact in fp32.
static_assert(15 * 15 * kMaxK < (int64_t(1) << 24), "a sum of products would not fit fp32");

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// 16 nibbles (p: eight, q: eight) to 16 E2M3 fields in 96 bits; FLIP: signed
// codes, offset by 8.  Fields 0 .. 15 are nibbles p0 p1 p3 p4 p6 p7 q1 q2 q4 q5
// q7 q0 p2 q3 p5 q6; p7 straddles the first two dwords.
template <bool FLIP>
__device__ __forceinline__ v3i spread6(uint32_t p, uint32_t q) {
  const uint32_t p2 = p << 2, q2 = __builtin_amdgcn_alignbit(q, p, 30);  // q << 2, p's top bits below
  auto mx = [](uint32_t a, uint32_t m, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, m, c, 0x6A); };  // (a & m) ^ c
  v3i r;
  r[0] = static_cast<int>(mx(p2, 0xC03C03C0u, mx(p, 0x0F00F00Fu, FLIP ? 0x08208208u : 0u)));
  r[1] = static_cast<int>(mx(q2, 0x03C03C03u, mx(q, 0xF00F00F0u, FLIP ? 0x82082082u : 0u)));
  r[2] = static_cast<int>(mx(q2, 0x3C03C03Cu, mx(p, 0x00F00F00u, FLIP ? 0x20820820u : 0u)));
  return r;
}
// Eight 2-bit codes (bytes B, B + 1 of w) to eight nibbles.
template <int B>
__device__ __forceinline__ uint32_t nibbles2(uint32_t w) {
  uint32_t x = __builtin_amdgcn_perm(w, w, B == 0 ? 0x0C010C00u : 0x0C030C02u);
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  return (x | (x << 2)) & 0x33333333u;
}

template <WeightFormat WF, int NFM, Epilogue EPI, bool HAS_BIAS, bool KTAIL>
__global__ __launch_bounds__(64 * kWaves, 1) void w4a4_wide_kernel(
    const uint8_t* __restrict__ qx, const float* __restrict__ sx, int M, int K,
    const uint8_t* __restrict__ qw, const float* __restrict__ sw, int N,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n, int grid_blocks) {
  constexpr bool kTern = WF == WeightFormat::kTernary;
  constexpr int kRows = 32 * NFM;
  constexpr uint32_t kSlot = NFM * 4 * kFrag;
  constexpr int kWL = kTern ? 2 : 4;  // weight loads per lane, band and step
  constexpr int oX = 8, oW = kTern ? 2 : 8;
  __shared__ __align__(16) uint8_t ring[2 * kSlot];
  __shared__ __align__(16) uint8_t stg[kWaves * 8192];  // output staging, two buffers of 32 rows x 64 bf16 per wave
  __shared__ float sc_x[kRows];
  __shared__ float sc_cx[kRows];              // oW sum c_x + oX oW K' of the tile's rows
  __shared__ __align__(16) float sc_w[kBN];
  __shared__ __align__(16) float sc_cw[kBN];  // oX sum c_w of its columns
  __shared__ __align__(16) uint16_t sc_b[kBN];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const uint32_t row_bytes = K / 2, wrow_bytes = kTern ? K / 4 : K / 2;
  const int T = (K + kStep - 1) / kStep;  // steps per tile, two or more
  const int last = T - 1;

  // As the int8 kernel's: virtual block ids of a grid of 8 * ceil(tiles / 8) in
  // the XCD-aware order.  (The loads run two steps ahead, at most into the next
  // tile: a tile has two steps or more.)
  int ntiles = 0;
  {
    const int vmax = (tiles_m * tiles_n + kNumXcd - 1) / kNumXcd * kNumXcd;
    TileCoord tc;
    for (int v = blockIdx.x; v < vmax && tile_of_block(v, tiles_m, tiles_n, &tc); v += grid_blocks) ++ntiles;
  }
  if (ntiles == 0) return;

  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(qx), 0, static_cast<int>(static_cast<int64_t>(M) * row_bytes), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rsw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(qw), 0, static_cast<int>(static_cast<int64_t>(N) * wrow_bytes), kBufferFlags);

  // Chunk c (32 codes) of a step belongs to k-step kstep(c), lane half half(c):
  // what a lane's 16 bytes of a weight row hold.
  const int xc = tid & 7, xr = tid >> 3;
  const int xk = kTern ? 2 * (xc >> 2) + (xc & 1) : xc >> 1, xh = kTern ? (xc >> 1) & 1 : xc & 1;
  struct Tile {
    int m0, n0;
    uint32_t x, w;  // per lane: byte offset of its first activation and weight row
  };
  auto tile_at = [&](int i) __attribute__((always_inline)) {
    TileCoord tc;
    tile_of_block(blockIdx.x + i * grid_blocks, tiles_m, tiles_n, &tc);
    Tile r;
    r.m0 = tc.tm * kRows;
    r.n0 = tc.tn * kBN;
    r.x = static_cast<uint32_t>(r.m0 + xr) * row_bytes + 16 * xc;
    r.w = static_cast<uint32_t>(r.n0 + 64 * wave + li) * wrow_bytes + 16 * lh;
    return r;
  };
  // XCD x walks K from step x T / 8 of it round to it, so that the XCDs read
  // different slices of the operands at any moment.
  auto next_k = [&](int ks) __attribute__((always_inline)) { return ks == last ? 0 : ks + 1; };

  uint4 gx[NFM];
  auto load_x = [&](uint32_t xo, int ks, int j) __attribute__((always_inline)) {
    uint32_t o = xo + static_cast<uint32_t>(32 * j) * row_bytes;
    if (KTAIL && static_cast<uint32_t>(128 * ks + 16 * xc) >= row_bytes) o = kOutsideOperand;
    gx[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsx, o, 128 * ks, 0));
  };
  int rs[NFM];
#pragma unroll
  for (int j = 0; j < NFM; ++j) rs[j] = 0;
  // Half h of band j's chunk to E2M3; the second half also stores the chunk as
  // its 24 bytes of a fragment.  Row r's place in the fragment is r ^ 2 c, which
  // spreads the eight chunks of a row over the LDS banks.
  v3i xg;
  uint8_t* const xf = ring + kFrag * xk;
  const int xl = (xr ^ (2 * xc)) + 32 * xh;
  auto conv_x = [&](uint32_t slot, int j, auto H) __attribute__((always_inline)) {
    constexpr int h = decltype(H)::value;
    const uint32_t p = h ? gx[j].z : gx[j].x, q = h ? gx[j].w : gx[j].y;
    rs[j] = __builtin_amdgcn_sdot8(static_cast<int>(p), 0x11111111, rs[j], false);
    rs[j] = __builtin_amdgcn_sdot8(static_cast<int>(q), 0x11111111, rs[j], false);
    const v3i g = spread6<true>(p, q);
    if constexpr (h == 0) {
      xg = g;
    } else {
      uint8_t* f = xf + 4 * kFrag * j;
      *reinterpret_cast<v4i*>(f + (slot + 16 * xl)) = v4i{xg[0], xg[1], xg[2], g[0]};
      *reinterpret_cast<v2u32*>(f + 1024 + (slot + 8 * xl)) =
          v2u32{static_cast<uint32_t>(g[1]), static_cast<uint32_t>(g[2])};
    }
  };
  auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NFM; ++j) {
      int v = rs[j];
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      v += __shfl_xor(v, 4, 64);
      if (xc == 0) sc_cx[32 * j + xr] = static_cast<float>(oW * v + oX * oW * kStep * T);
      rs[j] = 0;
    }
  };

  uint4 w[2][kWL];
  auto load_w = [&](uint32_t wo, int ks, int f, int q) __attribute__((always_inline)) {
    constexpr int kStep = kTern ? 64 : 128;
    uint32_t o = wo + static_cast<uint32_t>(32 * f) * wrow_bytes + 32 * q;
    if (KTAIL && static_cast<uint32_t>(kStep * ks + 16 * lh + 32 * q) >= wrow_bytes) o = kOutsideOperand;
    w[f][q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsw, o, kStep * ks, 0));
  };
  int cs[2] = {0, 0}, lead[2] = {0, 0};  // sums of the columns' codes; those of the next step's first k-step
  v8i aw[2][2];                          // [k-step parity][band]
  // Half h of the operand of band f, k-step s, and its codes' sum.
  auto conv_w = [&](auto F, auto S, auto H, int& sum) __attribute__((always_inline)) {
    constexpr int f = decltype(F)::value, s = decltype(S)::value, h = decltype(H)::value;
    v3i g;
    if constexpr (kTern) {
      const uint4 v = w[f][s / 2];
      const uint32_t x = (s & 1) ? (h ? v.w : v.z) : (h ? v.y : v.x);
      sum += __builtin_popcount(x & 0x55555555u) - 2 * __builtin_popcount(x & 0xAAAAAAAAu);
      const uint32_t n = x ^ 0xAAAAAAAAu;
      g = spread6<false>(nibbles2<0>(n), nibbles2<2>(n));
    } else {
      const uint32_t p = h ? w[f][s].z : w[f][s].x, q = h ? w[f][s].w : w[f][s].y;
      sum = __builtin_amdgcn_sdot8(static_cast<int>(p), 0x11111111, sum, false);
      sum = __builtin_amdgcn_sdot8(static_cast<int>(q), 0x11111111, sum, false);
      g = spread6<true>(p, q);
    }
    aw[s & 1][f][3 * h] = g[0];
    aw[s & 1][f][3 * h + 1] = g[1];
    aw[s & 1][f][3 * h + 2] = g[2];
  };
  auto read_b = [&](uint32_t slot, int s, int fm) __attribute__((always_inline)) {
    const uint8_t* p = ring + kFrag * (4 * fm + s);
    const int c = kTern ? 4 * (s >> 1) + 2 * lh + (s & 1) : 2 * s + lh;
    const int L = (li ^ (2 * c)) + 32 * lh;
    // (the 8-byte part as a relaxed atomic load: not paired with another's)
    const uint64_t hi = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p + 1024 + (slot + 8 * L)), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WAVEFRONT);
    const v4i lo = *reinterpret_cast<const v4i*>(p + (slot + 16 * L));
    return v8i{lo[0], lo[1], lo[2], lo[3], static_cast<int>(hi), static_cast<int>(hi >> 32), 0, 0};
  };

  v16f acc[2][NFM];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int fm = 0; fm < NFM; ++fm) acc[f][fm] = v16f{};

  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  Tile ct = tile_at(0), xt = ct;  // current and next tile
  if (ntiles > 1) xt = tile_at(1);
  const int k0 = static_cast<int>(blockIdx.x % kNumXcd) * T / kNumXcd;
  int k1 = next_k(k0), k2 = next_k(k1);  // the steps one and two ahead
  // Step 0's activations converted and its weights loaded, step 1's loading.
#pragma unroll
  for (int j = 0; j < NFM; ++j) load_x(ct.x, k0, j);
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int q = 0; q < kWL; ++q) load_w(ct.w, k0, f, q);
#pragma unroll
  for (int j = 0; j < NFM; ++j) {
    conv_x(0, j, C0{});
    conv_x(0, j, C1{});
    load_x(ct.x, k1, j);
  }
  static_for<2>([&](auto F) __attribute__((always_inline)) {
    constexpr int f = decltype(F)::value;
    conv_w(F, C0{}, C0{}, lead[f]);
    conv_w(F, C0{}, C1{}, lead[f]);
    if constexpr (!kTern) load_w(ct.w, k1, f, 0);
  });
  __builtin_amdgcn_s_waitcnt(kLgkm0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  uint32_t s0 = 0, s1 = kSlot;  // slots of this step and the next
  v8i bq[NFM];
#pragma unroll
  for (int fm = 0; fm < NFM; ++fm) bq[fm] = read_b(0, 0, fm);

  // Epilogue of the tile at (cm0, cn0): lane holds column m = cm0 + 32 fm +
  // (lane & 31) and rows n = cn0 + 64 wave + 32 f + 8 j + 4 (lane >> 5) + r of
  // y^T.  Bands go through LDS one at a time in two buffers and out as whole
  // 128-byte rows while the next is scaled.
  auto epilogue = [&](int cm0, int cn0) __attribute__((always_inline)) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // its addresses are computed here, not kept through the steps
    const int row = lane & 31, hl = lane >> 5;
    const int nl = 64 * wave + 4 * hl;
    const int mlim = min(M, cm0 + kRows);
    const bool full = (cm0 + kRows <= M) && (cn0 + kBN <= N);
    // each lane holds half of a column's sum; the wave's own columns
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const int v = cs[f] + __shfl_xor(cs[f], 32, 64);
      if (hl == 0) sc_cw[64 * wave + 32 * f + row] = static_cast<float>(oX * v);
      cs[f] = 0;
    }
    __builtin_amdgcn_wave_barrier();
    auto total = [&](int f, int fm, int j, int r, float cx, float cw) __attribute__((always_inline)) {
      return __builtin_fmaf(acc[f][fm][4 * j + r], 64.0f, -cx) - cw;  // both exact
    };
    if constexpr (EPI == Epilogue::kInt32) {
      int32_t* o = static_cast<int32_t*>(out);
#pragma unroll
      for (int fm = 0; fm < NFM; ++fm) {
        const int m = cm0 + row + 32 * fm;
        const float cx = sc_cx[32 * fm + row];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int c = nl + 32 * f + 8 * j, n = cn0 + c;
            const float4 cw = *reinterpret_cast<const float4*>(sc_cw + c);
            const int v0 = static_cast<int>(total(f, fm, j, 0, cx, cw.x)), v1 = static_cast<int>(total(f, fm, j, 1, cx, cw.y));
            const int v2 = static_cast<int>(total(f, fm, j, 2, cx, cw.z)), v3 = static_cast<int>(total(f, fm, j, 3, cx, cw.w));
            int32_t* p = o + static_cast<int64_t>(m) * N + n;
            if (full && N % 4 == 0) {
              *reinterpret_cast<int4*>(p) = make_int4(v0, v1, v2, v3);
            } else if (m < mlim) {
              if (n + 0 < N) p[0] = v0;
              if (n + 1 < N) p[1] = v1;
              if (n + 2 < N) p[2] = v2;
              if (n + 3 < N) p[3] = v3;
            }
          }
      }
    } else {
      uint16_t* o = static_cast<uint16_t*>(out);
      uint8_t* area = stg + 8192 * wave;
      auto put = [&](auto FM) __attribute__((always_inline)) {
        constexpr int fm = decltype(FM)::value;
        const float cx = sc_cx[32 * fm + row], sxv = sc_x[32 * fm + row];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int c = nl + 32 * f + 8 * j;
            const float4 s4 = *reinterpret_cast<const float4*>(sc_w + c), c4 = *reinterpret_cast<const float4*>(sc_cw + c);
            const float swa[4] = {s4.x, s4.y, s4.z, s4.w}, cwa[4] = {c4.x, c4.y, c4.z, c4.w};
            v2u32 b2 = {0, 0};
            if constexpr (HAS_BIAS) b2 = *reinterpret_cast<const v2u32*>(sc_b + c);
            uint16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float v = total(f, fm, j, r, cx, cwa[r]);
              v = v * sxv;
              v = v * swa[r];
              if constexpr (HAS_BIAS) v = v + __uint_as_float((r & 1) ? b2[r / 2] & 0xFFFF0000u : b2[r / 2] << 16);
              h[r] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
            }
            *reinterpret_cast<v2u32*>(area + 4096 * (fm & 1) + 128 * row + 16 * ((4 * f + j) ^ ((row >> 1) & 7)) +
                                      8 * hl) =
                v2u32{h[0] | (static_cast<uint32_t>(h[1]) << 16), h[2] | (static_cast<uint32_t>(h[3]) << 16)};
          }
      };
      // WHOLE: a whole tile with rows of a multiple of 16 bytes; otherwise rows
      // past M and columns past N are left out, element by element where
      // N % 8 != 0.
      auto bands = [&](auto WHOLE) __attribute__((always_inline)) {
        const int r0 = lane >> 3, c = lane & 7;
        const int n = cn0 + 64 * wave + 8 * c;
        uint16_t* p = o + static_cast<int64_t>(cm0 + r0) * N + n;
        const int mleft = n < N ? mlim - cm0 - r0 : 0;
        auto get = [&](int fm, int it) __attribute__((always_inline)) {
          return *reinterpret_cast<const v4u32*>(area + 4096 * (fm & 1) + 1024 * it + 128 * r0 +
                                                 16 * (c ^ ((4 * it + (r0 >> 1)) & 7)));
        };
        put(C0{});
        static_for<NFM>([&](auto FM) __attribute__((always_inline)) {
          constexpr int fm = decltype(FM)::value;
          __builtin_amdgcn_wave_barrier();
          if constexpr (decltype(WHOLE)::value) {
            v4u32 v[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) v[it] = get(fm, it);
            if constexpr (fm + 1 < NFM) put(std::integral_constant<int, fm + 1>{});
#pragma unroll
            for (int it = 0; it < 4; ++it) {
              __builtin_nontemporal_store(v[it], reinterpret_cast<v4u32*>(p));
              p += 8 * static_cast<int64_t>(N);
            }
          } else {
            if constexpr (fm + 1 < NFM) put(std::integral_constant<int, fm + 1>{});
#pragma unroll 1
            for (int it = 0; it < 4; ++it) {
              const v4u32 v = get(fm, it);
              if (32 * fm + 8 * it < mleft) {
                if (N % 8 == 0) {
                  __builtin_nontemporal_store(v, reinterpret_cast<v4u32*>(p));
                } else {
#pragma unroll
                  for (int e = 0; e < 8; ++e)
                    if (n + e < N) p[e] = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
                }
              }
              p += 8 * static_cast<int64_t>(N);
            }
          }
        });
        __builtin_amdgcn_wave_barrier();
      };
      if (full && N % 8 == 0) bands(std::true_type{});
      else bands(std::false_type{});
    }
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int fm = 0; fm < NFM; ++fm) acc[f][fm] = v16f{};
  };

  for (int ti = 0; ti < ntiles; ++ti) {
    for (int t = 0; t < T; ++t) {
      const uint32_t x2 = t + 2 < T ? ct.x : xt.x, w1 = t + 1 < T ? ct.w : xt.w, w2 = t + 2 < T ? ct.w : xt.w;
      // from here on the conversions are of the next tile's activations
      if (t == last) flush();
      cs[0] += lead[0], cs[1] += lead[1];
      lead[0] = lead[1] = 0;
      static_for<4>([&](auto S) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value;
        static_for<NFM>([&](auto FM) __attribute__((always_inline)) {
          constexpr int fm = decltype(FM)::value;
          acc[0][fm] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aw[s & 1][0], bq[fm], acc[0][fm], 2, 2, 0, 0, 0, 0);
          acc[1][fm] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aw[s & 1][1], bq[fm], acc[1][fm], 2, 2, 0, 0, 0, 0);
          if constexpr (s < 3) bq[fm] = read_b(s0, s + 1, fm);
          else bq[fm] = read_b(s1, 0, fm);
          // the next k-step's weights: four halves
          static_for<4>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value, f = q / 2, h = q % 2, n = (s + 1) % 4;
            if constexpr (q * NFM / 4 == fm) {
              using F = std::integral_constant<int, f>;
              using H = std::integral_constant<int, h>;
              conv_w(F{}, std::integral_constant<int, n>{}, H{}, n == 0 ? lead[f] : cs[f]);
              if constexpr (h == 1) {
                if constexpr (!kTern) load_w(n == 0 ? w2 : w1, n == 0 ? k2 : k1, f, n);
                else if constexpr (n & 1) load_w(w1, k1, f, n / 2);
              }
            }
          });
          // the next step's activations, in the first three k-steps
          static_for<2 * NFM>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            if constexpr (s < 3 && q * 3 / 2 == NFM * s + fm) {
              conv_x(s1, q / 2, std::integral_constant<int, q % 2>{});
              if constexpr (q % 2 == 1) load_x(x2, k2, q / 2);
            }
          });
          // Five vector instructions between the two MFMAs rather than all after
          // the second (4608 x 12288 -> 3072 at 8 bands 112 -> 103 us, at 7 97 ->
          // 96; ternary weights 104 -> 102.5 at 7, but 113 -> 115 at 8).
          if constexpr (!kTern || NFM < 8) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (s == 2) {
          // the next step's slot is whole, and this step's has been read
          __builtin_amdgcn_s_waitcnt(kLgkm0);
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
          if (EPI == Epilogue::kBf16 && t == 0) {
            // every wave is past the previous tile's epilogue
            if (tid < kRows) sc_x[tid] = sx[min(ct.m0 + tid, M - 1)];
            sc_w[tid] = sw[min(ct.n0 + tid, N - 1)];
            if constexpr (HAS_BIAS) sc_b[tid] = bias[min(ct.n0 + tid, N - 1)];
          }
        }
      });
      k1 = k2;
      k2 = next_k(k2);
      const uint32_t z = s0;
      s0 = s1, s1 = z;
    }
    epilogue(ct.m0, ct.n0);
    ct = xt;
    if (ti + 2 < ntiles) xt = tile_at(ti + 2);
  }
}

}  // namespace

// The tile height in bands of 32 rows (6, 7 or 8) with which a product takes
// this kernel, and the estimate it was picked by, or 0 for the int8 kernel.  A K
// of one step goes to the int8 kernel: here nothing runs under its loads (1147 x
// 192 -> 8960 13.4 us against 10.0, 1183 x 256 -> 8192 13.0 against 11.5; of 20
// such shapes ten were slower here by more than 2%, seven faster).  Both are
// estimated in ns for the XCD with most tiles, on its share of `cus`:
//   this kernel: its rounds, each 185 b + 299 per 256 codes (ternary 97 b + 936)
//   and 1545 b (1657 b) for the epilogue;
//   the int8 kernel: its rounds of two 128- or 112-row tiles per CU (a last
//   round of one per CU or fewer costs 0.67), 1190 per 128 codes and 10500 each.
// Fitted to 108 shapes per weight format (M 768..9216, K 512..12288, N
// 1024..12288).  The switch is where the estimate says 10% less: of 66 int4
// shapes that take it none is slower, the whole set is 10% faster on average
// (ternary 6.5%), and the best of all tiles would give 1.4% more.
int gemm_wide_bands(int64_t M, int64_t N, int64_t K, WeightFormat wf, int64_t cus, int64_t* ns) {
  if (K <= kStep) return 0;
  const bool tern = wf == WeightFormat::kTernary;
  const int64_t tiles_n = (N + kBN - 1) / kBN, xcd_cus = std::max<int64_t>(1, cus / kNumXcd);
  auto per_xcd = [&](int64_t rows) { return ((M + rows - 1) / rows * tiles_n + kNumXcd - 1) / kNumXcd; };
  int64_t best_ns = -1;
  for (const int64_t rows : {128, 112}) {
    const int64_t n = per_xcd(rows), rest = n % (2 * xcd_cus);
    const int64_t rounds = 100 * (n / (2 * xcd_cus)) + (rest == 0 ? 0 : rest <= xcd_cus ? 67 : 100);
    // 128 bits: a plan may be asked for sizes that no launch accepts
    const int64_t t = static_cast<int64_t>(static_cast<__int128>(rounds) * (rows == 128 ? 100 : 93) *
                                           (1190 * ((K + 127) / 128) + 10500) / 10000);
    if (best_ns < 0 || t < best_ns) best_ns = t;
  }
  best_ns = best_ns * 90 / 100;
  int best = 0;
  for (int b = 8; b >= 6; --b) {
    const int64_t t = (per_xcd(32 * b) + xcd_cus - 1) / xcd_cus *
                      ((K + kStep - 1) / kStep * (tern ? 97 * b + 936 : 185 * b + 299) + (tern ? 1657 : 1545) * b);
    if (t < best_ns) best = b, best_ns = t;
  }
  *ns = best_ns;
  return best;
}

hipError_t launch_gemm_wide(int bands, Epilogue epi, const uint8_t* qx, const float* sx, int64_t M, int64_t K,
                            const uint8_t* qw, const float* sw, int64_t N, const uint16_t* bias, void* out, int64_t cus,
                            hipStream_t st, WeightFormat wf) {
  const int tiles_m = static_cast<int>((M + 32 * bands - 1) / (32 * bands));
  const int tiles_n = static_cast<int>((N + kBN - 1) / kBN);
  const int64_t per_xcd = (static_cast<int64_t>(tiles_m) * tiles_n + kNumXcd - 1) / kNumXcd;
  const int blocks = static_cast<int>(std::min<int64_t>(per_xcd * kNumXcd, cus));
  const int Mi = static_cast<int>(M), Ki = static_cast<int>(K), Ni = static_cast<int>(N);
  const bool tail = K % kStep != 0;
#define JQ_W(W, NF, E, B, T)                                                                                      \
  hipLaunchKernelGGL((w4a4_wide_kernel<W, NF, E, B, T>), dim3(blocks), dim3(64 * kWaves), 0, st, qx, sx, Mi, Ki, qw, \
                     sw, Ni, bias, out, tiles_m, tiles_n, blocks)
#define JQ_W_EPI(W, NF)                                                 \
  if (epi == Epilogue::kInt32) {                                        \
    if (tail) JQ_W(W, NF, Epilogue::kInt32, false, true);               \
    else JQ_W(W, NF, Epilogue::kInt32, false, false);                   \
  } else if (bias != nullptr) {                                         \
    if (tail) JQ_W(W, NF, Epilogue::kBf16, true, true);                 \
    else JQ_W(W, NF, Epilogue::kBf16, true, false);                     \
  } else {                                                              \
    if (tail) JQ_W(W, NF, Epilogue::kBf16, false, true);                \
    else JQ_W(W, NF, Epilogue::kBf16, false, false);                    \
  }
#define JQ_W_ALL(W)                       \
  switch (bands) {                        \
    case 6: JQ_W_EPI(W, 6) break;         \
    case 7: JQ_W_EPI(W, 7) break;         \
    default: JQ_W_EPI(W, 8) break;        \
  }
  if (wf == WeightFormat::kTernary) {
    JQ_W_ALL(WeightFormat::kTernary)
  } else {
    JQ_W_ALL(WeightFormat::kInt4)
  }
#undef JQ_W_ALL
#undef JQ_W_EPI
#undef JQ_W
  return hipGetLastError();
}

}  // namespace jq
