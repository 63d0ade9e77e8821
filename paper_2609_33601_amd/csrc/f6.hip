// The W4A4 layer on gfx950's 6-bit matrix cores (v_mfma_f32_32x32x64_f8f6f4
// with BF6 = E3M2 operands), an exact alternative to the int8 MFMA path.
//
// Why it is exact.  Every int4 code -8..7 is a BF6 E3M2 value (|c| = 1.m * 2^e
// with two mantissa bits and e <= 3), so the matrix core multiplies the codes
// exactly.  Each product is an integer of magnitude <= 64 and every partial sum
// of a row of K <= 65536 products is an integer below 2^22, which fp32 holds
// exactly whatever the order of the additions.  The fp32 accumulator therefore
// equals the integer contraction acc[m,n] = sum_k qx[m,k] * qw[n,k], and the
// epilogue ((acc * s_x) * s_w) + bias sees the same operands as on the int8
// path.  Outputs are bit-identical to it.
//
// Why it is faster.  gfx950 issues the 6-bit MFMA at twice the int8 rate, and the
// operands reach it already encoded, so the loop holds no widening
// arithmetic at all:
//   * activations are quantised straight into BF6 by quantize_rows4_f6_kernel
//     (four rows per block) or quantize_rows_f6_kernel (longer rows), or the
//     kernel of f6_quant_few.hip (few rows), with
//     the same scale and codes as the packed-int4 quantiser;
//   * weights are converted once, offline, from the canonical packed int4
//     (or ternary) codes.
//
// The file also holds the group-wise form of the layer (one scale per G = 64
// or 128 codes): the same quantisers with group scales, and
// w4a4g_f6_gemm_kernel, which folds each group's exact product into fp32
// sums in k order.
//
// BF6 groups.  32 codes c[0..31] form a group of 192 bits, code p in bits
// 6p .. 6p+5 (six little-endian dwords d0..d5).  Rows are padded with zero
// codes to a multiple of 32 and taken in bands of 32; K is padded with zero
// codes to a multiple of 128 and cut into k-steps of 64 codes (KS of them, an
// even number).  Lane L = r + 32h of a v_mfma_*_32x32x64_f8f6f4 operand holds
// the group of codes 64s + 32h .. 64s + 32h + 31 of row r of the band for
// k-step s; A and B lanes use the same assignment, so the contraction is
// summed correctly.  Both operands take KS * 1536 bytes per band, band b at
// b * KS * 1536, in one of two orders within the band:
//   * activation layout (read by the GEMM through LDS): the fragment of
//     k-step s is 1536 bytes at s * 1536, lane L's d0..d3 at byte 16L and
//     d4, d5 at byte 1024 + 8L;
//   * weight layout (loaded by the GEMM straight into registers): k-steps 2u
//     and 2u + 1 share 3072 bytes at u * 3072, three planes of 1 KiB; lane L's
//     16 bytes of plane i are at 1024i + 16L, and its 48 bytes in plane order
//     are the six dwords of k-step 2u followed by those of k-step 2u + 1.
//     A wave thus loads two k-steps of a band with three 16-byte accesses per
//     lane (the vector memory path costs about the same per instruction
//     whatever its width).
//
// GEMM structure.  (Products with few output tiles go to f6_narrow.hip.)
// Persistent blocks of four waves walk the output tiles, 32 NFM rows x 256
// columns each, in an XCD-aware order.  Wave w owns weight bands 2w, 2w + 1 of
// the tile and all NFM activation bands: 2 x NFM tiles of 32x32.  f6_tile_bands
// picks, by the least estimated time,
//   * NFM = 5 .. 8 with one block per CU, one wave per SIMD and up to 256
//     accumulators per lane.  Each XCD's blocks walk K from stage x T / 8 of
//     it (XCD x) round to it, so that the eight XCDs read different slices of
//     the operands at any moment;
//   * NFM = 4 with two blocks per CU, which re-reads the operands more but
//     runs one block's epilogue beside the other's MFMAs.  So that the two
//     stay out of step, the blocks in the second half of each XCD's share
//     walk K from its middle stage round to it (the sum is exact in any
//     order).
// What bounds it.  A stage (128 codes of K) of a 256 x 256 tile is 32 MFMAs
// per SIMD, 1024 clocks, and 48 KiB of operands that pass the CU's vector
// memory path at 64 bytes per clock, 768 clocks.  With eight waves per block,
// four bands each, the two waves of a SIMD loaded the same weights twice (72
// KiB, 1152 clocks) and every wave had half the MFMAs to hide its other
// instructions under: 4096 x 12288 -> 4096 85 -> 76 us, 9216 x 12288 -> 3072
// 153 -> 131 us (codes of a heavy-tailed activation, back to back; both sides of
// every pair here in one run).  One wave per SIMD allows four tile heights, since
// no second wave has to have the same work: in 192-row tiles 6000 x 12288 ->
// 4096 152 -> 119 us and 3000 x 4096 -> 4096 34 -> 25 us.
// The rest is the stages' own stalls and what a tile costs beside its stages,
// 8.6 us at NFM = 8 by the fit of f6_tile_bands (the first loads, the epilogue
// and its stores); about 4 us of it are the epilogue's vector arithmetic (two
// multiplies and half a conversion per output, 256 outputs a lane) with only one
// wave per SIMD to run it.
//   * Activations: shared by the four waves, staged through LDS.  A stage is
//     3 KiB per band, consecutive in memory, moved by buffer_load ... lds (no
//     registers) into a ring of three stage slots, three stages ahead.
//   * Weights: loaded straight into registers one stage ahead, two register
//     sets (so the stage loop is unrolled by two; a tile with an odd number
//     of stages moves the loaded set over at its end).
//   * Per stage: the MFMAs of k-step 0 run while the wave reads its k-step 1
//     fragments from LDS and issues the next stage's weight loads, one after
//     each of the first fragments' MFMAs; then it waits for its share of the
//     next stage's DMA and meets the others at a barrier (no memory fence);
//     then the MFMAs of k-step 1 run while the next stage's k-step 0
//     fragments are read and the DMA three stages ahead goes into the slot
//     just read.  Issued in one burst, the same loads queue up behind each
//     other and hold the MFMAs back.  No arithmetic on vectors sits between
//     the MFMAs, and every address is scalar.
//   * Every vector-memory instruction of the stage loop (the weight loads
//     and the buffer -> LDS transfers) is issued as an instruction of its
//     own, and the loop orders it with explicit waits only (see the stage).
//     Left to the compiler, the transfers made it wait for every DMA in
//     flight before each LDS read.  The compiler does not know that these
//     loads complete after they issue, so the loaded registers pass through
//     an empty asm after their wait before any use, and the build checks the
//     generated code: no instruction may touch a load's registers before a
//     wait retires it (check_waits.py).  The file is also built without
//     machine sinking, which otherwise moved the first k-step's MFMAs below
//     the stage's barrier.
//   * The matrix instruction is the one without scales (mfma_bf6): with them
//     it is 2-4% slower in this loop.
//   * An activation fragment's 16- and 8-byte parts land next to each other
//     in registers (the 8-byte part read on its own, not paired with another
//     fragment's), and a band's three 16-byte weight parts of a stage are
//     the two k-steps' operands as two overlapping 6-dword windows.
//   * The weight fragment is operand A and the activation fragment operand B,
//     so the 32x32 result is y^T: lane L holds column m = L % 32 and rows
//     n = 8j + 4(L / 32) + r (j, r = 0..3).  The epilogue scales them, packs
//     bf16 and stages them through LDS to store whole 128-byte rows.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>

#include "f6_common.h"
#include "gemm_common.h"
#include "jq.h"
#include "jq_internal.h"

namespace jq {

namespace {

using namespace gemm_detail;
using namespace f6_detail;

typedef float v16f32 __attribute__((ext_vector_type(16)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h32 __attribute__((ext_vector_type(32)));
typedef unsigned v4u32 __attribute__((ext_vector_type(4)));

constexpr int kFBN = 256;    // block tile columns of the GEMM
constexpr int kF6Waves = 4;  // waves of a GEMM block
constexpr int kWLoads = 6;   // weight loads per wave and stage

// 32 codes (as exact fp32 integers, code p in q[p]) -> six dwords, code p in bits 6p..6p+5.
// The converter interleaves its two sources (field 2i <- src0[i], field 2i+1 <- src1[i]).
__device__ __forceinline__ v6u bf6_group(const float* q) {
  v16f32 ev, od;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    ev[i] = q[2 * i];
    od[i] = q[2 * i + 1];
  }
  return __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(ev, od, 1.0f);
}

// Codes of one 32-element group (16 dwords of bf16 pairs).  Reciprocal path
// with the exact IEEE division wherever the product sits next to a rounding
// decision point (the argument is that of the packed-int4 quantiser), or the
// division for every element when the reciprocal overflows.
__device__ __forceinline__ void codes32(const uint32_t* w, float s, float rcp, bool exact_row, float* q) {
  bool near = exact_row;
  if (!exact_row) {
    float dmax = 0.0f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float te = bf16_lo(w[j]) * rcp;
      const float to = bf16_hi(w[j]) * rcp;
      const float re = (te + kMagic) - kMagic;
      const float ro = (to + kMagic) - kMagic;
      dmax = fmaxf(dmax, fmaxf(fabsf(te - re), fabsf(to - ro)));
      q[2 * j] = re;
      q[2 * j + 1] = ro;
    }
    near = !(dmax < kNearTie);
  }
  if (near) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      q[2 * j] = fminf(fmaxf(__builtin_rintf(bf16_lo(w[j]) / s), -8.0f), 7.0f);
      q[2 * j + 1] = fminf(fmaxf(__builtin_rintf(bf16_hi(w[j]) / s), -8.0f), 7.0f);
    }
  }
}

// Store the BF6 group gi (= 2 * kstep + half) of row `row` into the activation layout.
__device__ __forceinline__ void store_group(uint8_t* out, int64_t ksteps, int64_t row, int gi, v6u d) {
  const int L = static_cast<int>(row & 31) + 32 * (gi & 1);
  uint8_t* p = out + ((row >> 5) * ksteps + (gi >> 1)) * kFragBytes;
  *reinterpret_cast<uint4*>(p + 16 * L) = make_uint4(d[0], d[1], d[2], d[3]);
  *reinterpret_cast<uint2*>(p + 1024 + 8 * L) = make_uint2(d[4], d[5]);
}

// Row of block b.  Blocks are dealt round-robin to the 8 XCDs; the 32 rows of
// a band all go to the blocks of one XCD, so the partial cache lines of a
// fragment are completed in one L2 before they are written back.
__device__ __forceinline__ int64_t row_of_block(int64_t b) {
  const int64_t x = b % kNumXcd, j = b / kNumXcd;
  return 32 * (kNumXcd * (j / 32) + x) + (j % 32);
}

// Per-token quantiser writing the BF6 operand.  One block per row of the
// padded operand; thread i handles groups i + T j (j < NJ) of 32 codes and
// keeps them in registers between the absmax and the quantisation.  A wave
// reads its 64 groups (4 KiB) as four 1 KiB loads of whole cache lines and
// hands each lane its own 64 bytes through LDS (the 16-byte chunk q of the
// wave's 256 at slot q ^ ((q >> 4) & 15), so that neither the writes nor the
// reads conflict).  The loads are non-temporal: the input is read once, and
// left to the caches it would evict the operands of the GEMM that follows.
// The scale and the codes are those of quantize_rows_kernel.  Padding rows
// (M <= row < 32 * ceil(M/32)) get zero codes and no scale.
//
// G = 64 or 128: one scale per G consecutive codes instead (scale [M, K/G]
// row-major, the codes and scales of quantize_groups_kernel).  A group is the
// 32-code groups of G/32 neighbouring lanes, which meet with shuffles.
template <int NJ, int G>
__global__ __launch_bounds__(512) void quantize_rows_f6_kernel(const uint16_t* __restrict__ x, int64_t M, int64_t K,
                                                               int64_t rows_padded, int64_t ksteps,
                                                               uint8_t* __restrict__ out, float* __restrict__ scale) {
  __shared__ uint32_t wave_max[8];
  const int T = blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = T >> 6;
  const int64_t row = row_of_block(blockIdx.x);
  if (row >= rows_padded) return;
  const bool live = row < M;
  const int groups = static_cast<int>(2 * ksteps);
  const uint16_t* xr = x + (live ? row : 0) * K;

  extern __shared__ v4u32 xt[];  // 256 chunks of 16 bytes per wave
  v4u32* xw = xt + 256 * wave;
  auto swz = [](int q) { return q ^ ((q >> 4) & 15); };
  uint4 v[NJ][4];
  u16x2 am = {0, 0};
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int64_t base = 32 * static_cast<int64_t>(T * j + 64 * wave);
    v4u32 t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // Out-of-range chunks (K padding, padding rows) load the first chunk
      // of x and are zeroed; no branch, so the four loads issue together.
      const int64_t e = base + 512 * c + 8 * lane;
      const bool ok = live && e < K;
      t[c] = __builtin_nontemporal_load(reinterpret_cast<const v4u32*>(ok ? xr + e : x));
      if (!ok) t[c] = v4u32{0, 0, 0, 0};
      am = __builtin_elementwise_max(am, __builtin_bit_cast(u16x2, t[c].x & 0x7FFF7FFFu));
      am = __builtin_elementwise_max(am, __builtin_bit_cast(u16x2, t[c].y & 0x7FFF7FFFu));
      am = __builtin_elementwise_max(am, __builtin_bit_cast(u16x2, t[c].z & 0x7FFF7FFFu));
      am = __builtin_elementwise_max(am, __builtin_bit_cast(u16x2, t[c].w & 0x7FFF7FFFu));
    }
    // Only this wave touches its chunks, and LDS runs a wave's accesses in
    // order: the fences just keep the compiler from moving them.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < 4; ++c) xw[swz(64 * c + lane)] = t[c];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const v4u32 r = xw[swz(4 * lane + c)];
      v[j][c] = make_uint4(r.x, r.y, r.z, r.w);
    }
  }
  if constexpr (G != 0) {
    (void)am;
    (void)wave_max;
    constexpr int kLanes = G / 32;  // lanes per group
    const int64_t KG = K / G;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      u16x2 gm = {0, 0};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].x & 0x7FFF7FFFu));
        gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].y & 0x7FFF7FFFu));
        gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].z & 0x7FFF7FFFu));
        gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].w & 0x7FFF7FFFu));
      }
      uint32_t gmax = gm.x > gm.y ? gm.x : gm.y;
#pragma unroll
      for (int off = 1; off < kLanes; off <<= 1) {
        const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(gmax), off, 64));
        gmax = gmax > o ? gmax : o;
      }
      const int gi = threadIdx.x + T * j;
      if (gi >= groups) continue;
      const float sg = __uint_as_float(gmax << 16) / 7.0f;
      if (live && gi % kLanes == 0 && 32 * static_cast<int64_t>(gi) < K) scale[row * KG + gi / kLanes] = sg;
      const float rcp = (sg == 0.0f) ? 0.0f : 1.0f / sg;
      float q[32];
      if (sg == 0.0f) {
#pragma unroll
        for (int p = 0; p < 32; ++p) q[p] = 0.0f;
      } else {
        const uint32_t w[16] = {v[j][0].x, v[j][0].y, v[j][0].z, v[j][0].w, v[j][1].x, v[j][1].y,
                                v[j][1].z, v[j][1].w, v[j][2].x, v[j][2].y, v[j][2].z, v[j][2].w,
                                v[j][3].x, v[j][3].y, v[j][3].z, v[j][3].w};
        codes32(w, sg, rcp, __builtin_isinf(rcp), q);
      }
      store_group(out, ksteps, row, gi, bf6_group(q));
    }
    return;
  }
  uint32_t amax = am.x > am.y ? am.x : am.y;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(amax), off, 64));
    amax = amax > o ? amax : o;
  }
  if (nwaves > 1) {
    if (lane == 0) wave_max[wave] = amax;
    __syncthreads();
    amax = wave_max[0];
    for (int w = 1; w < nwaves; ++w) amax = amax > wave_max[w] ? amax : wave_max[w];
  }
  // Non-negative floats order like their bit patterns.
  const float a = __uint_as_float(amax << 16);
  const float s = a / 7.0f;
  if (live && threadIdx.x == 0) scale[row] = s;
  const float rcp = (s == 0.0f) ? 0.0f : 1.0f / s;
  const bool exact_row = __builtin_isinf(rcp);

#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int gi = threadIdx.x + T * j;
    if (gi >= groups) continue;
    float q[32];
    if (s == 0.0f) {
#pragma unroll
      for (int p = 0; p < 32; ++p) q[p] = 0.0f;
    } else {
      const uint32_t w[16] = {v[j][0].x, v[j][0].y, v[j][0].z, v[j][0].w, v[j][1].x, v[j][1].y,
                              v[j][1].z, v[j][1].w, v[j][2].x, v[j][2].y, v[j][2].z, v[j][2].w,
                              v[j][3].x, v[j][3].y, v[j][3].z, v[j][3].w};
      codes32(w, s, rcp, exact_row, q);
    }
    store_group(out, ksteps, row, gi, bf6_group(q));
  }
}

// First row of block b in the four-rows-per-block quantiser: the eight
// blocks of a band are consecutive blocks of one XCD, so the lines of a
// fragment that they write piecewise meet in one L2.
__device__ __forceinline__ int64_t row0_of_block4(int64_t b) {
  const int64_t x = b % kNumXcd, j = b / kNumXcd;
  return 32 * (kNumXcd * (j / 8) + x) + 4 * (j % 8);
}

// The same quantiser for rows of up to 512 groups (K <= 16384), four rows
// per block: lane l of a wave takes row l % 4 and group slot l / 4, so that
// the four lanes of a group slot store the same fragment piece of four
// consecutive rows, 64 (and 32) contiguous bytes, instead of four scattered
// 16- and 8-byte pieces.  Wave w's j-th set of groups is the 16 groups from
// 16 (W j + w) in each of the four rows: four 1 KiB loads of whole lines (one
// per row), regrouped per lane through LDS (chunk q = 64 row + 4 slot +
// quarter at slot q ^ ((q >> 6) & 3): conflict-free both ways).  Per-row
// maxima meet by shuffles within a wave and through LDS across waves; group
// maxima (G = 64, 128) by shuffles between the lanes of a group.  The scales
// and codes are those of quantize_rows_f6_kernel.
//
// The body is shared with the batched form (several inputs in one launch):
// block b of the input, and nj <= NJ sets of groups per wave (the rest of the
// register arrays idle).
template <int NJ, int G>
__device__ __forceinline__ void q4_rows(const uint16_t* __restrict__ x, int64_t M, int64_t K, int64_t rows_padded,
                                        int64_t ksteps, uint8_t* __restrict__ out, float* __restrict__ scale,
                                        int64_t b, int nj) {
  __shared__ uint32_t wave_max[8][4];
  const int T = blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = T >> 6;
  const int64_t row0 = row0_of_block4(b);
  if (row0 >= rows_padded) return;
  const int rr = lane & 3, gslot = lane >> 2;
  const int64_t row = row0 + rr;
  const bool live = row < M;
  const int groups = static_cast<int>(2 * ksteps);

  extern __shared__ v4u32 xt[];  // 256 chunks of 16 bytes per wave
  v4u32* xw = xt + 256 * wave;
  auto swz = [](int q) { return q ^ ((q >> 6) & 3); };
  // All loads first (NJ x 4 of them in flight), then the regrouping.
  v4u32 t[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j >= nj) break;
    const int g0 = 16 * (nwaves * j + wave);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // row row0 + c, elements 32 g0 + 8 lane .. + 7; out-of-range chunks load
      // the first chunk of x and are zeroed (no branch between the loads)
      const int64_t e = 32 * static_cast<int64_t>(g0) + 8 * lane;
      const bool ok = row0 + c < M && e < K;
      t[j][c] = __builtin_nontemporal_load(reinterpret_cast<const v4u32*>(ok ? x + (row0 + c) * K + e : x));
      if (!ok) t[j][c] = v4u32{0, 0, 0, 0};
    }
  }
  uint4 v[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j >= nj) break;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < 4; ++c) xw[swz(64 * c + lane)] = t[j][c];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const v4u32 r = xw[swz(64 * rr + 4 * gslot + c)];
      v[j][c] = make_uint4(r.x, r.y, r.z, r.w);
    }
  }
  // The lane's maximum over each of its groups.
  uint32_t gmax[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) gmax[j] = 0;  // sets past nj stay 0
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j >= nj) break;
    u16x2 gm = {0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].x & 0x7FFF7FFFu));
      gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].y & 0x7FFF7FFFu));
      gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].z & 0x7FFF7FFFu));
      gm = __builtin_elementwise_max(gm, __builtin_bit_cast(u16x2, v[j][c].w & 0x7FFF7FFFu));
    }
    gmax[j] = gm.x > gm.y ? gm.x : gm.y;
  }
  float srow = 0.0f;
  if constexpr (G == 0) {
    uint32_t amax = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) amax = amax > gmax[j] ? amax : gmax[j];
#pragma unroll
    for (int off = 4; off <= 32; off <<= 1) {  // the 16 lanes of this row
      const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(amax), off, 64));
      amax = amax > o ? amax : o;
    }
    if (nwaves > 1) {
      if (gslot == 0) wave_max[wave][rr] = amax;
      __syncthreads();
      amax = wave_max[0][rr];
      for (int w = 1; w < nwaves; ++w) amax = amax > wave_max[w][rr] ? amax : wave_max[w][rr];
    }
    srow = __uint_as_float(amax << 16) / 7.0f;
    if (live && wave == 0 && gslot == 0) scale[row] = srow;
  } else {
    (void)wave_max;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j >= nj) break;
    float s = srow;
    if constexpr (G != 0) {
      constexpr int kLanes = G / 32;  // group slots per group, 4 lanes apart
      uint32_t gm = gmax[j];
#pragma unroll
      for (int off = 4; off < 4 * kLanes; off <<= 1) {
        const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(gm), off, 64));
        gm = gm > o ? gm : o;
      }
      s = __uint_as_float(gm << 16) / 7.0f;
    }
    const int gi = 16 * (nwaves * j + wave) + gslot;
    if (gi >= groups) continue;
    if constexpr (G != 0) {
      constexpr int kLanes = G / 32;
      if (live && gi % kLanes == 0 && 32 * static_cast<int64_t>(gi) < K) scale[row * (K / G) + gi / kLanes] = s;
    }
    const float rcp = (s == 0.0f) ? 0.0f : 1.0f / s;
    float q[32];
    if (s == 0.0f) {
#pragma unroll
      for (int p = 0; p < 32; ++p) q[p] = 0.0f;
    } else {
      const uint32_t w[16] = {v[j][0].x, v[j][0].y, v[j][0].z, v[j][0].w, v[j][1].x, v[j][1].y,
                              v[j][1].z, v[j][1].w, v[j][2].x, v[j][2].y, v[j][2].z, v[j][2].w,
                              v[j][3].x, v[j][3].y, v[j][3].z, v[j][3].w};
      codes32(w, s, rcp, __builtin_isinf(rcp), q);
    }
    store_group(out, ksteps, row, gi, bf6_group(q));
  }
}

template <int NJ, int G>
__global__ __launch_bounds__(512) void quantize_rows4_f6_kernel(const uint16_t* __restrict__ x, int64_t M, int64_t K,
                                                                int64_t rows_padded, int64_t ksteps,
                                                                uint8_t* __restrict__ out, float* __restrict__ scale) {
  q4_rows<NJ, G>(x, M, K, rows_padded, ksteps, out, scale, blockIdx.x, NJ);
}

// Several independent inputs quantised per token in one launch (rows of up
// to 512 groups each): input i takes the blocks from first[i] on, a multiple
// of 64 so that each band's blocks stay on one XCD, and runs with nj[i] of
// the NJ sets of groups per wave.  Each input's codes and scales are those
// of its own launch of quantize_rows4_f6_kernel.
struct Q4Input {
  const uint16_t* x;
  uint8_t* out;
  float* scale;
  int64_t M, K, rows_padded, ksteps, first;
  int nj;
};
struct Q4Batch {
  Q4Input in[kQuantBatchMax];
  int count;
};

template <int NJ>
__global__ __launch_bounds__(512) void quantize_rows4_f6_batch_kernel(Q4Batch b) {
  int i = 0;
  while (i + 1 < b.count && static_cast<int64_t>(blockIdx.x) >= b.in[i + 1].first) ++i;
  const Q4Input& e = b.in[i];
  q4_rows<NJ, 0>(e.x, e.M, e.K, e.rows_padded, e.ksteps, e.out, e.scale, blockIdx.x - e.first, e.nj);
}

// Canonical packed int4 codes (TERNARY false) or packed ternary codes (true)
// -> BF6 operand in the activation or the weight layout.  A wave takes
// kCvtUnits units of 128 codes of one band: lane L = r + 32h reads its two
// groups of a unit (codes 64s + 32h .. of row r, s = 0, 1) and stores them
// where they belong, so that every store instruction of a wave is a whole
// consecutive KiB (or 512 bytes).  Padding rows and codes are written as
// zeros.  Bound by memory: one thread per group, in row order, scattered its
// 16- and 8-byte stores over 64 lines each (12288 x 4096 int4 -> weight
// layout 31 us; now 11.3 us, 5.6 TB/s read + write).
constexpr int kCvtUnits = 4;

// Eight int4 codes (a dword, two's complement, code 2j in the low nibble of
// byte j) as f16 pairs: with the sign bits flipped a nibble is code + 8, and
// placed in the mantissa of 1024 (the high nibble of a byte 16 times larger)
// one multiply-add per pair brings it to the code, exactly.
__device__ __forceinline__ void codes8_f16(uint32_t p, h2* q) {
  p ^= 0x88888888u;
  const h2 mul = {1.0f, 0.0625f}, add = {-1032.0f, -72.0f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t b = __builtin_amdgcn_perm(0, p, 0x0C000C00u | (j << 16) | j);  // byte j in both halves
    q[j] = __builtin_elementwise_fma(__builtin_bit_cast(h2, (b & 0x00F0000Fu) | 0x64006400u), mul, add);
  }
}

template <bool WLAYOUT, bool TERNARY>
__global__ __launch_bounds__(256) void int4_to_f6_kernel(const uint8_t* __restrict__ q, int64_t rows, int64_t K,
                                                         int64_t bands, int64_t ksteps, uint8_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int64_t units = ksteps / 2, per_band = (units + kCvtUnits - 1) / kCvtUnits;
  const int64_t wv = static_cast<int64_t>(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t band = wv / per_band, u0 = wv % per_band * kCvtUnits;
  if (band >= bands) return;
  const int64_t row = 32 * band + r;
  const uint8_t* qr = q + row * (TERNARY ? K / 4 : K / 2);
  typedef typename std::conditional<TERNARY, uint2, uint4>::type packed;  // 32 codes
  packed v[kCvtUnits][2];
#pragma unroll
  for (int i = 0; i < kCvtUnits; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int64_t k = 128 * (u0 + i) + 64 * s + 32 * h;
      v[i][s] = packed{};
      if (row < rows && k < K) v[i][s] = *reinterpret_cast<const packed*>(qr + (TERNARY ? k / 4 : k / 2));
    }
#pragma unroll
  for (int i = 0; i < kCvtUnits; ++i) {
    if (u0 + i >= units) break;
    v6u d[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if constexpr (TERNARY) {
        const uint32_t w[2] = {v[i][s].x, v[i][s].y};
        float c[32];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int n = 0; n < 16; ++n)  // 2-bit field n of dword t is code 16t + n
            c[16 * t + n] = static_cast<float>(static_cast<int>(w[t] << (30 - 2 * n)) >> 30);
        d[s] = bf6_group(c);
      } else {
        const uint32_t w[4] = {v[i][s].x, v[i][s].y, v[i][s].z, v[i][s].w};
        h2 c[16];
#pragma unroll
        for (int t = 0; t < 4; ++t) codes8_f16(w[t], c + 4 * t);
        h32 all;
#pragma unroll
        for (int n = 0; n < 16; ++n) {
          all[2 * n] = c[n].x;
          all[2 * n + 1] = c[n].y;
        }
        d[s] = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(all, 1.0f);
      }
    }
    uint8_t* p = out + (band * units + u0 + i) * (2 * kFragBytes);
    if constexpr (WLAYOUT) {
      uint4* o = reinterpret_cast<uint4*>(p) + lane;
      o[0] = make_uint4(d[0][0], d[0][1], d[0][2], d[0][3]);
      o[64] = make_uint4(d[0][4], d[0][5], d[1][0], d[1][1]);
      o[128] = make_uint4(d[1][2], d[1][3], d[1][4], d[1][5]);
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        *reinterpret_cast<uint4*>(p + s * kFragBytes + 16 * lane) = make_uint4(d[s][0], d[s][1], d[s][2], d[s][3]);
        *reinterpret_cast<uint2*>(p + s * kFragBytes + 1024 + 8 * lane) = make_uint2(d[s][4], d[s][5]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// GEMM

typedef unsigned v2u32 __attribute__((ext_vector_type(2)));

struct WFrag {
  v8i f[2][2];  // [k-step][band]; dwords 0..5 used
};
// A wave's weights of one stage as loaded: three 16-byte parts per band
// (the six dwords of k-step 0, then those of k-step 1), turned into MFMA
// operands only once the stage's wait has passed.
struct WRaw {
  v4i32 p[2][3];  // [band][part]
};

__device__ __forceinline__ v8i join(v4i32 a, v2i32 b) { return v8i{a.x, a.y, a.z, a.w, b.x, b.y, 0, 0}; }

// f(integral_constant<int, i>) for i = 0 .. N - 1, in order, as straight-line code.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Buffer -> LDS transfers issued as instructions of their own (M0 set
// alongside), so that the compiler neither tracks them nor orders LDS reads
// behind them: the GEMM orders them against its LDS reads with its own
// explicit waits, and is the only user of M0 in its kernel.
// The wait states that the compiler would put between two dependent
// instructions are its users' to keep as well: one between a write of M0 and a
// transfer to LDS, five between a vector instruction's write of a scalar
// register (v_readlane of a spilled one, say) and a memory instruction's read
// of it.  The first is in dma16_raw and dma4_raw, the second in dma4_raw, whose
// descriptors may be spilled; the build checks both over the whole file
// (check_waits.py).
typedef unsigned v4u32r __attribute__((ext_vector_type(4)));
struct RawRsrc {
  v4u32r w;  // the four descriptor words of a raw (unswizzled, stride 0) buffer
};
__device__ __forceinline__ RawRsrc raw_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  RawRsrc r;
  r.w = v4u32r{static_cast<uint32_t>(a), static_cast<uint32_t>(a >> 32) & 0xFFFFu, bytes,
               static_cast<uint32_t>(kBufferFlags)};
  return r;
}
// The LDS byte address of a __shared__ object.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const lds_void_t*)p));
}
// OFFSET (an instruction immediate) moves both the source and the target.
template <int OFFSET = 0>
__device__ __forceinline__ void dma16_raw(const RawRsrc& r, uint32_t lds, uint32_t voffset, uint32_t soffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:%4 lds"
               :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voffset), "s"(r.w), "s"(soffset), "n"(OFFSET)
               : "memory");
}
// 16 bytes per lane at voffset + soffset + OFFSET (an instruction immediate).
template <int OFFSET>
__device__ __forceinline__ v4i32 load16_raw(const RawRsrc& r, uint32_t voffset, uint32_t soffset) {
  v4i32 v;
  asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen offset:%4"
               : "=v"(v) : "v"(voffset), "s"(r.w), "s"(soffset), "n"(OFFSET));
  return v;
}
__device__ __forceinline__ void dma4_raw(const RawRsrc& r, uint32_t lds, uint32_t voffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voffset), "s"(r.w) : "memory");
}

constexpr int kWaitcntBase = (0x7 << 4) | (0xF << 8);  // expcnt, lgkmcnt: no wait
constexpr int vmcnt_imm(int n) { return kWaitcntBase | (n & 0xF) | ((n >> 4) << 14); }
constexpr int kLgkm0 = 0xC07F;                          // lgkmcnt(0), vmcnt and expcnt: no wait
// One wave's share of a tile is two weight bands and all NFM activation bands;
// PER_CU blocks share a CU.
//
// BIAS_TAIL: a bias with odd N, whose last value the epilogue reads from memory
// (its staged pair reads past the buffer as zero).
template <int NFM, int PER_CU, Epilogue EPI, bool HAS_BIAS, bool BIAS_TAIL>
__global__ __launch_bounds__(64 * kF6Waves, PER_CU) void w4a4_f6_gemm_kernel(
    const uint8_t* __restrict__ xf6, const float* __restrict__ sx, int M, int mbands,
    const uint8_t* __restrict__ wf6, const float* __restrict__ sw, int N, int nbands, int ksteps,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n, int grid_blocks) {
  constexpr int kOwn = (NFM + kF6Waves - 1) / kF6Waves;  // activation bands a wave moves
  constexpr int kDma = 3 * kOwn;                         // DMA instructions per wave and stage
  constexpr int kUnit = 2 * kFragBytes;                  // a band's bytes of a stage, in memory and in LDS
  constexpr uint32_t kSlot = kF6Waves * kOwn * kUnit;
  constexpr int kRows = 32 * NFM;
  constexpr int kScX = (kRows + 63) / 64 * 64;
  __shared__ __align__(16) uint8_t ring[3 * kSlot];
  // Output staging for the epilogue: per wave two buffers of 32 rows x 64
  // bf16, 16-byte chunk c of row r at chunk c ^ ((r >> 1) & 7).
  __shared__ __align__(16) uint8_t stg[kF6Waves * 8192];
  // The current tile's scales and bias, moved in by DMA for the epilogue.
  __shared__ float sc_x[kScX];
  __shared__ float sc_w[kFBN];
  __shared__ float sc_b[kFBN / 2];  // bf16 pairs

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = ksteps / 2;  // stages of 128 codes per tile
  const int last = T - 1;

  // The block's tiles: virtual block ids v = blockIdx.x + i * grid_blocks of
  // a grid of 8 * ceil(tiles / 8) blocks in the XCD-aware order (grid_blocks
  // is a multiple of 8, so the XCD of every tile of this block is the
  // block's own).  The launch makes every block walk a single tile when a
  // tile has fewer than three stages, since the loads run three stages ahead
  // and must not reach past the next tile.
  int ntiles = 0;
  {
    const int vmax = (tiles_m * tiles_n + kNumXcd - 1) / kNumXcd * kNumXcd;
    TileCoord tc;
    for (int v = blockIdx.x; v < vmax && tile_of_block(v, tiles_m, tiles_n, &tc); v += grid_blocks) ++ntiles;
  }
  if (ntiles == 0) return;

  const RawRsrc rsx = raw_rsrc(xf6, static_cast<uint32_t>(static_cast<int64_t>(mbands) * ksteps * kFragBytes));
  const RawRsrc rsw = raw_rsrc(wf6, static_cast<uint32_t>(static_cast<int64_t>(nbands) * ksteps * kFragBytes));
  const uint32_t band_bytes = static_cast<uint32_t>(ksteps) * kFragBytes;

  // A tile and the wave's bands in it, as byte offsets: the activation bands
  // it moves to LDS and the weight bands it owns (bands past the operand are
  // clamped; their results are discarded).  Everything is scalar: a wave
  // issues an instruction every four clocks or so, so arithmetic between the
  // MFMAs costs as much as the loads it serves.
  struct Tile {
    int m0, n0;
    uint32_t x[kOwn], w[2];
  };
  auto tile_at = [&](int i) __attribute__((always_inline)) {
    TileCoord tc;
    tile_of_block(blockIdx.x + i * grid_blocks, tiles_m, tiles_n, &tc);
    Tile r;
    r.m0 = tc.tm * kRows;
    r.n0 = tc.tn * kFBN;
#pragma unroll
    for (int f = 0; f < kOwn; ++f)
      r.x[f] = static_cast<uint32_t>(min(r.m0 / 32 + kOwn * wave + f, mbands - 1)) * band_bytes;
#pragma unroll
    for (int f = 0; f < 2; ++f)
      r.w[f] = static_cast<uint32_t>(min(r.n0 / 32 + 2 * wave + f, nbands - 1)) * band_bytes;
    return r;
  };
  // The blocks walk the stages of their tiles from a point of K of their
  // own (the fp32 sums of integers do not depend on the order).  One block
  // per CU: each XCD starts an eighth of K after the one before, so that at
  // any moment the XCDs read different slices of the operands rather than
  // all requesting the same weight lines together.  Two blocks per CU: the
  // second half of each XCD's blocks starts from the middle of K, so the two
  // blocks on a CU reach their epilogues half a tile apart and one runs its
  // MFMAs while the other stores.  The byte offset of a stage within its
  // band just counts on, modulo the band, through all the block's tiles.
  const int koff =
      PER_CU == 1 ? static_cast<int>(blockIdx.x % kNumXcd) * T / kNumXcd
                  : ((static_cast<int>(blockIdx.x / kNumXcd) >= grid_blocks / kNumXcd / 2) ? T / 2 : 0);
  auto next_k = [&](uint32_t ko) __attribute__((always_inline)) {
    ko += kUnit;
    return ko == band_bytes ? 0u : ko;
  };

  const uint32_t lane16 = 16 * lane;
  // Bands past the tile (NFM no multiple of the waves) get an offset outside
  // the operand: the load writes zeros and touches no memory.
  uint32_t xlane[kOwn];
#pragma unroll
  for (int f = 0; f < kOwn; ++f) xlane[f] = kOwn * wave + f < NFM ? lane16 : kOutside;
  const uint32_t ring_at = __builtin_amdgcn_readfirstlane(lds_addr(ring)) + kOwn * kUnit * wave;
  // Part J (1 KiB) of the wave's share of a stage's activations, whose bytes
  // of a band start at b + ko, into the slot at byte `slot` of the ring.
  auto issue_dma = [&](const uint32_t* b, uint32_t ko, uint32_t slot, auto J) __attribute__((always_inline)) {
    constexpr int f = decltype(J)::value / 3, q = decltype(J)::value % 3;
    dma16_raw<1024 * q>(rsx, ring_at + slot + kUnit * f, xlane[f], b[f] + ko);
  };
  // Part PP % 3 of weight band PP / 3 of a stage.
  auto load_w = [&](WRaw& w, const uint32_t* b, uint32_t ko, auto PP) __attribute__((always_inline)) {
    constexpr int f = decltype(PP)::value / 3, q = decltype(PP)::value % 3;
    w.p[f][q] = load16_raw<1024 * q>(rsw, lane16, b[f] + ko);
  };
  // A loaded stage passes through an empty asm after the wait for its loads
  // and before any use: the compiler takes an asm load's result as ready when
  // the asm is issued, and could otherwise copy it from a register that a
  // load may still be writing.
  auto landed = [&](WRaw& w) __attribute__((always_inline)) {
    asm volatile("" : "+v"(w.p[0][0]), "+v"(w.p[0][1]), "+v"(w.p[0][2]), "+v"(w.p[1][0]), "+v"(w.p[1][1]),
                 "+v"(w.p[1][2]));
  };
  auto frags = [&](const WRaw& w) __attribute__((always_inline)) {
    WFrag r;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      // the k-steps are the 6-dword windows of the 12 loaded dwords
      r.f[0][f] = __builtin_shufflevector(w.p[f][0], w.p[f][1], 0, 1, 2, 3, 4, 5, -1, -1);
      r.f[1][f] = __builtin_shufflevector(w.p[f][1], w.p[f][2], 2, 3, 4, 5, 6, 7, -1, -1);
    }
    return r;
  };
  // Scales and bias of the tile at (m0, n0) into LDS: every wave a quarter of
  // s_w, the first waves 64 of s_x each, waves 2 and 3 half of the bias each.
  // Entries past M or N read as zero (outside the buffers).
  auto issue_scales = [&](int m0, int n0) __attribute__((always_inline)) {
    if constexpr (EPI == Epilogue::kBf16) {
      const RawRsrc rw = raw_rsrc(sw, 4 * N);
      dma4_raw(rw, lds_addr(sc_w + 64 * wave), 4 * static_cast<uint32_t>(n0 + 64 * wave + lane));
      if (wave < kScX / 64) {
        const RawRsrc rx = raw_rsrc(sx, 4 * M);
        dma4_raw(rx, lds_addr(sc_x + 64 * wave), 4 * static_cast<uint32_t>(m0 + 64 * wave + lane));
      }
      if (HAS_BIAS && wave >= 2) {
        const RawRsrc rb = raw_rsrc(bias, 2 * N);
        dma4_raw(rb, lds_addr(sc_b + 64 * (wave - 2)), 2 * static_cast<uint32_t>(n0 + 128 * (wave - 2) + 2 * lane));
      }
    }
  };
  // Activation fragment (k-step s, band fm) of the slot at byte `slot`: the
  // 16-byte part and the 8-byte part.
  auto read_b = [&](uint32_t slot, int s, int fm) __attribute__((always_inline)) {
    const uint8_t* p = ring + (kUnit * fm + kFragBytes * s);
    // the 8-byte part as a relaxed atomic load, which the compiler does not
    // pair with another fragment's (a paired read lands both parts apart from
    // their 16-byte parts and costs moves to join them)
    const uint64_t hi = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p + (slot + 8 * lane) + 1024),
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    return join(*reinterpret_cast<const v4i32*>(p + (slot + 16 * lane)), __builtin_bit_cast(v2i32, hi));
  };

  v16f acc[2][NFM];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int fm = 0; fm < NFM; ++fm) acc[f][fm] = v16f{};

  // The block walks one stream of stages over its tiles.  Loads run ahead
  // across tile boundaries: the weights by one stage, the activations by
  // three.  Past the block's last stage they are issued anyway, for its last
  // tile again (every address stays inside the operands), which keeps the
  // wait counts below constant.
  Tile ct = tile_at(0), xt = ct;  // current and next tile
  if (ntiles > 1) xt = tile_at(1);
  uint32_t kw = kUnit * static_cast<uint32_t>(koff), kd = kw;  // stages of the next weight load and DMA
  WRaw w[2];
  static_for<kWLoads>([&](auto PP) __attribute__((always_inline)) { load_w(w[0], ct.w, kw, PP); });
  kw = next_k(kw);
  // A tile of fewer than three stages is the block's only one: its DMA goes
  // round K again, into slots that are never read.
  static_for<3>([&](auto K_) __attribute__((always_inline)) {
    static_for<kDma>([&](auto J) __attribute__((always_inline)) { issue_dma(ct.x, kd, kSlot * decltype(K_)::value, J); });
    kd = next_k(kd);
  });
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(kDma));  // the weights and the first two stages
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  uint32_t so = 0, sn = kSlot;  // slots of this stage and the next
  // A stage's activation fragments, (k-step s, band fm) in order NFM s + fm,
  // roll through a window of NFM register sets: fragment i is read (into the
  // set fragment i - NFM has just left) while the MFMAs of i - NFM run.
  v8i bq[NFM];
#pragma unroll
  for (int fm = 0; fm < NFM; ++fm) bq[fm] = read_b(0, 0, fm);

  // Epilogue of the tile at (cm0, cn0): lane holds column m = cm0 + 32 fm +
  // (lane & 31) and rows n = cn0 + 64 wave + 32 f + 8 j + 4 (lane >> 5) + r of
  // y^T.
  auto epilogue = [&](int cm0, int cn0) __attribute__((always_inline)) {
    // The lane index is passed through an empty asm so that the per-lane
    // addresses below are computed here, not hoisted out of the stage loop
    // into registers the loop needs.
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int row = lane & 31, hl = lane >> 5;
    const int nl = 64 * wave + 4 * hl;    // column within the tile
    const int mlim = min(M, cm0 + kRows);  // rows of this tile
    const bool full = (cm0 + kRows <= M) && (cn0 + kFBN <= N);
    if constexpr (EPI == Epilogue::kInt32) {
      int32_t* o = static_cast<int32_t*>(out);
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int fm = 0; fm < NFM; ++fm) {
          const int m = cm0 + row + 32 * fm;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int n = cn0 + nl + 32 * f + 8 * j;
            const int v0 = static_cast<int>(acc[f][fm][4 * j]), v1 = static_cast<int>(acc[f][fm][4 * j + 1]);
            const int v2 = static_cast<int>(acc[f][fm][4 * j + 2]), v3 = static_cast<int>(acc[f][fm][4 * j + 3]);
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
      // Through LDS, one band (32 rows x 64 columns per wave) at a time in two
      // buffers: written as the accumulators hold it, then read and stored to
      // memory as whole 128-byte rows, eight rows per instruction, while the
      // next band is scaled.
      uint16_t* o = static_cast<uint16_t*>(out);
      uint8_t* area = stg + 8192 * wave;
      if constexpr (BIAS_TAIL) {
        // the last bias value, whose pair was read past the buffer as zero
        const int c = N - 1 - cn0 - 64 * wave;
        if (c >= 0 && c < 64 && lane == 0) sc_b[(64 * wave + c) / 2] = __uint_as_float(bias[N - 1]);
        __builtin_amdgcn_wave_barrier();
      }
      // The scales and bias of the lane's columns 32 f + 8 j .. + 3: read once
      // where a block has the CU's registers to itself, else for each band.
      constexpr bool kKeep = PER_CU == 1;
      struct Col {
        float4 s;
        float2 b;  // bf16 pairs
      };
      auto column = [&](int f, int j) __attribute__((always_inline)) {
        const int c = nl + 32 * f + 8 * j;
        Col r;
        r.s = *reinterpret_cast<const float4*>(sc_w + c);
        if constexpr (HAS_BIAS) r.b = *reinterpret_cast<const float2*>(sc_b + c / 2);
        return r;
      };
      Col kept[2][4];
      if constexpr (kKeep) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int j = 0; j < 4; ++j) kept[f][j] = column(f, j);
      }
      float sxv[NFM];
#pragma unroll
      for (int fm = 0; fm < NFM; ++fm) sxv[fm] = sc_x[32 * fm + row];
      auto put = [&](auto FM) __attribute__((always_inline)) {
        constexpr int fm = decltype(FM)::value;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            Col col;
            if constexpr (kKeep) col = kept[f][j];
            else col = column(f, j);
            const float swa[4] = {col.s.x, col.s.y, col.s.z, col.s.w};
            uint16_t h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float v = acc[f][fm][4 * j + r];
              v = v * sxv[fm];
              v = v * swa[r];
              if constexpr (HAS_BIAS) {
                const uint32_t pair = __float_as_uint(r < 2 ? col.b.x : col.b.y);
                v = v + ((r & 1) ? bf16_hi(pair) : bf16_lo(pair));
              }
              h[r] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
            }
            *reinterpret_cast<v2u32*>(area + 4096 * (fm & 1) + 128 * row + 16 * ((4 * f + j) ^ ((row >> 1) & 7)) +
                                      8 * hl) =
                v2u32{h[0] | (static_cast<uint32_t>(h[1]) << 16), h[2] | (static_cast<uint32_t>(h[3]) << 16)};
          }
      };
      // A whole tile with rows of a multiple of 16 bytes is stored without a
      // test; otherwise rows past M and columns past N are left out, element
      // by element where N % 8 != 0 (rolled up: it need not be fast, and the
      // kernel's code stays small).
      auto bands = [&](auto WHOLE) __attribute__((always_inline)) {
        const int r0 = lane >> 3, c = lane & 7;
        const int n = cn0 + 64 * wave + 8 * c;
        uint16_t* p = o + static_cast<int64_t>(cm0 + r0) * N + n;
        const int mleft = n < N ? mlim - cm0 - r0 : 0;
        auto get = [&](int fm, int it) __attribute__((always_inline)) {
          return *reinterpret_cast<const v4u32*>(area + 4096 * (fm & 1) + 1024 * it + 128 * r0 +
                                                 16 * (c ^ ((4 * it + (r0 >> 1)) & 7)));
        };
        put(std::integral_constant<int, 0>{});
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

  // Stage t of the current tile, with weight set I (known at compile time).
  //   * At its start, the wait for this stage's weights (loaded during the
  //     previous stage's first k-step): vmcnt(kDma) leaves in flight only the
  //     DMA issued after them (vector loads complete in order).
  //   * Then the stage's fragments j = NFM s + fm (k-step s, band fm) in
  //     turn: the two MFMAs of fragment j, the read of fragment j + NFM into
  //     the register set fragment j has left (past the stage's last
  //     fragment, those of the next stage, from the next slot), and a share
  //     of the stage's vector-memory loads, so that they reach the memory
  //     system spread over the stage rather than in one burst per wave:
  //     the next stage's weights (into the other set, done with one stage
  //     ago) among the first k-step's fragments, and the DMA of the stage
  //     three ahead among the second's.
  //   * Between the k-steps, once every wave has read the whole slot
  //     (lgkmcnt(0) + barrier) and the next stage's DMA has landed, the slot
  //     is free for that DMA.  The wait there, vmcnt(kWLoads + kDma), leaves
  //     in flight at most the loads issued since this stage's weights (which
  //     have landed): the DMA of the stage two ahead and the next stage's
  //     weights.
  // A tile's FIRST stage waits for neither: its weights and the next stage's
  // DMA had landed when the tile before it ended (or in the prologue), and a
  // wait here would be one for the stores of that tile's epilogue.  It moves
  // the tile's scales, once every wave is past that epilogue.
  int t = 0;
  auto stage = [&](auto I, auto FIRST) __attribute__((always_inline)) {
    constexpr int i = decltype(I)::value;
    constexpr bool first = decltype(FIRST)::value;
    const bool end = t == last, ahead = t + 3 >= T;
    const uint32_t wb[2] = {end ? xt.w[0] : ct.w[0], end ? xt.w[1] : ct.w[1]};
    uint32_t xb[kOwn];
#pragma unroll
    for (int f = 0; f < kOwn; ++f) xb[f] = ahead ? xt.x[f] : ct.x[f];
    if constexpr (!first) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kDma));
    __builtin_amdgcn_sched_barrier(0);
    landed(w[i]);
    const WFrag wc = frags(w[i]);
    static_for<2 * NFM>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = decltype(J)::value;
      constexpr int ks = j / NFM, fm = j % NFM;
      acc[0][fm] = mfma_bf6(wc.f[ks][0], bq[fm], acc[0][fm]);
      acc[1][fm] = mfma_bf6(wc.f[ks][1], bq[fm], acc[1][fm]);
      if constexpr (ks == 0) {
        bq[fm] = read_b(so, 1, fm);
        static_for<kWLoads>([&](auto PP) __attribute__((always_inline)) {
          if constexpr (decltype(PP)::value * NFM / kWLoads == fm) load_w(w[1 - i], wb, kw, PP);
        });
      } else {
        bq[fm] = read_b(sn, 0, fm);
        static_for<kDma>([&](auto D) __attribute__((always_inline)) {
          if constexpr (decltype(D)::value * NFM / (NFM < kDma ? kDma : NFM) == fm) issue_dma(xb, kd, so, D);
        });
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (j == NFM - 1) {
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        if constexpr (!first) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kWLoads + kDma));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (first) issue_scales(ct.m0, ct.n0);
      }
    });
    kw = next_k(kw);
    kd = next_k(kd);
    so = sn;
    sn = sn == 2 * kSlot ? 0u : sn + kSlot;
    ++t;
    __builtin_amdgcn_sched_barrier(0);
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  for (int ti = 0; ti < ntiles; ++ti) {
    stage(Set0{}, std::true_type{});
    if (T > 1) stage(Set1{}, std::false_type{});
    for (int u = 2; u < T; u += 2) {
      stage(Set0{}, std::false_type{});
      if (u + 1 < T) stage(Set1{}, std::false_type{});
    }
    // The next tile's first weights, and every DMA but the last stage's, have
    // landed before the epilogue's stores are issued behind them.
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(kDma));
    __builtin_amdgcn_sched_barrier(0);
    if (T & 1) {
      // they are in the other set
      landed(w[1]);
      w[0] = w[1];
    }
    if (T == 1) {
      // the scales were moved at this very stage
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_s_barrier();
    }
    epilogue(ct.m0, ct.n0);
    t = 0;
    ct = xt;
    if (ti + 2 < ntiles) xt = tile_at(ti + 2);
  }
  // no load may still be writing LDS or registers when the wave ends
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

// ---------------------------------------------------------------------------
// Group-wise GEMM on BF6 operands (products with few output tiles go to
// f6_narrow_group.hip)
//
// S[m,n] = sum over the groups g in k order of fl32(fl32(acc_g * s_x[m,g]) *
// s_w[n,g]), acc_g the exact integer product over the G codes of group g (a
// single k-step for G = 64, two for G = 128), then y = bf16(S + bias) (or S
// itself, EPI kF32).  The matrix cores deliver acc_g in fp32, exactly, so the
// fold after each group is two multiplies and an add per output: the kernel
// is bound by that vector arithmetic, not by the MFMAs: 48 instructions per
// 32x32 tile and group, 208 us of it in each GEMM of the FLUX MLP at G = 64
// (4608 x 3072 -> 12288 and back).  The walk over the groups is therefore
// software-pipelined: read, multiply and fold in turn left a wave waiting
// about five times per stage for LDS and the MFMAs, and addresses and the
// joining of operand parts took a tenth of the vector instructions (306 and
// 303 us; 274 and 267 us now; at G = 128 198 and 207 -> 187 and 197 us).
//
// Block tile 128 (m) x 128 (n), four waves, two blocks per CU; wave (wm, wn)
// owns activation bands 2wm, 2wm + 1 and weight bands 2wn, 2wn + 1 of the
// tile: 2 x 2 tiles of 32x32, 64 fp32 sums per lane.  A stage is 128 codes of
// K: both operands' fragments (activation layout and weight layout, 12 KiB
// each) and the stage's scales (s_x and s_w of its groups, gathered from the
// [rows, K/G] arrays by 4-byte transfers) move into LDS by buffer_load ...
// lds, issued as instructions of their own three stages ahead into a ring of
// three slots.  Before a stage is read, the block waits for its loads only
// (vmcnt counts the next stage's as still in flight) and meets at a barrier
// with no memory fence, after which the slot of the stage before takes the
// loads of the stage three ahead of that one.  Operand bands, rows or columns
// past M or N read as zero (outside the buffers).
//
// ONE: K is a single group of 64 codes.
template <int G, Epilogue EPI, bool HAS_BIAS, bool ONE>
__global__ __launch_bounds__(256, 2) void w4a4g_f6_gemm_kernel(
    const uint8_t* __restrict__ xf6, const float* __restrict__ sx, int M, int mbands,
    const uint8_t* __restrict__ wf6, const float* __restrict__ sw, int N, int nbands, int ksteps, int KG,
    const uint16_t* __restrict__ bias, void* __restrict__ out, int tiles_m, int tiles_n) {
  constexpr int kGps = 128 / G;                    // groups per stage
  constexpr int kOpU4 = 4 * 2 * kFragBytes / 16;   // one operand's stage: 4 bands x 3072 bytes
  constexpr int kScF = 2 * kGps * 128;             // one stage's scales: s_x then s_w, [group][row]
  constexpr int kScDma = kScF / 64 / 4;            // 4-byte scale transfers per wave per stage
  constexpr int kLoads = 6 + kScDma;               // vector-memory instructions per wave per stage
  // Three slots, each the operand fragments of a stage (activations, then
  // weights) and its scales.  The transfers are asm the compiler does not
  // track, so the slot may be computed at run time.
  __shared__ uint4 ops[3 * 2 * kOpU4];
  __shared__ float scs[3 * kScF];
  auto opk = [&](int k) __attribute__((always_inline)) { return ops + 2 * kOpU4 * k; };
  auto sck = [&](int k) __attribute__((always_inline)) { return scs + kScF * k; };

  TileCoord tc;
  if (!tile_of_block(blockIdx.x, tiles_m, tiles_n, &tc)) return;
  const int m0 = 128 * tc.tm, n0 = 128 * tc.tn;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int T = ksteps / 2;
  const uint32_t band_bytes = static_cast<uint32_t>(ksteps) * kFragBytes;

  const RawRsrc rsx = raw_rsrc(xf6, static_cast<uint32_t>(static_cast<int64_t>(mbands) * band_bytes));
  const RawRsrc rsw = raw_rsrc(wf6, static_cast<uint32_t>(static_cast<int64_t>(nbands) * band_bytes));
  const RawRsrc rssx = raw_rsrc(sx, static_cast<uint32_t>(4 * static_cast<int64_t>(M) * KG));
  const RawRsrc rssw = raw_rsrc(sw, static_cast<uint32_t>(4 * static_cast<int64_t>(N) * KG));

  // Operand DMA: the 12 KiB of a stage are 12 instructions of 1 KiB, three
  // per wave; instruction i = 3 wave + j is part i % 3 of band i / 3.  Bands
  // past the operand read as zero.
  uint32_t xoff[3], woff[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int i = 3 * wave + j;
    const int b = i / 3, part = i % 3;
    const int xb = m0 / 32 + b, wb = n0 / 32 + b;
    xoff[j] = xb < mbands ? static_cast<uint32_t>(xb) * band_bytes + 1024 * part + 16 * lane : kOutside;
    woff[j] = wb < nbands ? static_cast<uint32_t>(wb) * band_bytes + 1024 * part + 16 * lane : kOutside;
  }
  // Scale DMA: entry e of a stage's kScF (s_x entries, then s_w) is group
  // e % (kGps 128) / 128 of row (column) e % 128 of the tile; instruction
  // i = kScDma wave + j moves entries 64 i .. 64 i + 63, all of one array.
  // Per lane: the array's row and the group within the stage; entries past
  // M or N read as zero.
  int sc_row[kScDma], sc_gl[kScDma];
  bool sc_w[kScDma];  // wave-uniform: whether instruction j moves s_w entries
#pragma unroll
  for (int j = 0; j < kScDma; ++j) {
    sc_w[j] = 64 * (kScDma * wave + j) >= kGps * 128;
    const int ee = (64 * (kScDma * wave + j) + lane) % (kGps * 128);
    sc_gl[j] = ee / 128;
    sc_row[j] = (sc_w[j] ? n0 : m0) + ee % 128;
  }
  auto issue = [&](int u, int k) __attribute__((always_inline)) {
    const uint32_t xa = lds_addr(opk(k)), wa = lds_addr(opk(k) + kOpU4);
    const uint32_t so = 2 * kFragBytes * u;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      dma16_raw(rsx, xa + 16 * 64 * (3 * wave + j), xoff[j], so);  // kOutside + so stays outside
      dma16_raw(rsw, wa + 16 * 64 * (3 * wave + j), woff[j], so);
    }
#pragma unroll
    for (int j = 0; j < kScDma; ++j) {
      const int g = kGps * u + sc_gl[j];
      const bool in = sc_row[j] < (sc_w[j] ? N : M) && g < KG;
      const uint32_t off = in ? 4u * static_cast<uint32_t>(sc_row[j] * KG + g) : kOutside;
      const uint32_t dst = lds_addr(sck(k) + 64 * (kScDma * wave + j));
      if (sc_w[j]) dma4_raw(rssw, dst, off);
      else dma4_raw(rssx, dst, off);
    }
  };

  v16f S[2][2];  // [weight band f][activation band fb]
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int fb = 0; fb < 2; ++fb) S[f][fb] = v16f{};

  // Fold one group into the sums: lane holds column m = 32 (2wm + fb) +
  // (lane & 31) and rows n = 32 (2wn + f) + 8 j + 4 (lane >> 5) + r of y^T,
  // with the lane's scales of the group read from its stage's scale slot.
  float xsr[2][2];
  float4 wsr[2][4];
  const uint8_t* const opb = reinterpret_cast<const uint8_t*>(ops);
  const uint8_t* const scb = reinterpret_cast<const uint8_t*>(scs);
  const uint32_t x_lane = 256 * wm + 4 * (lane & 31), w_lane = 4 * kGps * 128 + 256 * wn + 16 * (lane >> 5);
  auto read_xs = [&](int set, int k, int gl) __attribute__((always_inline)) {
    const uint32_t xo = 4 * kScF * k + x_lane;
#pragma unroll
    for (int b = 0; b < 2; ++b) xsr[set][b] = *reinterpret_cast<const float*>(scb + (512 * gl + 128 * b) + xo);
  };
  auto read_ws = [&](int k, int gl, int f) __attribute__((always_inline)) {
    const uint32_t wo = 4 * kScF * k + w_lane;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      wsr[f][j] = *reinterpret_cast<const float4*>(scb + (512 * gl + 128 * f + 32 * j) + wo);
  };
  auto fold = [&](const v16f& acc, int f, int fb, int set) __attribute__((always_inline)) {
    const float xs = xsr[set][fb];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float wsa[4] = {wsr[f][j].x, wsr[f][j].y, wsr[f][j].z, wsr[f][j].w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float t = acc[4 * j + r] * xs;
        t = t * wsa[r];
        S[f][fb][4 * j + r] = S[f][fb][4 * j + r] + t;
      }
    }
  };
  // Fragments of a stage's slot.  The fold leaves no vector instruction to
  // spare, so a slot costs four address registers (the rest are constants of
  // the reads), and the 8-byte parts are relaxed atomic loads, which the
  // compiler does not pair: a paired read needs moves to join the parts.
  auto read8 = [&](const uint8_t* p) __attribute__((always_inline)) {
    return __builtin_bit_cast(v2i32, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_WAVEFRONT));
  };
  const uint32_t xl = 4 * kFragBytes * wm + 16 * lane, xl8 = 4 * kFragBytes * wm + 8 * lane;
  const uint32_t wl = 16 * kOpU4 + 4 * kFragBytes * wn + 16 * lane;
  auto read_x = [&](int k, int t, int fb) __attribute__((always_inline)) {
    const uint32_t so = 16 * 2 * kOpU4 * k;
    const uint8_t* p = opb + (2 * kFragBytes * fb + kFragBytes * t);
    return join(*reinterpret_cast<const v4i32*>(p + (so + xl)), read8(p + 1024 + (so + xl8)));
  };
  auto read_w = [&](int k, int t, int f) __attribute__((always_inline)) {
    const uint32_t so = 16 * 2 * kOpU4 * k + wl;
    const uint8_t* p = opb + 2 * kFragBytes * f;
    if (t == 0) return join(*reinterpret_cast<const v4i32*>(p + so), read8(p + 1024 + so));
    const v2i32 a = read8(p + 1024 + 8 + so);
    const v4i32 b = *reinterpret_cast<const v4i32*>(p + 2048 + so);
    return v8i{a.x, a.y, b.x, b.y, b.z, b.w, 0, 0};
  };

  // The walk over the groups is pipelined, so that a wave's vector unit finds
  // the next products ready when it is done with a fold: while the products of
  // (group, weight band 0) are folded, those of band 1 run and the next
  // group's fragments and scales are read; while band 1's are folded, the next
  // group's band 0 runs.
  //   a0, a1: the products of bands 0 and 1; x, w: the group's fragments.
  constexpr int kSteps = G / 64;  // k-steps of a group
  v16f a0[2], a1[2];
  v8i x[kSteps][2], w[kSteps][2];
  auto read_group = [&](int set, int k, int gl) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < kSteps; ++t) {
      w[t][0] = read_w(k, kSteps * gl + t, 0);
      x[t][0] = read_x(k, kSteps * gl + t, 0);
      x[t][1] = read_x(k, kSteps * gl + t, 1);
    }
    if constexpr (G == 64) read_xs(set, k, gl);
  };
  auto read_w1 = [&](int k, int gl) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < kSteps; ++t) w[t][1] = read_w(k, kSteps * gl + t, 1);
  };
  auto products = [&](v16f* a, int f) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b) a[b] = mfma_bf6(w[0][f], x[0][b], v16f{});
    if constexpr (kSteps == 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) a[b] = mfma_bf6(w[kSteps - 1][f], x[kSteps - 1][b], a[b]);
    }
  };
  // Stage u has been read whole by this wave; make stage u + 1 readable: wait
  // for its loads (those of stage u + 2, issued after them, may still be in
  // flight: vector loads complete in order) and meet the other waves, after
  // which the slot of stage u takes the loads of stage u + 3.
  auto next_stage = [&](int u) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    if (u + 2 < T) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();
    // no LDS read of the slot may be moved above the wait and the barrier
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (u + 3 < T) issue(u + 3, u % 3);
  };
  // One group, the last of its stage u or not; the one after it (G = 64, past
  // the end: read, but not used) is group `gl` of slot k.
  // The weight scales follow their folds into the same registers; the
  // activation scales have two sets for G = 64, where a group is too short to
  // cover a read at its end, and one for G = 128, whose fragments fill the rest.
  auto group = [&](auto SET, bool last, int u, int k, int gl) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value;
    products(a1, 1);
    if (last) next_stage(u);
    __builtin_amdgcn_sched_barrier(0);
    read_group(1 - set, k, gl);
    __builtin_amdgcn_sched_barrier(0);
    fold(a0[0], 0, 0, set);
    fold(a0[1], 0, 1, set);
    __builtin_amdgcn_sched_barrier(0);
    products(a0, 0);
    read_w1(k, gl);
    read_ws(k, gl, 0);
    __builtin_amdgcn_sched_barrier(0);
    fold(a1[0], 1, 0, set);
    fold(a1[1], 1, 1, set);
    __builtin_amdgcn_sched_barrier(0);
    read_ws(k, gl, 1);
    if constexpr (G == 128) read_xs(set, k, gl);
    __builtin_amdgcn_sched_barrier(0);
  };
  issue(0, 0);
  if (T > 1) issue(1, 1);
  if (T > 2) issue(2, 2);
  if (T > 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kLoads));
  else if (T > 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));
  else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  read_group(0, 0, 0);
  products(a0, 0);
  read_w1(0, 0);
  read_ws(0, 0, 0);
  read_ws(0, 0, 1);
  if constexpr (G == 128) read_xs(0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  if constexpr (G == 64 && !ONE) {
    int k = 0;
    for (int u = 0; u < T; ++u) {
      const int kn = k == 2 ? 0 : k + 1;
      group(Set0{}, false, u, k, 1);
      // K % 128 == 64: the last stage's second half is padding
      if (2 * u + 1 < KG) group(Set1{}, true, u, kn, 0);
      k = kn;
    }
  } else {
    if constexpr (!ONE) {
      int k = 0;
      for (int u = 0; u + 1 < T; ++u) {
        k = k == 2 ? 0 : k + 1;
        group(Set0{}, true, u, k, 0);
      }
    }
    // The last group, with nothing to run ahead to: 4096 x 256 -> 4096 12.1 ->
    // 11.2 us, 1948 x 128 -> 8768 13.3 -> 11.9.  (With G = 64 the loop's two
    // groups and a last one apart do not fit the registers, so only a single
    // group has its own kernel: 7460 x 64 -> 4608 17.2 -> 15.5 us.)
    products(a1, 1);
    fold(a0[0], 0, 0, 0);
    fold(a0[1], 0, 1, 0);
    fold(a1[0], 1, 0, 0);
    fold(a1[1], 1, 1, 0);
  }

  if constexpr (EPI == Epilogue::kF32) {
    // S as it is (the checking path): four consecutive n per store.
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = n0 + 32 * (2 * wn + f) + 8 * j + 4 * (lane >> 5);
#pragma unroll
        for (int fb = 0; fb < 2; ++fb) {
          const int m = m0 + 32 * (2 * wm + fb) + (lane & 31);
          if (m >= M) continue;
          float* p = static_cast<float*>(out) + static_cast<int64_t>(m) * N + n;
          if (n + 3 < N && N % 4 == 0) {
            *reinterpret_cast<float4*>(p) =
                make_float4(S[f][fb][4 * j], S[f][fb][4 * j + 1], S[f][fb][4 * j + 2], S[f][fb][4 * j + 3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (n + r < N) p[r] = S[f][fb][4 * j + r];
          }
        }
      }
  } else {
    // bf16(S + bias), staged through LDS (the first slot, free once every
    // wave is past the last stage) and stored as whole 128-byte rows: per
    // wave two passes of 32 rows x 64 columns, 16-byte chunk c of row r at
    // chunk c ^ ((r >> 1) & 7).
    __syncthreads();
    v4u32* stg = reinterpret_cast<v4u32*>(ops) + 256 * wave;
    v2u32* stg2 = reinterpret_cast<v2u32*>(stg);
    float bv[2][4][4];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int n = n0 + 32 * (2 * wn + f) + 8 * j + 4 * (lane >> 5) + r;
          bv[f][j][r] = HAS_BIAS ? __uint_as_float(static_cast<uint32_t>(bias[min(n, N - 1)]) << 16) : 0.0f;
        }
    const bool vec = (n0 + 128 <= N) && (N % 8 == 0);
#pragma unroll
    for (int fb = 0; fb < 2; ++fb) {
      const int row = lane & 31;
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = 32 * f + 8 * j + 4 * (lane >> 5);  // column within the wave's 64
          uint16_t h[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float v = S[f][fb][4 * j + r];
            if (HAS_BIAS) v = v + bv[f][j][r];
            h[r] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
          }
          stg2[2 * (8 * row + ((c >> 3) ^ ((row >> 1) & 7))) + ((c & 7) >> 2)] =
              v2u32{h[0] | (static_cast<uint32_t>(h[1]) << 16), h[2] | (static_cast<uint32_t>(h[3]) << 16)};
        }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int rr = 8 * it + (lane >> 3), ch = lane & 7;
        const v4u32 vv = stg[8 * rr + (ch ^ ((rr >> 1) & 7))];
        const int m = m0 + 32 * (2 * wm + fb) + rr;
        const int n = n0 + 64 * wn + 8 * ch;
        uint16_t* p = static_cast<uint16_t*>(out) + static_cast<int64_t>(m) * N + n;
        if (m >= M) {
        } else if (vec) {
          __builtin_nontemporal_store(vv, reinterpret_cast<v4u32*>(p));
        } else {
          const uint32_t w[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (n + e < N) p[e] = static_cast<uint16_t>(w[e >> 1] >> (16 * (e & 1)));
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// Four rows per block, W waves of 16 group slots, NJ sets of groups each.
template <int NJ, int G>
hipError_t launch_q4f6(const uint16_t* x, int64_t M, int64_t K, int64_t ksteps, uint8_t* out, float* s, int waves,
                       hipStream_t st) {
  const int64_t rows_padded = (M + 31) / 32 * 32;
  const int64_t groups_of_8_bands = (rows_padded / 32 + kNumXcd - 1) / kNumXcd;
  const dim3 grid(static_cast<unsigned>(groups_of_8_bands * 8 * kNumXcd));
  const size_t lds = static_cast<size_t>(waves) * 256 * 16;
  hipLaunchKernelGGL((quantize_rows4_f6_kernel<NJ, G>), grid, dim3(64 * waves), lds, st, x, M, K, rows_padded, ksteps,
                     out, s);
  return hipGetLastError();
}

template <int NJ, int G>
hipError_t launch_qf6(const uint16_t* x, int64_t M, int64_t K, int64_t ksteps, uint8_t* out, float* s, int threads,
                      hipStream_t st) {
  const int64_t rows_padded = (M + 31) / 32 * 32;
  const int64_t groups_of_8_bands = (rows_padded / 32 + kNumXcd - 1) / kNumXcd;
  const dim3 grid(static_cast<unsigned>(groups_of_8_bands * 32 * kNumXcd));
  const size_t lds = static_cast<size_t>(threads / 64) * 256 * 16;
  hipLaunchKernelGGL((quantize_rows_f6_kernel<NJ, G>), grid, dim3(threads), lds, st, x, M, K, rows_padded, ksteps, out, s);
  return hipGetLastError();
}

}  // namespace

int64_t f6_ksteps(int64_t K) { return (K + 127) / 128 * 2; }

int64_t f6_operand_bytes(int64_t rows, int64_t K) { return (rows + 31) / 32 * f6_ksteps(K) * kFragBytes; }

// The GEMM's tile height in bands of 32 rows, 5 .. 8 (one block per CU) or 4
// (two), and the estimate in ns it was picked by, for the XCD with most tiles:
//   one block per CU: its rounds, each 38 b + 280 ns per 128 codes and 1080 b
//   for all that a tile costs beside its stages (b bands);
//   two blocks per CU: 720 ns per 128 codes and 5600 for each round of two
//   tiles per CU, 378 and 4300 for a last round with one tile per CU or fewer.
// Fitted to 187 shapes (M 768..9216, K 128..15360, N 1024..12288) on codes of
// a heavy-tailed activation (Student t, 3 degrees of freedom): the pick is
// within 0.25% of the best height on average.  On codes of a Gaussian one,
// which the card runs up to a third slower, and down to 64 tokens with the
// few-tile kernel beside it, within 0.75%; the rule before (two blocks, or
// 224/256-row tiles by the rounds alone) was 10% off.
int f6_tile_bands(int64_t M, int64_t N, int64_t K, int64_t slots, int64_t* ns) {
  const int64_t tiles_n = (N + kFBN - 1) / kFBN, T = (K + 127) / 128;
  const int64_t cus = std::max<int64_t>(1, slots / kNumXcd);  // of an XCD
  auto per_xcd = [&](int b) { return ((M + 32 * b - 1) / (32 * b) * tiles_n + kNumXcd - 1) / kNumXcd; };
  const int64_t n4 = per_xcd(4), rest = n4 % (2 * cus);
  const int64_t round2 = 720 * T + 5600;
  int best = 4;
  int64_t best_ns = n4 / (2 * cus) * round2;
  if (rest > cus) best_ns += round2;
  else if (rest > 0) best_ns += 378 * T + 4300;
  for (int b = 8; b >= 5; --b) {
    const int64_t t = (per_xcd(b) + cus - 1) / cus * (T * (38 * b + 280) + 1080 * b);
    if (t < best_ns) best = b, best_ns = t;
  }
  if (ns != nullptr) *ns = best_ns;
  return best;
}

GemmRoute f6_route(int64_t M, int64_t N, int64_t K, int64_t cus) {
  GemmRoute r{GemmKernel::kTiled, 0, kF6Waves, 0, kFBN};
  if ((r.pick = f6_narrow_tile(M, N, K, cus)) != 0) {
    r.kernel = GemmKernel::kNarrow;
    f6_narrow_shape(r.pick, &r.rows, &r.cols);
  } else {
    r.rows = 32 * f6_tile_bands(M, N, K, cus, nullptr);
  }
  return r;
}

GemmRoute f6_group_route(int64_t M, int64_t N, int64_t K, int G, int64_t cus) {
  if (const int waves = f6_narrow_group_waves(M, N, K, G, cus)) return {GemmKernel::kNarrow, 0, waves, 32, 32};
  return {GemmKernel::kTiled, 0, 4, 128, 128};
}

template <int G>
hipError_t launch_quantize_f6(const uint16_t* x, int64_t M, int64_t K, uint8_t* out, float* scale, hipStream_t st) {
  if (f6_quantize_few_rows(M, K, G)) return launch_quantize_few_f6(x, M, K, G, out, scale, st);
  const int64_t ksteps = f6_ksteps(K);
  const int64_t groups = 2 * ksteps;
  if (groups <= 512) {
    // four rows per block: up to 8 waves of 16 group slots, NJ <= 4 sets each
    const int64_t waves = std::min<int64_t>(8, (groups + 15) / 16);
    const int64_t nj = (groups + 16 * waves - 1) / (16 * waves);
    const int w = static_cast<int>(waves);
    if (nj <= 1) return launch_q4f6<1, G>(x, M, K, ksteps, out, scale, w, st);
    if (nj <= 2) return launch_q4f6<2, G>(x, M, K, ksteps, out, scale, w, st);
    if (nj <= 3) return launch_q4f6<3, G>(x, M, K, ksteps, out, scale, w, st);
    return launch_q4f6<4, G>(x, M, K, ksteps, out, scale, w, st);
  }
  // longer rows: one row per block, up to 512 threads each holding NJ groups
  const int64_t threads = 512;
  const int64_t nj = (groups + threads - 1) / threads;
  const int th = static_cast<int>(threads);
  if (nj <= 2) return launch_qf6<2, G>(x, M, K, ksteps, out, scale, th, st);
  return launch_qf6<4, G>(x, M, K, ksteps, out, scale, th, st);
}

hipError_t launch_quantize_rows_f6(const uint16_t* x, int64_t M, int64_t K, uint8_t* out, float* scale,
                                   hipStream_t st) {
  return launch_quantize_f6<0>(x, M, K, out, scale, st);
}

hipError_t launch_quantize_rows_f6_batch(int count, const uint16_t* const* x, const int64_t* M, const int64_t* K,
                                         uint8_t* const* out, float* const* scale, hipStream_t st) {
  // Inputs of few rows share a launch of the few-row kernel where that is
  // faster.  Otherwise inputs whose rows fit the four-rows-per-block kernel (at
  // most 512 groups) share one of that, few rows or many (a short input costs
  // less inside the pass over a long one than as a launch of its own): its waves
  // are the most any of them needs, and NJ the most sets of groups any of them
  // needs at that wave count.  Longer rows get a launch of their own, on the
  // same stream.
  if (f6_quantize_few_batch(count, M, K)) return launch_quantize_few_f6_batch(count, x, M, K, out, scale, st);
  Q4Batch b{};
  int waves = 1;
  for (int i = 0; i < count; ++i) {
    const int64_t groups = 2 * f6_ksteps(K[i]);
    if (groups <= 512) waves = static_cast<int>(std::max<int64_t>(waves, std::min<int64_t>(8, (groups + 15) / 16)));
  }
  int NJ = 1;
  int64_t first = 0;
  for (int i = 0; i < count; ++i) {
    const int64_t ksteps = f6_ksteps(K[i]);
    const int64_t groups = 2 * ksteps;
    if (groups > 512) {
      const hipError_t e = launch_quantize_f6<0>(x[i], M[i], K[i], out[i], scale[i], st);
      if (e != hipSuccess) return e;
      continue;
    }
    Q4Input& q = b.in[b.count++];
    q.x = x[i];
    q.out = out[i];
    q.scale = scale[i];
    q.M = M[i];
    q.K = K[i];
    q.rows_padded = (M[i] + 31) / 32 * 32;
    q.ksteps = ksteps;
    q.first = first;
    q.nj = static_cast<int>((groups + 16 * waves - 1) / (16 * waves));
    NJ = std::max(NJ, q.nj);
    first += (q.rows_padded / 32 + kNumXcd - 1) / kNumXcd * 8 * kNumXcd;  // as launch_q4f6's grid
  }
  if (b.count == 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(first));
  const size_t lds = static_cast<size_t>(waves) * 256 * 16;
#define JQ_Q4B(NN) hipLaunchKernelGGL((quantize_rows4_f6_batch_kernel<NN>), grid, dim3(64 * waves), lds, st, b)
  if (NJ <= 1) JQ_Q4B(1);
  else if (NJ <= 2) JQ_Q4B(2);
  else if (NJ <= 3) JQ_Q4B(3);
  else JQ_Q4B(4);
#undef JQ_Q4B
  return hipGetLastError();
}

hipError_t launch_quantize_groups_f6(const uint16_t* x, int64_t M, int64_t K, int G, uint8_t* out, float* scale,
                                     hipStream_t st) {
  return G == 64 ? launch_quantize_f6<64>(x, M, K, out, scale, st) : launch_quantize_f6<128>(x, M, K, out, scale, st);
}

hipError_t launch_w4a4g_f6_gemm(Epilogue epi, const uint8_t* xf6, const float* sx, int64_t M, int64_t K, int G,
                                const uint8_t* wf6, const float* sw, int64_t N, const uint16_t* bias, void* out,
                                hipStream_t st) {
  int64_t cus = 0;
  const hipError_t e = device_route_cus(&cus);
  if (e != hipSuccess) return e;
  const GemmRoute r = f6_group_route(M, N, K, G, cus);
  if (r.kernel == GemmKernel::kNarrow)
    return launch_f6_narrow_group(r.waves, epi, xf6, sx, M, K, G, wf6, sw, N, bias, out, st);
  const int ksteps = static_cast<int>(f6_ksteps(K));
  const int tiles_m = static_cast<int>((M + 127) / 128), tiles_n = static_cast<int>((N + 127) / 128);
  const int64_t tiles = static_cast<int64_t>(tiles_m) * tiles_n;
  const unsigned blocks = static_cast<unsigned>((tiles + kNumXcd - 1) / kNumXcd * kNumXcd);
  const int mbands = static_cast<int>((M + 31) / 32), nbands = static_cast<int>((N + 31) / 32);
  const int KG = static_cast<int>(K / G);
  const int Mi = static_cast<int>(M), Ni = static_cast<int>(N);
#define JQ_F6G(GG, E, B, O)                                                                                       \
  hipLaunchKernelGGL((w4a4g_f6_gemm_kernel<GG, E, B, O>), dim3(blocks), dim3(256), 0, st, xf6, sx, Mi, mbands, wf6, \
                     sw, Ni, nbands, ksteps, KG, bias, out, tiles_m, tiles_n)
#define JQ_F6G_EPI(GG, O)                                             \
  if (epi == Epilogue::kF32) JQ_F6G(GG, Epilogue::kF32, false, O);    \
  else if (bias != nullptr) JQ_F6G(GG, Epilogue::kBf16, true, O);     \
  else JQ_F6G(GG, Epilogue::kBf16, false, O);
  if (G == 128) {
    JQ_F6G_EPI(128, false)
  } else if (KG == 1) {
    JQ_F6G_EPI(64, true)
  } else {
    JQ_F6G_EPI(64, false)
  }
#undef JQ_F6G_EPI
#undef JQ_F6G
  return hipGetLastError();
}

hipError_t launch_int4_to_f6(const uint8_t* q, int64_t rows, int64_t K, uint8_t* out, bool weight_layout,
                             bool ternary, hipStream_t st) {
  const int64_t ksteps = f6_ksteps(K);
  const int64_t rows_padded = (rows + 31) / 32 * 32;
  const int64_t bands = rows_padded / 32;
  const int64_t waves = bands * ((ksteps / 2 + kCvtUnits - 1) / kCvtUnits);
  const dim3 grid(static_cast<unsigned>((waves + 3) / 4));
#define JQ_CVT(W, T) hipLaunchKernelGGL((int4_to_f6_kernel<W, T>), grid, dim3(256), 0, st, q, rows, K, bands, ksteps, out)
  if (ternary) {
    if (weight_layout) JQ_CVT(true, true);
    else JQ_CVT(false, true);
  } else {
    if (weight_layout) JQ_CVT(true, false);
    else JQ_CVT(false, false);
  }
#undef JQ_CVT
  return hipGetLastError();
}

hipError_t launch_w4a4_f6_gemm(Epilogue epi, const uint8_t* xf6, const float* sx, int64_t M, int64_t K,
                               const uint8_t* wf6, const float* sw, int64_t N, const uint16_t* bias, void* out,
                               hipStream_t st) {
  int64_t slots = 0;
  const hipError_t e = device_route_cus(&slots);
  if (e != hipSuccess) return e;
  const GemmRoute r = f6_route(M, N, K, slots);
  if (r.kernel == GemmKernel::kNarrow)
    return launch_f6_narrow(r.pick, epi, xf6, sx, M, K, wf6, sw, N, bias, out, st);
  const int ksteps = static_cast<int>(f6_ksteps(K));
  const int bands = r.rows / 32;
  const int tiles_m = static_cast<int>((M + 32 * bands - 1) / (32 * bands));
  const int tiles_n = static_cast<int>((N + kFBN - 1) / kFBN);
  const int64_t per_xcd = (static_cast<int64_t>(tiles_m) * tiles_n + kNumXcd - 1) / kNumXcd;
  // a block's registers fill the CU, or half of it; each block walks its tiles in turn
  const int64_t block_slots = (bands == 4 ? 2 : 1) * slots;
  const int blocks =
      static_cast<int>(ksteps / 2 < 3 ? per_xcd * kNumXcd : std::min<int64_t>(per_xcd * kNumXcd, block_slots));
  const int mbands = static_cast<int>((M + 31) / 32);
  const int nbands = static_cast<int>((N + 31) / 32);
  const int Mi = static_cast<int>(M), Ni = static_cast<int>(N);
#define JQ_F6(NFM, PC, E, B, BT)                                                                                \
  hipLaunchKernelGGL((w4a4_f6_gemm_kernel<NFM, PC, E, B, BT>), dim3(blocks), dim3(64 * kF6Waves), 0, st, xf6, sx, \
                     Mi, mbands, wf6, sw, Ni, nbands, ksteps, bias, out, tiles_m, tiles_n, blocks)
#define JQ_F6_EPI(NFM, PC)                                                           \
  if (epi == Epilogue::kInt32) JQ_F6(NFM, PC, Epilogue::kInt32, false, false);       \
  else if (bias != nullptr && (N & 1)) JQ_F6(NFM, PC, Epilogue::kBf16, true, true);  \
  else if (bias != nullptr) JQ_F6(NFM, PC, Epilogue::kBf16, true, false);            \
  else JQ_F6(NFM, PC, Epilogue::kBf16, false, false);
  switch (bands) {
    case 4: JQ_F6_EPI(4, 2) break;
    case 5: JQ_F6_EPI(5, 1) break;
    case 6: JQ_F6_EPI(6, 1) break;
    case 7: JQ_F6_EPI(7, 1) break;
    default: JQ_F6_EPI(8, 1) break;
  }
#undef JQ_F6_EPI
#undef JQ_F6
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Library-held scratch of the allocation-free entry point
// (jq_w4a4_f6_linear_noalloc): the BF6 activation operand and the scales of
// one call, JQ_NOALLOC_SCRATCH_BYTES at most.  Each device the library runs
// on holds its own copy until the process ends.  In host code the name is
// only a handle for hipGetSymbolAddress; kernels get the device address it
// returns, as they get a workspace.

static __device__ __align__(256) uint8_t scratch[JQ_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    // once per device, with that device current
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

}  // namespace jq
