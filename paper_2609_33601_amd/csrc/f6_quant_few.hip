// BF6 quantisers for few rows: the layouts, codes and scales (per token or
// per group) of quantize_rows4_f6_kernel in f6.hip, byte for byte.
// f6_quantize_few_rows says which inputs go here, f6_quantize_few_batch which
// batches.
//
// What bounds few rows.  Four rows per block of 32 codes per lane leave 64
// rows to 16 blocks, on the two XCDs their bands belong to, and each lane
// works through up to 96 codes one after the other: 16.8 us for 64 x 12288,
// of which the bytes need less than one.  Here a block takes one row and a
// lane eight codes at a time, so a row of 4096 is one load, one maximum and
// one conversion deep, and the rows go round the XCDs.  What is left is the
// launch and one trip to memory (4.5 us back to back, the same as for one
// short row).  Measured: 64 x 4096 7.0 -> 4.7 us, 64 x 12288 16.8 -> 5.5 us,
// 512 x 12288 13.7 -> 10.8 us, group128 33 x 12288 12.8 -> 6.0 us.  From
// about 1024 rows the wider stores of the four-row kernel win (1024 x 4096
// 5.9 against 8.7 us): a quarter of the lanes store here.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "f6_common.h"
#include "jq_internal.h"

namespace jq {

namespace {

using namespace f6_detail;

typedef unsigned v4u32 __attribute__((ext_vector_type(4)));

constexpr int64_t kFewRows = 512;
constexpr int64_t kFourRowsMaxK = 16384;  // the four-row kernel's longest row

// The lane's value of v at lane perm[l % 4] of its quad (CTRL as in quad_perm).
template <int CTRL>
__device__ __forceinline__ uint32_t quad(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xF, 0xF, true));
}
constexpr int kNext = 0xF9;   // lanes 1 2 3 3
constexpr int kNext2 = 0xFE;  // lanes 2 3 3 3

__device__ __forceinline__ uint32_t max8(v4u32 t) {
  u16x2 a = __builtin_bit_cast(u16x2, t.x & 0x7FFF7FFFu);
  a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, t.y & 0x7FFF7FFFu));
  a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, t.z & 0x7FFF7FFFu));
  a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, t.w & 0x7FFF7FFFu));
  return a.x > a.y ? a.x : a.y;
}

template <int FROM, int TO>
__device__ __forceinline__ uint32_t lanes_max(uint32_t v) {
#pragma unroll
  for (int off = FROM; off >= TO; off >>= 1) {
    const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), off, 64));
    v = v > o ? v : o;
  }
  return v;
}

// One row of an operand per block: thread t takes the 8-code chunks
// t + blockDim.x * j, j < nc <= NC, and keeps them in registers between the
// maximum and the conversion.  Four neighbouring lanes hold a group of 32
// codes, 48 bits each, and put its six dwords together: lane 0 stores d0..d3,
// lane 2 d4 and d5.  Chunks past K and rows past M load the first chunk of x
// and are zeroed (no branch between the loads).
template <int NC, int G>
__device__ __forceinline__ void few_row(const uint16_t* __restrict__ x, int64_t M, int64_t K, int64_t ksteps,
                                        uint8_t* __restrict__ out, float* __restrict__ scale, int64_t row, int nc) {
  __shared__ uint32_t wave_max[16];
  const int T = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool live = row < M;
  const int chunks = static_cast<int>(8 * ksteps);
  const uint16_t* xr = x + (live ? row : 0) * K;
  v4u32 v[NC];
  uint32_t cmax[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    if (j >= nc) break;
    const int64_t e = 8 * static_cast<int64_t>(T * j + tid);
    const bool ok = live && e < K;
    v[j] = __builtin_nontemporal_load(reinterpret_cast<const v4u32*>(ok ? xr + e : x));
    if (!ok) v[j] = v4u32{0, 0, 0, 0};
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) cmax[j] = j < nc ? max8(v[j]) : 0;

  float srow = 0.0f, rrow = 0.0f;
  if constexpr (G == 0) {
    uint32_t amax = cmax[0];
#pragma unroll
    for (int j = 1; j < NC; ++j) amax = amax > cmax[j] ? amax : cmax[j];
    amax = lanes_max<32, 1>(amax);
    if (T > 64) {
      if (lane == 0) wave_max[wave] = amax;
      __syncthreads();
      const int w = lane & 15;
      amax = lanes_max<8, 1>(w < (T >> 6) ? wave_max[w] : 0);
    }
    // Non-negative floats order like their bit patterns.
    srow = __uint_as_float(amax << 16) / 7.0f;
    if (live && tid == 0) scale[row] = srow;
    rrow = srow == 0.0f ? 0.0f : 1.0f / srow;
  } else {
    (void)wave_max;
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    if (j >= nc) break;
    const int c = T * j + tid;
    float s = srow, rcp = rrow;
    if constexpr (G != 0) {
      s = __uint_as_float(lanes_max<G / 16, 1>(cmax[j]) << 16) / 7.0f;
      rcp = s == 0.0f ? 0.0f : 1.0f / s;
      if (live && c % (G / 8) == 0 && 8 * static_cast<int64_t>(c) < K) scale[row * (K / G) + c / (G / 8)] = s;
    }
    // Codes by the reciprocal, and by the division for the whole group of 32
    // where one of its codes sits next to a rounding decision point or the
    // reciprocal overflows (as codes32 in f6.hip).
    const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
    float q[8];
    float dmax = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float te = bf16_lo(w[i]) * rcp, to = bf16_hi(w[i]) * rcp;
      const float re = (te + kMagic) - kMagic, ro = (to + kMagic) - kMagic;
      dmax = fmaxf(dmax, fmaxf(fabsf(te - re), fabsf(to - ro)));
      q[2 * i] = re;
      q[2 * i + 1] = ro;
    }
    const bool mine = !(dmax < kNearTie) || __builtin_isinf(rcp);
    const uint64_t quads = 0xFull << (lane & 60);
    if ((__ballot(mine) & quads) != 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        q[2 * i] = fminf(fmaxf(__builtin_rintf(bf16_lo(w[i]) / s), -8.0f), 7.0f);
        q[2 * i + 1] = fminf(fmaxf(__builtin_rintf(bf16_hi(w[i]) / s), -8.0f), 7.0f);
      }
    }
    if (s == 0.0f) {
#pragma unroll
      for (int i = 0; i < 8; ++i) q[i] = 0.0f;
    }
    // Fields 0..7 of the converter's 32 (it interleaves its two sources).
    v16f even, odd;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      even[i] = q[2 * (i & 3)];
      odd[i] = q[2 * (i & 3) + 1];
    }
    const v6u f = __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(even, odd, 1.0f);
    // Lane k of the quad holds bits 48k .. 48k + 47 of the group: lo, hi.
    const uint32_t lo = f[0], hi = f[1] & 0xFFFFu;
    const uint32_t d14 = hi | (quad<kNext>(lo) << 16);             // lane 0: d1, lane 2: d4
    const uint32_t d25 = quad<kNext>((lo >> 16) | (hi << 16));     // lane 0: d2, lane 2: d5
    const uint32_t d3 = quad<kNext2>(lo);                          // lane 0: d3
    if (c >= chunks) continue;
    const int gi = c >> 2;
    const int L = static_cast<int>(row & 31) + 32 * (gi & 1);
    uint8_t* p = out + ((row >> 5) * ksteps + (gi >> 1)) * kFragBytes;
    if ((c & 3) == 0) *reinterpret_cast<uint4*>(p + 16 * L) = make_uint4(lo, d14, d25, d3);
    if ((c & 3) == 2) *reinterpret_cast<uint2*>(p + 1024 + 8 * L) = make_uint2(d14, d25);
  }
}

template <int NC, int G>
__global__ __launch_bounds__(1024) void quantize_few_f6_kernel(const uint16_t* __restrict__ x, int64_t M, int64_t K,
                                                               int64_t ksteps, uint8_t* __restrict__ out,
                                                               float* __restrict__ scale) {
  few_row<NC, G>(x, M, K, ksteps, out, scale, blockIdx.x, NC);
}

// Several inputs in one launch: input i takes the blocks from first[i] on.
struct FewInput {
  const uint16_t* x;
  uint8_t* out;
  float* scale;
  int64_t M, K, ksteps, first;
  int nc;
};
struct FewBatch {
  FewInput in[kQuantBatchMax];
  int count;
};

template <int NC>
__global__ __launch_bounds__(1024) void quantize_few_f6_batch_kernel(FewBatch b) {
  int i = 0;
  while (i + 1 < b.count && static_cast<int64_t>(blockIdx.x) >= b.in[i + 1].first) ++i;
  const FewInput& e = b.in[i];
  few_row<NC, 0>(e.x, e.M, e.K, e.ksteps, e.out, e.scale, blockIdx.x - e.first, e.nc);
}

// 512 threads (1024 for rows of more than 16384 codes), fewer for short rows.
int threads_for(int64_t chunks) {
  const int64_t most = chunks > 2048 ? 1024 : 512;
  return static_cast<int>(std::min<int64_t>(most, (chunks + 63) / 64 * 64));
}

template <int G>
hipError_t launch_few(const uint16_t* x, int64_t M, int64_t K, uint8_t* out, float* scale, hipStream_t st) {
  const int64_t ksteps = f6_ksteps(K), chunks = 8 * ksteps;
  const int t = threads_for(chunks);
  const int64_t nc = (chunks + t - 1) / t;
  const dim3 grid(static_cast<unsigned>((M + 31) / 32 * 32));
#define JQ_FEW(NN) hipLaunchKernelGGL((quantize_few_f6_kernel<NN, G>), grid, dim3(t), 0, st, x, M, K, ksteps, out, scale)
  if (nc <= 1) JQ_FEW(1);
  else if (nc <= 2) JQ_FEW(2);
  else if (nc <= 3) JQ_FEW(3);
  else if (nc <= 4) JQ_FEW(4);
  else if (nc <= 6) JQ_FEW(6);  // (as 8, loads of nothing made 96 x 49152 13.9 us, against 13.4 by the one-row kernel)
  else JQ_FEW(8);
#undef JQ_FEW
  return hipGetLastError();
}

}  // namespace

// Rows of up to 16384 codes: against the four-row kernel this one is 15 to 60%
// faster up to 512 rows (G 0, 64 and 128, K 64..16384); from 1024 rows on it is
// slower.  Longer rows go to the one-row kernel of f6.hip otherwise, which reads
// them with 512 threads instead of 1024: per token it is faster or level for
// fewer than 32 rows (2 x 49152 8.7 against 9.8 us) and for more than 160 (384 x
// 65536 28.6 against 38.4), between them 2 to 35% slower; with group scales,
// which need no maximum over the row, it is faster from 16 rows on (256 x 20480
// 7.5 against 10.1, 512 x 20480 11.5 against 17.3) and up to 4 rows slower by 5
// to 40%.
bool f6_quantize_few_rows(int64_t M, int64_t K, int G) {
  if (K <= kFourRowsMaxK) return M <= kFewRows;
  return G == 0 ? M >= 32 && M <= 160 : M <= 4;
}

// Whether a batch takes one launch of the few-row kernel, by estimated times in
// ns.  The few-row kernel: 2300, 1 per 900 codes and half of one per row, at
// least the walk along the longest row.  Otherwise the inputs of up to 16384
// codes a row share a launch of the four-row kernel, whose blocks start every
// input on XCD 0: the walk (0.6 per code of the longest row) and the codes of
// that XCD (x 8, at 1300) overlap in part; and longer rows take a launch of
// their own each.  Fitted to 180 batches and 110 single inputs (1..8 inputs, M
// 1..512, K 64..16384, some to 65536): 0.1% off the better of the two on
// average.  (8 x 128 x 4096 11.1 us by the four-row kernel, 8.7 by this one; 4 x
// 512 x 4096 10.0 and 14.5.)
bool f6_quantize_few_batch(int count, const int64_t* M, const int64_t* K) {
  int64_t rows = 0, codes = 0, longest = 0, four_longest = 0, xcd_codes = 0, apart = 0;
  for (int i = 0; i < count; ++i) {
    if (M[i] > kFewRows) return false;
    rows += M[i];
    codes += M[i] * K[i];
    longest = std::max(longest, K[i]);
    if (K[i] <= kFourRowsMaxK) {
      four_longest = std::max(four_longest, K[i]);
      xcd_codes += (M[i] < 32 ? M[i] : (M[i] + 255) / 256 * 32) * K[i];
    } else {
      apart += std::max(3000 + K[i] * 1000 / 8192, 3000 + M[i] * K[i] / 1000);
    }
  }
  const int64_t few = std::max(2500 + longest * 1000 / 8192, 2300 + codes / 900 + rows / 2);
  int64_t other = apart;
  if (four_longest > 0) {
    const int64_t walk = 3400 + four_longest * 6 / 10, load = 1000 + 8 * xcd_codes / 1300;
    other += std::max(walk, load) + std::min(walk, load) * 3 / 10;
  }
  return few <= other;
}

hipError_t launch_quantize_few_f6(const uint16_t* x, int64_t M, int64_t K, int G, uint8_t* out, float* scale,
                                  hipStream_t st) {
  if (G == 64) return launch_few<64>(x, M, K, out, scale, st);
  if (G == 128) return launch_few<128>(x, M, K, out, scale, st);
  return launch_few<0>(x, M, K, out, scale, st);
}

hipError_t launch_quantize_few_f6_batch(int count, const uint16_t* const* x, const int64_t* M, const int64_t* K,
                                        uint8_t* const* out, float* const* scale, hipStream_t st) {
  FewBatch b{};
  int t = 64;
  for (int i = 0; i < count; ++i) t = std::max(t, threads_for(8 * f6_ksteps(K[i])));
  int64_t first = 0;
  int NC = 1;
  for (int i = 0; i < count; ++i) {
    FewInput& e = b.in[b.count++];
    e.x = x[i];
    e.out = out[i];
    e.scale = scale[i];
    e.M = M[i];
    e.K = K[i];
    e.ksteps = f6_ksteps(K[i]);
    e.first = first;
    e.nc = static_cast<int>((8 * e.ksteps + t - 1) / t);
    NC = std::max(NC, e.nc);
    first += (M[i] + 31) / 32 * 32;
  }
  const dim3 grid(static_cast<unsigned>(first));
#define JQ_FEWB(NN) hipLaunchKernelGGL((quantize_few_f6_batch_kernel<NN>), grid, dim3(t), 0, st, b)
  if (NC <= 1) JQ_FEWB(1);
  else if (NC <= 2) JQ_FEWB(2);
  else if (NC <= 3) JQ_FEWB(3);
  else if (NC <= 4) JQ_FEWB(4);
  else JQ_FEWB(8);
#undef JQ_FEWB
  return hipGetLastError();
}

}  // namespace jq
