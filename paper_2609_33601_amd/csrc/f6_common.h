// Types and constants shared by the BF6 kernels (f6.hip, f6_narrow.hip).
#ifndef JQ_F6_COMMON_H
#define JQ_F6_COMMON_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jq {
namespace f6_detail {

typedef int v8i __attribute__((ext_vector_type(8)));      // MFMA operand; dwords 0..5 used
typedef float v16f __attribute__((ext_vector_type(16)));  // a 32x32 MFMA result
typedef int v4i32 __attribute__((ext_vector_type(4)));
typedef int v2i32 __attribute__((ext_vector_type(2)));
typedef unsigned v6u __attribute__((ext_vector_type(6)));  // a 32-code group
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int kFragBytes = 1536;             // one 32-row x 64-code fragment
constexpr uint32_t kOutside = 0x80000000u;   // a buffer offset past every operand: loads read as zero
constexpr int kQuantBatchMax = 8;            // inputs of one batched quantiser launch

// The quantisers' rounding: t + kMagic rounds t to an integer in the fp32
// adder, and codes with |t - rne(t)| at or above kNearTie take the division.
constexpr float kMagic = 12582912.0f;        // 1.5 * 2^23
constexpr float kNearTie = 0.5f - 0x1p-17f;

// acc + a b for two BF6 fragments (format 3).  With both scale operands the
// constant 0 the builtin is v_mfma_f32_32x32x64_f8f6f4, which takes no scales;
// with 127 (a scale of 1) it is v_mfma_scale_..., which also loads a scale per
// operand: 16 bytes of code instead of 8 and an issue slot more per MFMA, for
// the same sums.
__device__ __forceinline__ v16f mfma_bf6(const v8i& a, const v8i& b, const v16f& acc) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 3, 3, 0, 0, 0, 0);
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

}  // namespace f6_detail
}  // namespace jq

#endif  // JQ_F6_COMMON_H
