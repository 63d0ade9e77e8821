// Types and constants shared by the BF6 kernels (f6.hip, f6_narrow.hip).
#ifndef JQ_F6_COMMON_H
#define JQ_F6_COMMON_H

#include <stdint.h>

namespace jq {
namespace f6_detail {

typedef int v8i __attribute__((ext_vector_type(8)));      // MFMA operand; dwords 0..5 used
typedef float v16f __attribute__((ext_vector_type(16)));  // a 32x32 MFMA result
typedef int v4i32 __attribute__((ext_vector_type(4)));
typedef int v2i32 __attribute__((ext_vector_type(2)));

constexpr int kFragBytes = 1536;             // one 32-row x 64-code fragment
constexpr uint32_t kOutside = 0x80000000u;   // a buffer offset past every operand: loads read as zero

}  // namespace f6_detail
}  // namespace jq

#endif  // JQ_F6_COMMON_H
