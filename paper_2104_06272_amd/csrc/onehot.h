// The 0/1 board as an operand of the matrix instruction, two samples to a register (first_layer.hip, learn_one.hip).
#pragma once
#include "split_terms.h"

namespace ank {

typedef uint16_t us2_f __attribute__((ext_vector_type(2)));

// 1.0 (bfloat16) in each half of c that is zero.  `ones` is 1 in both halves, from a register that the compiler cannot see
// through: it would turn the saturating subtraction into compares and selects of single halves.
__device__ __forceinline__ uint32_t one_where_zero(uint32_t c, uint32_t ones)
{
    const us2_f bf1 = {0x3f80, 0x3f80};
    const us2_f m = __builtin_elementwise_sub_sat(__builtin_bit_cast(us2_f, ones), __builtin_bit_cast(us2_f, c));
    return __builtin_bit_cast(uint32_t, (us2_f)(m * bf1));
}
__device__ __forceinline__ uint32_t min_pair(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2_f, a), __builtin_bit_cast(us2_f, b)));
}
__device__ __forceinline__ f16v_s mfma_f(u4v_s a, u4v_s b, f16v_s c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8_s, a), __builtin_bit_cast(bf8_s, b), c, 0, 0, 0);
}

}  // namespace ank
