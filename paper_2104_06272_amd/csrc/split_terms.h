// A binary32 value as three packed bfloat16 terms, and the weights of the fp32 backward products in that form (gemm_split.hip
// says why and how they are used).
#pragma once
#include "gemm.h"

namespace ank {

// LDS between the lanes of one wavefront: its accesses are carried out in order, only the compiler has to keep that order
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef __bf16 bf8_s __attribute__((ext_vector_type(8)));
typedef __bf16 bf2_s __attribute__((ext_vector_type(2)));
typedef float f16v_s __attribute__((ext_vector_type(16)));
typedef float f4v_s __attribute__((ext_vector_type(4)));
typedef uint32_t u4v_s __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pk_bf16_s(float lo, float hi)
{
    bf2_s v; v[0] = (__bf16)lo; v[1] = (__bf16)hi;               // round to nearest even, one instruction for the pair
    return __builtin_bit_cast(uint32_t, v);
}
// Pair i of eight values as three packed terms, t[0] + t[1] + t[2] = x exactly where x is 0 or 2^-102 <= |x| <= 3.3895e38
// (the largest bfloat16).  Below, the last terms fall under the smallest normal bfloat16 and may be lost: up to 2^-126 per
// term, whatever is left of values that a gradient's sum does not see.  Above, the first term is infinite and the remainder
// is not a number, so a sum with such an operand is NaN (where a binary32 product could still be finite).  An activation or
// a gradient there is a sum about to overflow; a weight can stand there for good -- the type's lowest value as the mask of a
// unit that never fires, whose gradient of 0 it meets in the product -- so weights take WHOLE: the first term no larger
// than the largest bfloat16, the rest of up to 1.4e36 left to the others, exact up to 3.4028e38.  (The partial products reach
// infinity when the sum is within 1 % of it.)  An infinite x is NaN in either form, and NaN stays NaN.
template <bool WHOLE = false>
__device__ __forceinline__ void split_pair(float x0, float x1, u4v_s (&t)[3], int i)
{
    constexpr float big = 0x1.fep127f;
    uint32_t p = WHOLE ? pk_bf16_s(__builtin_amdgcn_fmed3f(x0, -big, big), __builtin_amdgcn_fmed3f(x1, -big, big)) : pk_bf16_s(x0, x1);
    asm("" : "+v"(p));                                           // else the low half is rounded a second time on its own
    t[0][i] = p;
    const float r0 = x0 - f_from_bits(p << 16), r1 = x1 - f_from_bits(p & 0xffff0000u);
    uint32_t q = pk_bf16_s(r0, r1);
    asm("" : "+v"(q));
    t[1][i] = q;
    t[2][i] = pk_bf16_s(r0 - f_from_bits(q << 16), r1 - f_from_bits(q & 0xffff0000u));
}
template <bool WHOLE = false>
__device__ __forceinline__ void split_terms(const float (&x)[8], u4v_s (&t)[3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair<WHOLE>(x[2 * i], x[2 * i + 1], t, i);
}
// Weights as the B operand of gemm_nt: for every block of 32 rows i of W[K][N] and every step of 16 reduction indices j
// the three terms of the 64 lanes' 16-byte pieces, one KiB each: piece ((ib * N/16 + ks) * 3 + term) * 64 + lane.
// The kernels that take the loss have a few workgroups more for this: as a launch of its own it took 3 us of an update.
inline int split_weights_blocks(const SplitWeightsArgs& a)
{
    int pieces = 0;
    for (int l = 0; l < a.n; ++l) pieces += a.K[l] * a.N[l] / 8;
    return (pieces + WG - 1) / WG;
}
__device__ __forceinline__ void split_weights(const SplitWeightsArgs& a, int block)
{
    int p = block * WG + (int)threadIdx.x;                       // piece: eight consecutive j of one row i
    for (int l = 0; l < a.n; ++l) {
        const int pieces = a.K[l] * a.N[l] / 8;
        if (p >= pieces) { p -= pieces; continue; }
        const int ng = a.N[l] / 8, i = p / ng, jg = p % ng;
        const f4v_s* src = reinterpret_cast<const f4v_s*>(a.w[l] + (size_t)i * a.N[l] + 8 * jg);
        const f4v_s v0 = src[0], v1 = src[1];
        const float x[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
        u4v_s t[3];
        if (a.bf16) {                                            // a bf16 net's weights are rounded: the first term alone
            split_terms(x, t);
#pragma unroll
            for (int i = 0; i < 4; ++i) { t[1][i] = 0; t[2][i] = 0; }
        } else split_terms<true>(x, t);
        u4v_s* dst = reinterpret_cast<u4v_s*>(a.out[l]) + ((size_t)((i >> 5) * (a.N[l] >> 4) + (jg >> 1)) * 3) * 64 + 32 * (jg & 1) + (i & 31);
#pragma unroll
        for (int k = 0; k < 3; ++k) dst[k * 64] = t[k];
        return;
    }
}

}  // namespace ank
