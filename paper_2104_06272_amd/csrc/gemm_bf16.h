// What the backward kernels of bf16 networks share: the matrix instruction, roundings and masks, and the argument block of
// the launch that runs both products of a layer in whole 256-wide tiles (backward_bf16.hip).
#pragma once
#include "gemm.h"

namespace ank {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f16v mfma_bf16(bf8 a, bf8 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi)
{
    bf2v v; v[0] = (__bf16)lo; v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// two ReLU outputs as bfloat16 in a word (never negative, never -0: relu() returns +0 for every non-positive input)
// -> 0xffff in the halves that are positive, i.e. not zero, and 0 in the others.  Packed 16-bit integer instructions:
// min(h, 1) is 0 or 1, and 0 - that is 0 or 0xffff.
__device__ __forceinline__ uint32_t positive_mask_pk(uint32_t w)
{
    uint32_t r;
    const uint32_t zero = 0u, one = 0x00010001u;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(w), "v"(one));
    asm("v_pk_sub_u16 %0, %1, %2" : "=v"(r) : "v"(zero), "v"(r));
    return r;
}

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
// row j of the head matrix, eight entries (zero past NH)
__device__ __forceinline__ u4v head_row(const uint16_t* wh16, int NH, int j)
{
    uint32_t w8[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w8[k] = (uint32_t)wh16[(size_t)j * NH + (k < NH ? k : 0)];
#pragma unroll
    for (int k = 0; k < 8; ++k) w8[k] = k < NH ? w8[k] : 0u;
    u4v r; r[0] = w8[0] | (w8[1] << 16); r[1] = w8[2] | (w8[3] << 16); r[2] = w8[4] | (w8[5] << 16); r[3] = w8[6] | (w8[7] << 16);
    return r;
}

typedef short s2v __attribute__((ext_vector_type(2)));
// the flags of pair P of a ReLU mask word (relu_mask_bit: low half in bit P, high half in bit 16 + P) as 0xffff / 0 in the halves
__device__ __forceinline__ uint32_t mask_pair(uint32_t w, int P)
{
    const s2v v = __builtin_bit_cast(s2v, w) << (short)(15 - P);
    return __builtin_bit_cast(uint32_t, v >> (short)15);
}

struct BwdBf16Args {
    int M, K, N, NH, NHP;         // samples (a multiple of 32), inputs and outputs of the layer (multiples of 256), head outputs
    int splits, ranges;           // chunks of the dW product; row ranges of the dX product
    int rev;                      // samples from the last to the first
    int tiles_i, tiles, tn_blocks;
    const uint16_t* xP;           // packed h_{l-1}: [M/8][K][8]
    const uint16_t* dyP;          // packed dZ_l: [M/8][N][8] (not the top layer)
    const uint16_t* hTop;         // top layer: packed h_L [M/8][N][8]
    const uint32_t* maskTop;      // top layer: ReLU mask words of h_L (relu_mask_index)
    const uint32_t* maskLo;       // ReLU mask words of h_{l-1}, or null: the mask is then taken from xP
    const float* dhead;           // [M][NHP]
    const uint16_t* wh16;         // bf16 copy of Wh: [N][NH]
    const uint16_t* w16;          // [K][N]
    uint16_t* dxP;                // packed dZ_{l-1}: [M/8][K][8]
    float* partial;               // [splits][split_stride]: K x N partial, then the N column sums
    size_t split_stride;
    float* head_partial;          // [splits][head_stride]: N x NH partial of dWh, then dbh
    size_t head_stride;
};
hipError_t launch_backward_bf16_tiles(BwdBf16Args a, bool top, bool dx, hipStream_t s);

}  // namespace ank
