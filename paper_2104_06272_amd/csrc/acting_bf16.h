// Pieces that the acting kernels of bf16 nets share: operand types, rounding, arguments.
#pragma once
#include "internal.h"

namespace ank {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int BWG = 512;                // threads per workgroup: two wavefronts per SIMD
constexpr int BOBS = 12;                // observation words per env (as in the fp32 kernels)

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32v2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return bf16_to_f(h); }
// two floats rounded to bfloat16 (round to nearest even), low half first
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    bf2 v;
    v[0] = (__bf16)lo; v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float relu(float x) { return x > 0.0f ? x : 0.0f; }
// two packed ReLU outputs (never negative, never -0) -> 1 in bit 0 resp. bit 16 where the half is not zero
__device__ __forceinline__ uint32_t nonzero_flags_pk(uint32_t w)
{
    uint32_t r;
    const uint32_t one = 0x00010001u;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(w), "v"(one));
    return r;
}

struct RolloutBf16Args {
    EnvDims env;
    NetShape net;
    TrajPtrs tp;                         // tp.act[] point to bf16 buffers here
    const float* theta;                  // fp32 master (biases are read from here)
    const uint16_t* w;                   // bf16 copy of theta, same indexing
    const uint16_t* wt;                  // bf16 copy in matrix-core operand tiles (heads: [NH][HL])
    int B, T, ldx;                       // ldx: LDS row stride in bf16 elements
    int keep_acts;                       // store the packed hidden activations for the update
    int tend, tseg;                      // REPLAY: steps evaluated (T, or T + 1 with the bootstrap state), steps per workgroup (grid y)
    uint64_t seed, gstep;
};

// what: 0 the acting unroll, 1 the actor of a decoupled step, 2 the learner's replay
void fill_bf16_args(anakin* h, int what, RolloutBf16Args& a);
bool pinned_bf16_ok(const anakin* h);
hipError_t launch_pinned_bf16(anakin* h, int what);

}  // namespace ank
