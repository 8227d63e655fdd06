// Pieces that the fp32 acting kernels share: 16-byte loads, the observation words in LDS, the maze's wall sums.
#pragma once
#include "internal.h"

namespace ank {

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float bfr(float x) { return bf16_to_f(bf16_bits(x)); }

template <bool BF>
__device__ __forceinline__ float4 ldw4(const float* p)
{
    float4 w = ld4(p);
    if (BF) { w.x = bfr(w.x); w.y = bfr(w.y); w.z = bfr(w.z); w.w = bfr(w.w); }
    return w;
}

// per-env observation descriptor in LDS: 12 words per env
//   Catch: [0] ball cell, [1] paddle cell;  Pendulum: [0..2] = (cos, sin, theta_dot) as floats;
//   Maze: [0..7] wall words, [8] agent cell
constexpr int OBS_WORDS = 12;

// Maze: pre[TM][H1] = b1 + the wall rows of the environment's maze, cells ascending -- the part of the first layer
// that never changes within a launch.  The dense scan of the wall plane used to run in every step of the unroll (14 of
// 15 us per step of the 117-cell maze with a 128-64 net); it now runs once per launch, and the sums stay in LDS in the
// canonical order, so the logits are the same bits.
//
// A thread takes an environment and four columns and reads the rows of the cells that are walls, found bit by bit, sixteen
// in flight; a missing one is a load past the end of the buffer, which is zero and reads nothing.  (Every row read and
// masked, eight in flight, took 7 of the 61 us of an unroll with the 9 x 13 maze's 128-64 net, this 2; scalar loops over a wavefront's environment as long: this code
// runs once per launch, and instructions that were not fetched yet cost more than what they do.)
template <bool BF, int NTHR>
__device__ __forceinline__ void maze_prefix(const RolloutArgs& a, int TM, const uint32_t* __restrict__ obs, const float* __restrict__ w1,
                                            const float* __restrict__ b1, float* __restrict__ pre, int tid)
{
    typedef float f4v __attribute__((ext_vector_type(4)));
    const int N = a.net.dims[1], n = a.env.rows * a.env.cols, groups = TM * N / 4, lg4 = 29 - __builtin_clz((uint32_t)N);
    constexpr int CB = 16;                                       // weight rows in flight
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w1), 0, (uint32_t)(n * N) * 4u, 0x00020000);
#pragma unroll 1
    for (int i = tid; i < groups; i += NTHR) {
        const int c0 = (i & ((1 << lg4) - 1)) << 2, m = i >> lg4;
        f4v acc = *reinterpret_cast<const f4v*>(b1 + c0);
#pragma unroll 1
        for (int cb = 0; cb < n; cb += 64) {
            uint64_t bits = obs[m * OBS_WORDS + (cb >> 5)] | (uint64_t)obs[m * OBS_WORDS + (cb >> 5) + 1] << 32;   // bits past the last cell are zero
#pragma unroll 1
            while (bits) {
                f4v w[CB];
#pragma unroll
                for (int u = 0; u < CB; ++u) {
                    const uint32_t off = bits ? (uint32_t)((cb + __builtin_ctzll(bits)) * N + c0) * 4u : 0xffffffffu;
                    w[u] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
                    bits &= bits - 1u;
                }
#pragma unroll
                for (int u = 0; u < CB; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += BF ? bfr(w[u][e]) : w[u][e];
            }
        }
        *reinterpret_cast<f4v*>(pre + m * N + c0) = acc;
    }
}

}  // namespace ank
