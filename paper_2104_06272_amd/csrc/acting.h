// Pieces that the fp32 acting kernels share: 16-byte loads, the observation words in LDS, the maze's wall sums.
#pragma once
#include "internal.h"

namespace ank {

typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float bfr(float x) { return bf16_to_f(bf16_bits(x)); }

template <bool BF>
__device__ __forceinline__ float4 ldw4(const float* p)
{
    float4 w = ld4(p);
    if (BF) { w.x = bfr(w.x); w.y = bfr(w.y); w.z = bfr(w.z); w.w = bfr(w.w); }
    return w;
}
// BF: two values rounded to bfloat16 in place, by the conversion instruction (bfr's bits for every finite value)
template <bool BF>
__device__ __forceinline__ void round2(float& a, float& b)
{
    if (!BF) return;
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    b2 v;
    v[0] = (__bf16)a; v[1] = (__bf16)b;
    const uint32_t p = __builtin_bit_cast(uint32_t, v);
    a = f_from_bits(p << 16); b = f_from_bits(p & 0xffff0000u);
}
template <bool BF, class V>
__device__ __forceinline__ void round4(V& v)
{
    float a = v[0], b = v[1], c = v[2], d = v[3];
    round2<BF>(a, b); round2<BF>(c, d);
    v[0] = a; v[1] = b; v[2] = c; v[3] = d;
}
template <bool BF>
__device__ __forceinline__ float round1(float x) { return BF ? bfr(x) : x; }

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

// lane Q of each row of 16 lanes, in all of them
template <int Q>
__device__ __forceinline__ float row_lane(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + Q, 0xf, 0xf, true)); }
template <int Q>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + Q, 0xf, 0xf, true); }

// Sample and step of an environment that a row of 16 lanes owns, lane j holding head j; all lanes of the row do the same.
// dr: the step's draws, wl: the maze's walls.
template <int ENV>
__device__ __forceinline__ void row_step(const EnvDims& env, EnvState& st, float sine, float hv, const uint4 dr, const uint32_t* wl,
                                         float& eps, float& actf, int& act, float& rew, int& done)
{
    constexpr int A = ENV == ENV_CATCH ? 3 : 4;
    if (ENV == ENV_PENDULUM) {
        eps = f_from_bits(dr.x);
        actf = gaussian_action(row_lane<0>(hv), row_lane<1>(hv), eps);
        pendulum_step_sn(env, st, sine, actf, dr.z, dr.w, rew, done);
    } else {
        const float l0 = row_lane<0>(hv), l1 = row_lane<1>(hv), l2 = row_lane<2>(hv), l3 = A > 3 ? row_lane<3>(hv) : 0.0f;
        float mx = l0;
        mx = l1 > mx ? l1 : mx;
        mx = l2 > mx ? l2 : mx;
        if (A > 3) mx = l3 > mx ? l3 : mx;
        const float ex = det_exp(hv - mx);                     // lane j: the exponential of logit j
        const float c0 = row_lane<0>(ex), c1 = c0 + row_lane<1>(ex), c2 = c1 + row_lane<2>(ex), c3 = A > 3 ? c2 + row_lane<3>(ex) : c2;
        const float thr = u01(dr.x) * c3;
        act = A - 1;
        if (A > 3 && c2 > thr) act = 2;
        if (c1 > thr) act = 1;
        if (c0 > thr) act = 0;
        if (ENV == ENV_CATCH) catch_step(env, st, act, dr.z, rew, done);
        else maze_step(env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, rew, done);
    }
}

// acc += sum over 16 k of x[row's lane k] * w[k], k ascending, one fused multiply-add each.  (As one block: between single
// statements the compiler puts a wait state each.  The leading wait is what a DPP operand needs after a vector write.)
__device__ __forceinline__ void chain16(float x, f4v w0, f4v w1, f4v w2, f4v w3, float& acc)
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(x), "v"(w0[0]), "v"(w0[1]), "v"(w0[2]), "v"(w0[3]), "v"(w1[0]), "v"(w1[1]), "v"(w1[2]), "v"(w1[3]), "v"(w2[0]), "v"(w2[1]), "v"(w2[2]), "v"(w2[3]), "v"(w3[0]), "v"(w3[1]), "v"(w3[2]), "v"(w3[3]));
}

// the same over eight of the row's lanes, LO .. LO + 7
template <int LO>
__device__ __forceinline__ void chain8(float x, f4v w0, f4v w1, float& acc)
{
    static_assert(LO == 0 || LO == 8, "half a row");
#define ANK_CHAIN8(a, b, c, d, e, f, g, h) \
    asm("s_nop 1\n\t" \
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:" #a " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:" #b " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:" #c " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:" #d " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:" #e " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:" #f " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:" #g " row_mask:0xf bank_mask:0xf\n\t" \
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:" #h " row_mask:0xf bank_mask:0xf" \
        : "+v"(acc) : "v"(x), "v"(w0[0]), "v"(w0[1]), "v"(w0[2]), "v"(w0[3]), "v"(w1[0]), "v"(w1[1]), "v"(w1[2]), "v"(w1[3]))
    if (LO == 0) ANK_CHAIN8(0, 1, 2, 3, 4, 5, 6, 7);
    else ANK_CHAIN8(8, 9, 10, 11, 12, 13, 14, 15);
#undef ANK_CHAIN8
}

}  // namespace ank
