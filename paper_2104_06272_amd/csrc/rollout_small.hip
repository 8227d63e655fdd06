// Acting for two layers of 64 units at small batches (paper section 3.1, the persistent unroll): one wavefront owns four
// environments for the whole unroll and passes nothing to any other.
//
// A step of such a net is latency only.  Spread over four wavefronts (rollout_resident64_kernel) it took 3.6 k cycles, of which
// the layer on the matrix cores was 0.5 k: four barriers, and between them hand-overs of observations, activations and heads
// through LDS.  Here the whole chain stays in one wavefront's registers:
//  - the hidden matrix is one register per input, its column the lane; v_mfma_f32_4x4x1 multiplies it with four environments,
//    chained along the inputs as the canonical order wants (12.5 cycles each, 0.8 k for the layer);
//  - the first layer is taken straight into that instruction's A operand (lane 4 b + i: input 16 r + b of environment i), from
//    an LDS copy of its matrix whose columns are in that order;
//  - four lane swaps turn the layer's outputs (register: environment, lane: unit) into a row of 16 lanes per environment, whose
//    lane j sums head j out of registers by row broadcast (chain16), and in which every lane samples and steps.
// A fifth wavefront draws the next step's random numbers for the four, behind the one barrier of a step.
// Catch, 64 environments, T = 20: 31.8 -> 23.4 us an unroll, 2.7 k cycles a step.
#include "acting.h"

namespace ank {

constexpr int SMW = 4, SMT = 4 * SMW;            // acting wavefronts and environments of a workgroup

typedef __amdgpu_buffer_rsrc_t rsrc_sm;
typedef uint32_t u2_sm __attribute__((ext_vector_type(2)));

// rows of 16 lanes and the four registers change places: register s of row e becomes register e of row s
__device__ __forceinline__ void swap_rows(float (&r)[4])
{
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const u2_sm p = __builtin_bit_cast(u2_sm, __builtin_amdgcn_permlane32_swap(bits_from_f(r[u]), bits_from_f(r[u + 2]), false, false));
        r[u] = f_from_bits(p[0]); r[u + 2] = f_from_bits(p[1]);
    }
#pragma unroll
    for (int u = 0; u < 4; u += 2) {
        const u2_sm p = __builtin_bit_cast(u2_sm, __builtin_amdgcn_permlane16_swap(bits_from_f(r[u]), bits_from_f(r[u + 1]), false, false));
        r[u] = f_from_bits(p[0]); r[u + 1] = f_from_bits(p[1]);
    }
}
// a value that is the same in all lanes of a row: row lane % 4's, in every lane
__device__ __forceinline__ uint32_t row_of_quad(uint32_t v, int lane)
{
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return lane & 2 ? (lane & 1 ? d : c) : (lane & 1 ? b : a);
}

template <int KK>
__device__ __forceinline__ void layer16(float x, const float* w, f4v& acc)
{
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, w[KK], acc, 4, KK, 0);
    if constexpr (KK < 15) layer16<KK + 1>(x, w, acc);
}

template <int ENV>
__global__ __launch_bounds__(64 * (SMW + 1)) void rollout_small_kernel(const RolloutArgs a)
{
    constexpr int H = 64, NTHR = 64 * (SMW + 1);
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH > 4 ? 8 : 4;
    extern __shared__ float4 smem4[];
    uint32_t* rng = reinterpret_cast<uint32_t*>(smem4);            // [2][SMT][4] draws: the action's two words (pendulum: noise), the reset's
    uint32_t* obs = rng + 2 * SMT * 4;                             // maze: [SMT][OBS_WORDS] walls
    float* w1s = reinterpret_cast<float*>(obs + (ENV == ENV_MAZE ? SMT * OBS_WORDS : 0));   // first-layer rows (maze: the agent plane), columns 4 b + r: 16 r + b
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * SMT, B = a.B, T = a.T, cells = a.env.rows * a.env.cols;
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];
    const float* b1g = a.theta + a.net.b_off[0];
    float* pre = w1s + (ENV == ENV_MAZE ? cells * H : 0);          // maze: [SMT][H] wall sums, then biases [H]

    auto draw = [&](int t) {                                       // (the last wavefront)
        if (lane >= (ENV == ENV_MAZE ? SMT : 2 * SMT)) return;
        const int m = lane & (SMT - 1);
        const bool reset = lane >= SMT;
        const u32x4 w = philox(a.seed, (uint32_t)(b0 + m), a.gstep + (uint64_t)t, reset ? DOM_RESET : DOM_ACTION);
        const uint32_t w0 = (ENV == ENV_PENDULUM && !reset) ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;
        *reinterpret_cast<uint2*>(rng + ((t & 1) * SMT + m) * 4 + (reset ? 2 : 0)) = make_uint2(w0, w.y);
    };

    // ---- what an acting wavefront keeps in registers ----
    const int i = lane & 3, b = lane >> 2, e = lane >> 4, j = lane & 15;   // as A operand: environment, input % 16; as a row: environment, head
    const int row0 = 4 * (wave < SMW ? wave : 0);
    float w2[H], hw[H], b1v[4], wp[3][4];
    float b2 = 0.0f, hbias = 0.0f;
    EnvState st{0u, 0.0f, 0.0f};
    if (wave < SMW) {
#pragma unroll
        for (int k = 0; k < H; ++k) w2[k] = a.theta[a.net.w_off[1] + k * H + lane];
        const float* hs = a.theta + a.net.wh_off + (j < NH ? j : 0);
#pragma unroll
        for (int k = 0; k < H; ++k) hw[k] = hs[k * NH];
        b2 = a.theta[a.net.b_off[1] + lane];
        hbias = a.theta[a.net.bh_off + (j < NH ? j : 0)];
#pragma unroll
        for (int r = 0; r < 4; ++r) b1v[r] = b1g[16 * r + b];
        if (ENV == ENV_PENDULUM) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) wp[k][r] = w1g[k * H + 16 * r + b];
        } else if (ENV == ENV_MAZE) {
#pragma unroll
            for (int r = 0; r < 4; ++r) wp[0][r] = w1g[(size_t)(3 * cells - 1) * H + 16 * r + b];
        }
        st.s0 = tp.s0[b0 + row0 + e];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b0 + row0 + e]; st.f1 = tp.f1[b0 + row0 + e]; }
    } else draw(0);
    if (ENV != ENV_PENDULUM) {
        const float* src = w1g + (ENV == ENV_MAZE ? (size_t)cells * H : 0);
        const int n4 = cells * (H / 4);
        for (int p = tid; p < n4; p += NTHR) {                     // four consecutive columns of a row
            const f4v v = *reinterpret_cast<const f4v*>(src + 4 * (size_t)p);
            const int row = p / (H / 4), c = 4 * (p % (H / 4));
#pragma unroll
            for (int q = 0; q < 4; ++q) w1s[row * H + 4 * ((c + q) & 15) + (c >> 4)] = v[q];
        }
    }
    if (ENV == ENV_MAZE) {
        for (int p = tid; p < SMT * 8; p += NTHR) obs[(p >> 3) * OBS_WORDS + (p & 7)] = tp.walls[(size_t)(p & 7) * B + b0 + (p >> 3)];
        float* b1s = pre + SMT * H;
        if (tid < H) b1s[tid] = b1g[tid];
        __syncthreads();
        maze_prefix<false, NTHR>(a, SMT, obs, w1g, b1s, pre, tid);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) b1v[r] = pre[(row0 + i) * H + 16 * r + b];
    }
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0): inside the loop a wait for a load would be one for every older store

    if (wave == SMW) {
        for (int t = 0; t < T; ++t) {
            if (t + 1 < T) draw(t + 1);
            __syncthreads();
        }
        return;
    }
    float sine = 0.0f, hv = 0.0f, rew = 0.0f, actf = 0.0f, eps = 0.0f;
    int act = 0, done = 0;
    auto rsrc = [&](const void* p, bool on) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, on ? 0x7fffffffu : 0u, 0x00020000); };
    // records, as stores without branches (what is not to be written has a descriptor of no bytes); they go between the MFMAs,
    // whose chain leaves two thirds of the issue slots
    const int o4 = j == 0 ? 4 * e : -1, o1 = j == 0 ? e : -1;
    auto store_state = [&](int t) {
        const size_t te = (size_t)t * B + b0 + row0;
        __builtin_amdgcn_raw_buffer_store_b32(st.s0, rsrc(tp.tr_s0 + te, true), o4, 0, 0);
        if (ENV == ENV_PENDULUM) {
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f0), rsrc(tp.tr_f0 + te, true), o4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f1), rsrc(tp.tr_f1 + te, true), o4, 0, 0);
        }
    };
    auto store_heads = [&](int t, bool on) {
        const size_t te = (size_t)t * B + b0 + row0;
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(j < NH ? hv : 0.0f), rsrc(tp.tr_head + te * NHP, on), j < NHP ? 4 * (e * NHP + j) : -1, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(hv), rsrc(tp.tr_val + te, on), j == NH - 1 ? 4 * e : -1, 0, 0);
    };
    auto store_step = [&](int t, bool on) {
        const size_t te = (size_t)t * B + b0 + row0;
        if (ENV == ENV_PENDULUM) {
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(eps), rsrc(tp.tr_eps + te, on), o4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(actf), rsrc(tp.tr_actf + te, on), o4, 0, 0);
        } else __builtin_amdgcn_raw_buffer_store_b8((uint8_t)act, rsrc(tp.tr_act + te, on), o1, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(rew), rsrc(tp.tr_rew + te, on), o4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)done, rsrc(tp.tr_done + te, on), o1, 0, 0);
    };
    for (int t = 0; t <= T; ++t) {
        // ---- observe, first layer ----
        float x[4];
        if (ENV == ENV_PENDULUM) {
            float cs;
            det_sincos(st.f0, sine, cs);
            const float f[3] = {f_from_bits(row_of_quad(bits_from_f(cs), lane)), f_from_bits(row_of_quad(bits_from_f(sine), lane)), f_from_bits(row_of_quad(bits_from_f(st.f1), lane))};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[r] = b1v[r];
#pragma unroll
                for (int k = 0; k < 3; ++k) x[r] = fmaf(f[k], wp[k][r], x[r]);
            }
        } else if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            const uint32_t c = row_of_quad((uint32_t)bc | (uint32_t)pc << 16, lane);
            const f4v u = *reinterpret_cast<const f4v*>(w1s + (c & 0xffffu) * H + 4 * b), v = *reinterpret_cast<const f4v*>(w1s + (c >> 16) * H + 4 * b);
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = (b1v[r] + u[r]) + v[r];
        } else {
            const uint32_t c = row_of_quad(st.s0 & 0xffffu, lane);
            const f4v u = *reinterpret_cast<const f4v*>(w1s + c * H + 4 * b);
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = (b1v[r] + u[r]) + wp[0][r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = x[r] > 0.0f ? x[r] : 0.0f;
        // ---- second layer, records beside it ----
        const bool keep = t < T && a.keep_acts;
        f4v acc = {b2, b2, b2, b2};
        {
            const rsrc_sm d = rsrc(tp.act[0] + ((size_t)t * B + b0 + row0) * H, keep);
            __builtin_amdgcn_sched_barrier(0);
            layer16<0>(x[0], w2, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(x[r]), d, 4 * (i * H + b), 64 * r, 0);
            store_state(t);
            layer16<0>(x[1], w2 + 16, acc);
            store_heads(t - 1, t > 0);
            layer16<0>(x[2], w2 + 32, acc);
            store_step(t - 1, t > 0);
            layer16<0>(x[3], w2 + 48, acc);
        }
        float y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = acc[r] > 0.0f ? acc[r] : 0.0f;
        const rsrc_sm d1 = rsrc(tp.act[1] + ((size_t)t * B + b0 + row0) * H, keep);
#pragma unroll
        for (int r = 0; r < 4; ++r) __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(y[r]), d1, 4 * lane, 4 * H * r, 0);
        // ---- heads ----
        swap_rows(y);
        hv = hbias;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            chain16(y[s], f4v{hw[16 * s], hw[16 * s + 1], hw[16 * s + 2], hw[16 * s + 3]}, f4v{hw[16 * s + 4], hw[16 * s + 5], hw[16 * s + 6], hw[16 * s + 7]},
                    f4v{hw[16 * s + 8], hw[16 * s + 9], hw[16 * s + 10], hw[16 * s + 11]}, f4v{hw[16 * s + 12], hw[16 * s + 13], hw[16 * s + 14], hw[16 * s + 15]}, hv);
        if (t == T) break;
        // ---- sample, step; all lanes of a row do the same ----
        const uint4 dr = *reinterpret_cast<const uint4*>(rng + ((t & 1) * SMT + row0 + e) * 4);
        row_step<ENV>(a.env, st, sine, hv, dr, obs + (row0 + e) * OBS_WORDS, eps, actf, act, rew, done);
        __syncthreads();                                           // the next step's draws are there, this step's are used
    }
    store_heads(T, true);
    if (j == 0) {
        tp.s0[b0 + row0 + e] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b0 + row0 + e] = st.f0; tp.f1[b0 + row0 + e] = st.f1; }
    }
}

static size_t small_lds_bytes(const EnvDims& env)
{
    const size_t cells = env.kind == ENV_PENDULUM ? 0 : (size_t)env.rows * env.cols;
    return (size_t)2 * SMT * 16 + cells * 64 * 4 + (env.kind == ENV_MAZE ? (size_t)SMT * OBS_WORDS * 4 + (size_t)(SMT + 1) * 64 * 4 : 0);
}

// Up to one workgroup per compute unit: two share its SIMDs badly, and rollout_resident64_kernel multiplies 16 environments at a
// time.  Unrolls of 21 passes, that kernel / this one: Catch 64 environments 31.8 / 23.4 us, 1024 36.6 / 29.1, 4096 34.0 / 27.5,
// 8192 43.2 / 53.3, 65536 247 / 364; 16 x 16 maze 64 46.2 / 37.0, 4096 47.0 / 40.8; 8 x 8 maze 8192 51.3 / 63.5.
bool rollout_small_ok(const anakin* h)
{
    const NetShape& n = h->net;
    if (n.bf16 || n.L != 2 || n.dims[1] != 64 || n.dims[2] != 64 || small_lds_bytes(h->env) > 160 * 1024) return false;
    return h->B <= SMT * 256;
}

hipError_t launch_small(anakin* h, const RolloutArgs& a)
{
    const size_t lds = small_lds_bytes(h->env);
    auto launch = [&](auto kern) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        ProfScope prof(h, "rollout");
        hipLaunchKernelGGL(kern, dim3(h->B / SMT), dim3(64 * (SMW + 1)), lds, h->stream, a);
        return hipGetLastError();
    };
    switch (h->env.kind) {
        case ENV_CATCH:    return launch(rollout_small_kernel<ENV_CATCH>);
        case ENV_PENDULUM: return launch(rollout_small_kernel<ENV_PENDULUM>);
        default:           return launch(rollout_small_kernel<ENV_MAZE>);
    }
}

}  // namespace ank
