// Acting (and replay) of one-hidden-layer nets wider than a lane holds, of mazes and of bf16 nets on the canonical path: a
// wavefront owns four environments, a row of 16 lanes each, and needs nobody else.
//
// Lane i of a row computes the hidden units i, 16 + i, 32 + i, ... of its environment, which is at once the operand order of
// the head chains (chain16: the row's 16 inputs handed round by the DPP row broadcast, lane j sums head j), so the
// activations never leave the registers and the time loop has no barrier.  All lanes of a row sample and step the same
// environment.  A lane makes one draw of eight steps' two at a time (16 lanes: 8 steps x action, reset), so a step pays an
// eighth of a Philox call.  Head weights are in registers up to 128 units, in LDS beyond; the first layer's rows in LDS where
// a few workgroups still fit beside each other.  The arithmetic is the canonical one, bit for bit.
//
// What bounds it: at small batches the chain (first layer 0.3 k cycles, heads 6 to 7 cycles per unit, sample and step 0.4 to
// 0.8 k), at large ones the same instructions' issue slots.  An unroll against the vector-ALU kernel (four barriers a step, a
// thread per four units), fp32: pendulum 128, 336 environments, T = 20 47 -> 25 us; 256, 4240 122 -> 56; Catch 256, 80, T = 61
// 174 -> 98; 128, 58608, T = 40 638 -> 305; maze 9 x 13, 256, 16400, T = 20 385 -> 134.
#include <type_traits>
#include "acting.h"

namespace ank {

constexpr int OTM = 16;                                            // environments per workgroup: four wavefronts
struct OneArgs {
    RolloutArgs r;
    int w1_lds;                  // first-layer rows (maze: agent plane) in LDS
    int o_wh, o_obs, o_pre, o_w1;
    int tseg, tend;              // REPLAY: time steps per workgroup (grid y), time steps evaluated
};
typedef const __attribute__((address_space(4))) OneArgs* kernarg_one;

template <int ENV, int H, bool BF, bool REPLAY>
__global__ __launch_bounds__(WG, H >= 128 ? 2 : ENV == ENV_MAZE && H == 64 ? 3 : 4) void rollout_one_kernel(const OneArgs q)
{
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH <= 4 ? 4 : 8, A = NH - 1;
    constexpr int U = H / 16, LDW1 = H + 16, LDWH = H + 4;
    constexpr bool HREG = H <= 128;
    const RolloutArgs& a = q.r;
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int D = a.net.dims[0], B = a.B, T = a.T, n_cells = a.env.rows * a.env.cols;
    float* whs = smem + q.o_wh;                                    // [NH][H + 4] head weights, transposed (not HREG)
    uint32_t* obs = reinterpret_cast<uint32_t*>(smem + q.o_obs);   // maze: [16][OBS_WORDS], walls
    float* pre = smem + q.o_pre;                                   // maze: [16][H] wall sums; then b1
    float* w1s = smem + q.o_w1;                                    // first-layer rows, [H + 16] apart
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * OTM, row0 = 4 * wave, r16 = lane >> 4, i16 = lane & 15;
    const int b = b0 + row0 + r16;

    float hw[HREG ? H : 16];                                       // lane j: weights of head j
    if (HREG) {
        const float* src = a.theta + a.net.wh_off + (i16 < NH ? i16 : 0);
#pragma unroll
        for (int u = 0; u < H; ++u) hw[HREG ? u : 0] = src[u * NH];
    }
    float base[U];                                                 // bias, or the maze's wall sums: what every step starts from
#pragma unroll
    for (int u = 0; u < U; ++u) base[u] = a.theta[a.net.b_off[0] + 16 * u + i16];
    float wp[ENV == ENV_PENDULUM ? 3 : 1][U];                      // pendulum: the three rows; maze: the goal's
#pragma unroll
    for (int k = 0; k < (ENV == ENV_PENDULUM ? 3 : 1); ++k)
#pragma unroll
        for (int u = 0; u < U; ++u)
            wp[k][u] = ENV == ENV_CATCH ? 0.0f : w1g[(size_t)(ENV == ENV_PENDULUM ? k : 3 * n_cells - 1) * H + 16 * u + i16];
    if (!HREG)
        for (int i = tid; i < H * NH; i += WG) whs[(i % NH) * LDWH + i / NH] = round1<BF>(a.theta[a.net.wh_off + i]);
    if (q.w1_lds) {
        const float* src = w1g + (ENV == ENV_MAZE ? (size_t)n_cells * H : 0);
        const int n4 = (ENV == ENV_MAZE ? n_cells : D) * (H / 4);
#pragma unroll 1
        for (int i0 = tid; i0 < n4; i0 += 4 * WG) {
            f4v v[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) v[p] = reinterpret_cast<const f4v*>(src)[i0 + p * WG < n4 ? i0 + p * WG : i0];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int i = i0 + p * WG;
                if (i < n4) { round4<BF>(v[p]); *reinterpret_cast<f4v*>(w1s + i / (H / 4) * LDW1 + i % (H / 4) * 4) = v[p]; }
            }
        }
    }
    if (ENV == ENV_MAZE) {
        float* b1s = pre + OTM * H;
        for (int i = tid; i < OTM * 8; i += WG) obs[(i >> 3) * OBS_WORDS + (i & 7)] = tp.walls[(size_t)(i & 7) * B + b0 + (i >> 3)];
        for (int i = tid; i < H; i += WG) b1s[i] = a.theta[a.net.b_off[0] + i];
        __syncthreads();
        maze_prefix<BF, WG>(a, OTM, obs, w1g, b1s, pre, tid);
    }
    __syncthreads();
    if (ENV == ENV_MAZE) {
#pragma unroll
        for (int u = 0; u < U; ++u) base[u] = pre[(row0 + r16) * H + 16 * u + i16];
    }
    if (BF) {
#pragma unroll
        for (int u = 0; u < (HREG ? H : 0); u += 2) round2<BF>(hw[u], hw[u + 1]);
#pragma unroll
        for (int k = 0; k < (ENV == ENV_PENDULUM ? 3 : 1); ++k)
#pragma unroll
            for (int u = 0; u < U; u += 2) round2<BF>(wp[k][u], wp[k][u + 1]);
    }
    const float hbias = a.theta[a.net.bh_off + (i16 < NH ? i16 : 0)];
    EnvState st{0u, 0.0f, 0.0f};
    const int t_begin = REPLAY ? (int)blockIdx.y * q.tseg : 0;
    const int t_end = REPLAY ? (t_begin + q.tseg < q.tend ? t_begin + q.tseg : q.tend) : T + 1;
    EnvState nx{0u, 0.0f, 0.0f};                                   // REPLAY: the next step's state, asked for a step ahead
    auto ask = [&](int t) __attribute__((always_inline)) {
        const size_t tb = (size_t)(t < t_end ? t : t_end - 1) * B + b;
        nx.s0 = tp.tr_s0[tb];
        if (ENV == ENV_PENDULUM) { nx.f0 = tp.tr_f0[tb]; nx.f1 = tp.tr_f1[tb]; }
    };
    if (REPLAY) ask(t_begin);
    else {
        st.s0 = tp.s0[b];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0): nothing loaded so far is waited for inside the loop

    auto rsrc = [&](const void* p) __attribute__((always_inline)) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffffu, 0x00020000); };
    uint32_t dr0 = 0u, dr1 = 0u;                                   // lane i: draws of step i % 8 of the current eight (i < 8: action, else reset)
#pragma unroll 1
    for (int t = t_begin; t < t_end; ++t) {
        kernarg_one k = (kernarg_one)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(k));
        const size_t te = (size_t)t * B + b0 + row0;               // this wavefront's first environment
        const int o4 = i16 == 0 ? 4 * r16 : -1, o1 = i16 == 0 ? r16 : -1;
        if (REPLAY) { st = nx; ask(t + 1); }
        else {
            __builtin_amdgcn_raw_buffer_store_b32(st.s0, rsrc(k->r.tp.tr_s0 + te), o4, 0, 0);
            if (ENV == ENV_PENDULUM) {
                __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f0), rsrc(k->r.tp.tr_f0 + te), o4, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f1), rsrc(k->r.tp.tr_f1 + te), o4, 0, 0);
            }
            if ((t & 7) == 0) {
                const u32x4 d = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)(t + (i16 & 7)), i16 < 8 ? DOM_ACTION : DOM_RESET);
                dr0 = ENV == ENV_PENDULUM && i16 < 8 ? bits_from_f(gaussian_noise(d.x, d.y)) : d.x;
                dr1 = d.y;
            }
        }
        // ---- first layer: lane i of the row, units 16 u + i ----
        float h[U];
        float sine = 0.0f;
        if (ENV == ENV_PENDULUM) {
            float cs;
            det_sincos(st.f0, sine, cs);
            const float x[3] = {round1<BF>(cs), round1<BF>(sine), round1<BF>(st.f1)};
#pragma unroll
            for (int u = 0; u < U; ++u) {
                h[u] = base[u];
#pragma unroll
                for (int c = 0; c < 3; ++c) h[u] = fmaf(x[c], wp[ENV == ENV_PENDULUM ? c : 0][u], h[u]);
            }
        } else {
            int c0, c1 = 0;
            if (ENV == ENV_CATCH) catch_obs_cells(a.env, st.s0, c0, c1);
            else c0 = (int)(st.s0 & 0xffffu);
            float x0[U], x1[U];
            if (q.w1_lds) {
                const float* r0 = w1s + __umul24((unsigned)c0, (unsigned)LDW1) + i16;
                const float* r1 = w1s + __umul24((unsigned)c1, (unsigned)LDW1) + i16;
#pragma unroll
                for (int u = 0; u < U; ++u) { x0[u] = r0[16 * u]; if (ENV == ENV_CATCH) x1[u] = r1[16 * u]; }
            } else {
                const float* r0 = w1g + (size_t)(ENV == ENV_MAZE ? n_cells + c0 : c0) * H + i16;
                const float* r1 = w1g + (size_t)c1 * H + i16;
#pragma unroll
                for (int u = 0; u < U; ++u) { x0[u] = r0[16 * u]; if (ENV == ENV_CATCH) x1[u] = r1[16 * u]; }
                if (BF) {
#pragma unroll
                    for (int u = 0; u < U; u += 2) { round2<BF>(x0[u], x0[u + 1]); if (ENV == ENV_CATCH) round2<BF>(x1[u], x1[u + 1]); }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) h[u] = (base[u] + x0[u]) + (ENV == ENV_CATCH ? x1[u] : wp[0][u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) h[u] = h[u] > 0.0f ? h[u] : 0.0f;
        if (BF) {
#pragma unroll
            for (int u = 0; u < U; u += 2) round2<BF>(h[u], h[u + 1]);
        }
        // ---- heads: lane j of the row head j ----
        float hv = hbias;
        if (HREG) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float* w = hw + (HREG ? 16 * u : 0);
                chain16(h[u], f4v{w[0], w[1], w[2], w[3]}, f4v{w[4], w[5], w[6], w[7]}, f4v{w[8], w[9], w[10], w[11]}, f4v{w[12], w[13], w[14], w[15]}, hv);
            }
        } else {
            const f4v* wr = reinterpret_cast<const f4v*>(whs + (i16 < NH ? i16 : 0) * LDWH);
            f4v w[2][4];
#pragma unroll
            for (int p = 0; p < 4; ++p) w[0][p] = wr[p];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u + 1 < U) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) w[(u + 1) & 1][p] = wr[4 * (u + 1) + p];
                }
                __builtin_amdgcn_sched_barrier(0);
                chain16(h[u], w[u & 1][0], w[u & 1][1], w[u & 1][2], w[u & 1][3], hv);
            }
        }
        if (t < T && a.keep_acts) {
            const __amdgpu_buffer_rsrc_t d = rsrc(k->r.tp.act[0] + te * H);
            const int off = 4 * (r16 * H + i16);
#pragma unroll
            for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(h[u]), d, off, 64 * u, 0);
        }
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(i16 < NH ? hv : 0.0f), rsrc(k->r.tp.tr_head + te * NHP), i16 < NHP ? 4 * (r16 * NHP + i16) : -1, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(hv), rsrc(k->r.tp.tr_val + te), i16 == NH - 1 ? 4 * r16 : -1, 0, 0);
        if (REPLAY || t == T) continue;
        // ---- sample, step; all lanes of a row do the same (row_step of acting.h in place: called, Catch with 256 units and
        // 8192 environments took 56.9 us instead of 55.9) ----
        const int src = 4 * ((lane & 48) + (t & 7));
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)dr0);
        const uint32_t e0 = (uint32_t)__builtin_amdgcn_ds_bpermute(src + 32, (int)dr0), e1 = (uint32_t)__builtin_amdgcn_ds_bpermute(src + 32, (int)dr1);
        float rew;
        int done;
        if (ENV == ENV_PENDULUM) {
            const float eps = f_from_bits(d0), actf = gaussian_action(row_lane<0>(hv), row_lane<1>(hv), eps);
            pendulum_step_sn(a.env, st, sine, actf, e0, e1, rew, done);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(eps), rsrc(k->r.tp.tr_eps + te), o4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(actf), rsrc(k->r.tp.tr_actf + te), o4, 0, 0);
        } else {
            const float l0 = row_lane<0>(hv), l1 = row_lane<1>(hv), l2 = row_lane<2>(hv), l3 = A > 3 ? row_lane<3>(hv) : 0.0f;
            float mx = l0;
            mx = l1 > mx ? l1 : mx;
            mx = l2 > mx ? l2 : mx;
            if (A > 3) mx = l3 > mx ? l3 : mx;
            const float ex = det_exp(hv - mx);                     // lane j: the exponential of logit j
            const float c0 = row_lane<0>(ex), c1 = c0 + row_lane<1>(ex), c2 = c1 + row_lane<2>(ex), c3 = A > 3 ? c2 + row_lane<3>(ex) : c2;
            const float thr = u01(d0) * c3;
            int act = A - 1;
            if (A > 3 && c2 > thr) act = 2;
            if (c1 > thr) act = 1;
            if (c0 > thr) act = 0;
            if (ENV == ENV_CATCH) catch_step(a.env, st, act, e0, rew, done);
            else {
                const uint32_t* wl = obs + (row0 + r16) * OBS_WORDS;
                maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, rew, done);
            }
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)act, rsrc(k->r.tp.tr_act + te), o1, 0, 0);
        }
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(rew), rsrc(k->r.tp.tr_rew + te), o4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)done, rsrc(k->r.tp.tr_done + te), o1, 0, 0);
    }
    if (!REPLAY && i16 == 0) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// LDS of a workgroup; offsets in floats
static size_t one_lds(const NetShape& net, const EnvDims& env, int workgroups, OneArgs& q)
{
    const int H = net.dims[1], cells = env.rows * env.cols;
    int off = 0;
    q.o_wh = off; off += H > 128 ? 8 * (H + 4) : 0;
    q.o_obs = off; off += env.kind == ENV_MAZE ? OTM * OBS_WORDS : 0;
    q.o_pre = off; off += env.kind == ENV_MAZE ? OTM * H + H : 0;
    q.o_w1 = off;
    // the rows in LDS where four workgroups fit beside each other, or where there are not so many that several would share
    // a compute unit
    const size_t w1 = (size_t)(env.kind == ENV_MAZE ? cells : net.dims[0]) * (H + 16), all = ((size_t)off + w1) * 4;
    q.w1_lds = env.kind != ENV_PENDULUM && (all <= 40 * 1024 || (workgroups <= 256 && all <= 160 * 1024)) ? 1 : 0;
    return q.w1_lds ? all : (size_t)off * 4;
}

bool rollout_one_ok(const anakin* h)
{
    const NetShape& n = h->net;
    return n.L == 1 && n.dims[1] <= 256 && !(h->mode & (ANAKIN_MODE_CANONICAL_ACTING | ANAKIN_MODE_STREAM_WEIGHTS));
}

template <int ENV, bool BF, bool REPLAY>
static hipError_t launch_one_env(anakin* h, const OneArgs& q, dim3 grid, size_t lds)
{
    const int H = h->net.dims[1];
    auto kern = H == 32 ? rollout_one_kernel<ENV, 32, BF, REPLAY> : H == 64 ? rollout_one_kernel<ENV, 64, BF, REPLAY> : H == 128 ? rollout_one_kernel<ENV, 128, BF, REPLAY> : rollout_one_kernel<ENV, 256, BF, REPLAY>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, REPLAY ? "replay_forward" : "rollout");
    hipLaunchKernelGGL(kern, grid, dim3(WG), lds, h->stream, q);
    return hipGetLastError();
}

hipError_t launch_rollout_one(anakin* h, const RolloutArgs& args, bool replay)
{
    OneArgs q;
    q.r = args;
    const int tiles = h->B / OTM;
    q.tend = args.T + (args.bootstrap ? 1 : 0);
    q.tseg = replay ? replay_segment(tiles, q.tend) : q.tend;
    const dim3 grid(tiles, replay ? (q.tend + q.tseg - 1) / q.tseg : 1);
    const size_t lds = one_lds(h->net, h->env, (int)(grid.x * grid.y), q);
    auto go = [&](auto env) {
        constexpr int E = decltype(env)::value;
        if (h->net.bf16) return replay ? launch_one_env<E, true, true>(h, q, grid, lds) : launch_one_env<E, true, false>(h, q, grid, lds);
        return replay ? launch_one_env<E, false, true>(h, q, grid, lds) : launch_one_env<E, false, false>(h, q, grid, lds);
    };
    switch (h->env.kind) {
        case ENV_CATCH:    return go(std::integral_constant<int, ENV_CATCH>());
        case ENV_PENDULUM: return go(std::integral_constant<int, ENV_PENDULUM>());
        default:           return go(std::integral_constant<int, ENV_MAZE>());
    }
}

}  // namespace ank
