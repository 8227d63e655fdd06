// Acting: one persistent launch runs the whole T-step unroll (paper figure 2
// top; section 2.1 loop).  A workgroup owns a tile of TM environments for all T
// steps -- environments never interact, so no grid-wide synchronisation is
// needed -- and per step does: observe, policy/value forward, sample, env step,
// trajectory write.  Env state lives in registers, activations in LDS, the
// trajectory and the hidden activations (reused by the update, paper section
// 3.1) go to HBM time-major.
//
// The forward pass follows the canonical order: every output starts from its
// bias and accumulates x_k * W[k][j] by fused multiply-add for k ascending.
// Each thread owns an RM x 4 register tile of a layer's outputs and walks k
// from 0 upwards, which is exactly that order, so logits are reproducible bit
// for bit and independent of the tiling.  One-hot observations (Catch, Maze)
// turn the first layer into a gather-sum of weight rows in ascending row
// order: fma(0,w,acc) = acc and fma(1,w,acc) = acc + w, the same bits.
//
// Kernels: rollout_kernel (vector ALU), rollout_stream_kernel (matrix cores, weights streamed),
// rollout_resident_kernel and rollout_resident64_kernel (two equal layers of 128 or 256 resp. 64
// units, W2 in registers), rollout_pinned_kernel (other nets whose hidden matrices fit the registers, at
// most 4096 environments; rollout_pinned.hip), rollout_wide_kernel (wider nets and two equal layers of 256 at up to
// 2048 environments; rollout_wide.hip), rollout_lane_kernel (one narrow hidden layer, very many
// environments: one lane per env), rollout_one_kernel (other nets of one hidden layer; rollout_one.hip).  All but
// the resident, pinned and wide ones have a REPLAY form, the learner's forward pass over a stored unroll (decoupled
// steps, several updates per unroll); those replay with streamed weights, two equal layers of 128 or 256 units on
// Catch and the pendulum from 4096 samples on with resident ones (rollout_replay.hip).
// BF: bf16 nets that the bf16 matrix instructions do not take (batches that are no multiple of 64, mazes of other
// sizes): the same kernels on weights and activations rounded to bfloat16, products and sums in binary32 -- the
// vector-ALU kernel's bits at the matrix instruction's rate (256-256, 1040 environments, T = 20: 1197 -> 207 us;
// maze 512-256, 5568, T = 17: 3908 -> 633).
#include "acting.h"

namespace ank {

template <int RM, bool BF>
__device__ __forceinline__ void finish_rows(float (&acc)[RM][4], float* __restrict__ Y, int ldx, int m0, int c0,
                                            float* __restrict__ gout, int N)
{
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        float4 o;
        o.x = acc[r][0] > 0.0f ? acc[r][0] : 0.0f;
        o.y = acc[r][1] > 0.0f ? acc[r][1] : 0.0f;
        o.z = acc[r][2] > 0.0f ? acc[r][2] : 0.0f;
        o.w = acc[r][3] > 0.0f ? acc[r][3] : 0.0f;
        if (BF) { o.x = bfr(o.x); o.y = bfr(o.y); o.z = bfr(o.z); o.w = bfr(o.w); }
        *reinterpret_cast<float4*>(Y + (m0 + r) * ldx + c0) = o;
        if (gout) *reinterpret_cast<float4*>(gout + (size_t)(m0 + r) * N + c0) = o;
    }
}

// Y[TM][N] = relu(X[TM][K] W[K][N] + b), X and Y in LDS (row stride ldx), W in global memory
template <int RM, bool BF>
__device__ __forceinline__ void dense_layer(const float* __restrict__ X, float* __restrict__ Y, int ldx,
                                            const float* __restrict__ W, const float* __restrict__ bias,
                                            int K, int N, int tid, float* __restrict__ gout)
{
    const int CG = N >> 2, tn = tid % CG, m0 = (tid / CG) * RM, c0 = tn << 2;
    float acc[RM][4];
    const float4 b = ld4(bias + c0);
#pragma unroll
    for (int r = 0; r < RM; ++r) { acc[r][0] = b.x; acc[r][1] = b.y; acc[r][2] = b.z; acc[r][3] = b.w; }
    const float* wp = W + c0;
    for (int k0 = 0; k0 < K; k0 += 4) {
        const float4 w0 = ldw4<BF>(wp + (size_t)(k0 + 0) * N);
        const float4 w1 = ldw4<BF>(wp + (size_t)(k0 + 1) * N);
        const float4 w2 = ldw4<BF>(wp + (size_t)(k0 + 2) * N);
        const float4 w3 = ldw4<BF>(wp + (size_t)(k0 + 3) * N);
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            const float4 x = ld4(X + (m0 + r) * ldx + k0);
            acc[r][0] = fmaf(x.x, w0.x, acc[r][0]); acc[r][1] = fmaf(x.x, w0.y, acc[r][1]);
            acc[r][2] = fmaf(x.x, w0.z, acc[r][2]); acc[r][3] = fmaf(x.x, w0.w, acc[r][3]);
            acc[r][0] = fmaf(x.y, w1.x, acc[r][0]); acc[r][1] = fmaf(x.y, w1.y, acc[r][1]);
            acc[r][2] = fmaf(x.y, w1.z, acc[r][2]); acc[r][3] = fmaf(x.y, w1.w, acc[r][3]);
            acc[r][0] = fmaf(x.z, w2.x, acc[r][0]); acc[r][1] = fmaf(x.z, w2.y, acc[r][1]);
            acc[r][2] = fmaf(x.z, w2.z, acc[r][2]); acc[r][3] = fmaf(x.z, w2.w, acc[r][3]);
            acc[r][0] = fmaf(x.w, w3.x, acc[r][0]); acc[r][1] = fmaf(x.w, w3.y, acc[r][1]);
            acc[r][2] = fmaf(x.w, w3.z, acc[r][2]); acc[r][3] = fmaf(x.w, w3.w, acc[r][3]);
        }
    }
    finish_rows<RM, BF>(acc, Y, ldx, m0, c0, gout, N);
}

// first layer: gather-sum for the one-hot boards, three fmas for the pendulum
template <int ENV, int RM, bool BF>
__device__ __forceinline__ void first_layer(const RolloutArgs& a, const uint32_t* __restrict__ obs,
                                            float* __restrict__ Y, int ldx, int tid, float* __restrict__ gout,
                                            const float* w1, const float* b1, const float* pre)
{
    const int N = a.net.dims[1];
    const int CG = N >> 2, tn = tid % CG, m0 = (tid / CG) * RM, c0 = tn << 2;
    const float* wp = w1 + c0;
    float acc[RM][4];
    if (ENV == ENV_MAZE && pre) {
        // bias and wall plane come summed (maze_prefix); what changes from step to step is one row per environment
        const int n = a.env.rows * a.env.cols;
        float4 w[RM];
#pragma unroll
        for (int r = 0; r < RM; ++r) w[r] = ldw4<BF>(wp + (size_t)(n + (int)obs[(m0 + r) * OBS_WORDS + 8]) * N);
        const float4 g = ldw4<BF>(wp + (size_t)(3 * n - 1) * N);
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            const float4 p = ld4(pre + (m0 + r) * N + c0);
            acc[r][0] = (p.x + w[r].x) + g.x; acc[r][1] = (p.y + w[r].y) + g.y;
            acc[r][2] = (p.z + w[r].z) + g.z; acc[r][3] = (p.w + w[r].w) + g.w;
        }
        finish_rows<RM, BF>(acc, Y, ldx, m0, c0, gout, N);
        return;
    }
    const float4 b = ld4(b1 + c0);
#pragma unroll
    for (int r = 0; r < RM; ++r) { acc[r][0] = b.x; acc[r][1] = b.y; acc[r][2] = b.z; acc[r][3] = b.w; }
    if (ENV == ENV_CATCH) {
#pragma unroll
        for (int r = 0; r < RM; ++r) {
#pragma unroll
            for (int which = 0; which < 2; ++which) {
                const int cell = (int)obs[(m0 + r) * OBS_WORDS + which];
                const float4 w = ldw4<BF>(wp + (size_t)cell * N);
                acc[r][0] += w.x; acc[r][1] += w.y; acc[r][2] += w.z; acc[r][3] += w.w;
            }
        }
    } else if (ENV == ENV_PENDULUM) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float4 w = ldw4<BF>(wp + (size_t)k * N);
#pragma unroll
            for (int r = 0; r < RM; ++r) {
                float x = f_from_bits(obs[(m0 + r) * OBS_WORDS + k]);
                if (BF) x = bfr(x);
                acc[r][0] = fmaf(x, w.x, acc[r][0]); acc[r][1] = fmaf(x, w.y, acc[r][1]);
                acc[r][2] = fmaf(x, w.z, acc[r][2]); acc[r][3] = fmaf(x, w.w, acc[r][3]);
            }
        }
    } else {
        const int n = a.env.rows * a.env.cols;
        for (int c = 0; c < n; ++c) {                       // wall plane, ascending cell index
            const float4 w = ldw4<BF>(wp + (size_t)c * N);
#pragma unroll
            for (int r = 0; r < RM; ++r) {
                if ((obs[(m0 + r) * OBS_WORDS + (c >> 5)] >> (c & 31)) & 1u) {
                    acc[r][0] += w.x; acc[r][1] += w.y; acc[r][2] += w.z; acc[r][3] += w.w;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RM; ++r) {                      // agent plane
            const int cell = (int)obs[(m0 + r) * OBS_WORDS + 8];
            const float4 w = ldw4<BF>(wp + (size_t)(n + cell) * N);
            acc[r][0] += w.x; acc[r][1] += w.y; acc[r][2] += w.z; acc[r][3] += w.w;
        }
        {                                                   // goal plane: always the last cell
            const float4 w = ldw4<BF>(wp + (size_t)(3 * n - 1) * N);
#pragma unroll
            for (int r = 0; r < RM; ++r) { acc[r][0] += w.x; acc[r][1] += w.y; acc[r][2] += w.z; acc[r][3] += w.w; }
        }
    }
    finish_rows<RM, BF>(acc, Y, ldx, m0, c0, gout, N);
}

template <int ENV, bool BF>
__device__ __forceinline__ void run_first_layer(const RolloutArgs& a, int TM, const uint32_t* obs, float* Y, int tid, float* gout,
                                                const float* w1, const float* pre)
{
    const float* b1 = a.theta + a.net.b_off[0];
    const int RM = TM * a.net.dims[1] / 1024;
    switch (RM) {
        case 1: first_layer<ENV, 1, BF>(a, obs, Y, a.ldx, tid, gout, w1, b1, pre); break;
        case 2: first_layer<ENV, 2, BF>(a, obs, Y, a.ldx, tid, gout, w1, b1, pre); break;
        case 4: first_layer<ENV, 4, BF>(a, obs, Y, a.ldx, tid, gout, w1, b1, pre); break;
        case 8: first_layer<ENV, 8, BF>(a, obs, Y, a.ldx, tid, gout, w1, b1, pre); break;
        default: first_layer<ENV, 16, BF>(a, obs, Y, a.ldx, tid, gout, w1, b1, pre); break;
    }
}

template <bool BF>
__device__ __forceinline__ void run_dense_layer(const RolloutArgs& a, int TM, int l, const float* X, float* Y, int tid, float* gout)
{
    const int K = a.net.dims[l], N = a.net.dims[l + 1];
    const float* W = a.theta + a.net.w_off[l];
    const float* bias = a.theta + a.net.b_off[l];
    const int RM = TM * N / 1024;
    switch (RM) {
        case 1: dense_layer<1, BF>(X, Y, a.ldx, W, bias, K, N, tid, gout); break;
        case 2: dense_layer<2, BF>(X, Y, a.ldx, W, bias, K, N, tid, gout); break;
        case 4: dense_layer<4, BF>(X, Y, a.ldx, W, bias, K, N, tid, gout); break;
        case 8: dense_layer<8, BF>(X, Y, a.ldx, W, bias, K, N, tid, gout); break;
        default: dense_layer<16, BF>(X, Y, a.ldx, W, bias, K, N, tid, gout); break;
    }
}


typedef float f16v __attribute__((ext_vector_type(16)));

template <int NT>
__device__ __forceinline__ void load_nt(const float* __restrict__ p, float (&b)[NT])
{
    if (NT == 1) { b[0] = p[0]; }
    else if (NT == 2) { const float2 v = *reinterpret_cast<const float2*>(p); b[0] = v.x; b[1] = v.y; }
    else {
#pragma unroll
        for (int q = 0; q < NT / 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(p + 4 * q);
            b[4 * q + 0] = v.x; b[4 * q + 1] = v.y; b[4 * q + 2] = v.z; b[4 * q + 3] = v.w;
        }
    }
}
template <int NT>
__device__ __forceinline__ void store_nt(float* __restrict__ p, const float (&b)[NT])
{
    if (NT == 1) { p[0] = b[0]; }
    else if (NT == 2) { *reinterpret_cast<float2*>(p) = make_float2(b[0], b[1]); }
    else {
#pragma unroll
        for (int q = 0; q < NT / 4; ++q)
            *reinterpret_cast<float4*>(p + 4 * q) = make_float4(b[4 * q + 0], b[4 * q + 1], b[4 * q + 2], b[4 * q + 3]);
    }
}

// Heads: out[m][j] = bh[j] + sum_k X[m][k] Wh[k][j], one sequential fused multiply-add chain
// per (env, head) as the canonical order demands.  The chain is latency-bound, so what matters
// is that its operands are already in registers: lane (m, j) streams row m of X and row j of
// the transposed head matrix (both k-contiguous in LDS, 16-byte reads), 32 k at a time, with
// the next block in flight while the current one is consumed.
// whT: [NH][ldw] in LDS (ldw = HL + 4).
template <int U>
__device__ __forceinline__ void heads_load(const float* __restrict__ x, const float* __restrict__ w, float4 (&xv)[U], float4 (&wv)[U])
{
#pragma unroll
    for (int u = 0; u < U; ++u) { xv[u] = *reinterpret_cast<const float4*>(x + 4 * u); wv[u] = *reinterpret_cast<const float4*>(w + 4 * u); }
}
template <int U>
__device__ __forceinline__ float heads_fma(const float4 (&xv)[U], const float4 (&wv)[U], float acc)
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        acc = fmaf(xv[u].x, wv[u].x, acc);
        acc = fmaf(xv[u].y, wv[u].y, acc);
        acc = fmaf(xv[u].z, wv[u].z, acc);
        acc = fmaf(xv[u].w, wv[u].w, acc);
    }
    return acc;
}
typedef float f4v_h __attribute__((ext_vector_type(4)));
// The chains on the vector ALU with the operand reads taken off the critical path: lane (m, j)
// keeps a ring of PF blocks of four k (16-byte LDS reads of row m of X and row j of the transposed
// head matrix) and refills each slot, PF blocks ahead, before the four dependent fused multiply-adds
// of the block it just handed over.  HL is a multiple of 4 * PF.
template <int PF, int HL, int NTHR = WG>
__device__ __forceinline__ void heads_pipe(const float* __restrict__ X, int ldx, const float* __restrict__ whT, int ldw,
                                           const float* __restrict__ bhs, float* __restrict__ heads,
                                           int NH, int NHP, int TM, int tid)
{
    constexpr int S = HL >> 2;
    for (int idx = tid; idx < TM * NH; idx += NTHR) {
        const int m = idx % TM, j = idx / TM;
        const f4v_h* x = reinterpret_cast<const f4v_h*>(X + m * ldx);
        const f4v_h* w = reinterpret_cast<const f4v_h*>(whT + j * ldw);
        f4v_h xr[PF], wr[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u) { xr[u] = x[u]; wr[u] = w[u]; }
        float acc = bhs[j];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const f4v_h xv = xr[s % PF], wv = wr[s % PF];
            if (s + PF < S) { xr[s % PF] = x[s + PF]; wr[s % PF] = w[s + PF]; }
            __builtin_amdgcn_sched_barrier(0);
            acc = fmaf(xv[0], wv[0], acc);
            acc = fmaf(xv[1], wv[1], acc);
            acc = fmaf(xv[2], wv[2], acc);
            acc = fmaf(xv[3], wv[3], acc);
        }
        heads[m * NHP + j] = acc;
    }
}

// U: float4 per register block (a block covers 4U values of k; HL is a multiple of 4U)
template <int U, int NTHR>
__device__ __forceinline__ void heads_chain(const float* __restrict__ X, int ldx, const float* __restrict__ whT, int ldw,
                                            const float* __restrict__ bhs, float* __restrict__ heads,
                                            int HL, int NH, int NHP, int TM, int tid)
{
    constexpr int KB = 4 * U;
    for (int idx = tid; idx < TM * NH; idx += NTHR) {
        const int m = idx % TM, j = idx / TM;
        float acc = bhs[j];
        const float* x = X + m * ldx;
        const float* w = whT + j * ldw;
        float4 xa[U], wa[U], xb[U], wb[U];                      // two register blocks, used alternately
        heads_load<U>(x, w, xa, wa);
        for (int k0 = 0; k0 < HL; k0 += 2 * KB) {
            const bool more = k0 + KB < HL;
            if (more) heads_load<U>(x + k0 + KB, w + k0 + KB, xb, wb);
            acc = heads_fma<U>(xa, wa, acc);
            if (more) {
                if (k0 + 2 * KB < HL) heads_load<U>(x + k0 + 2 * KB, w + k0 + 2 * KB, xa, wa);
                acc = heads_fma<U>(xb, wb, acc);
            }
        }
        heads[m * NHP + j] = acc;
    }
}

template <int NTHR>
__device__ __forceinline__ void run_heads(const float* X, int ldx, const float* whT, int ldw, const float* bhs, float* heads,
                                          int HL, int NH, int NHP, int TM, int tid)
{
    switch (HL) {
        case 64: heads_pipe<4, 64, NTHR>(X, ldx, whT, ldw, bhs, heads, NH, NHP, TM, tid); break;
        case 128: heads_pipe<4, 128, NTHR>(X, ldx, whT, ldw, bhs, heads, NH, NHP, TM, tid); break;
        case 256: heads_pipe<4, 256, NTHR>(X, ldx, whT, ldw, bhs, heads, NH, NHP, TM, tid); break;
        case 512: heads_pipe<4, 512, NTHR>(X, ldx, whT, ldw, bhs, heads, NH, NHP, TM, tid); break;
        default: heads_chain<8, NTHR>(X, ldx, whT, ldw, bhs, heads, HL, NH, NHP, TM, tid);
    }
}

// REPLAY: the learner's pass over a stored unroll (decoupled acting and learning): the state of
// step t comes from the stored snapshots, the forward pass is the acting one with the parameters
// in a.theta, head outputs and values go to tp.tr_head / tp.tr_val (the caller points them at the
// learner's buffers) and hidden activations to tp.act; nothing is sampled or stepped.
template <int ENV, bool BF, bool REPLAY>
__global__ __launch_bounds__(WG) void rollout_kernel(const RolloutArgs a, const int TM)
{
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int ldx = a.ldx, NH = a.net.NH, NHP = a.net.NHP, L = a.net.L, HL = a.net.dims[a.net.L];
    float* bufA = smem;
    float* bufB = bufA + TM * ldx;
    float* whs = bufB + TM * ldx;                 // [8][HL + 4] head weights, transposed
    float* bhs = whs + 8 * (HL + 4);              // [8] head biases
    float* heads = bhs + 8;                       // [TM][NHP]
    uint32_t* obs = reinterpret_cast<uint32_t*>(heads + TM * NHP);   // [TM][OBS_WORDS]
    uint32_t* rng = obs + TM * OBS_WORDS;                            // [TM][4] draws of the current step
    float* pre = ENV == ENV_MAZE && a.maze_prefix ? reinterpret_cast<float*>(rng + TM * 4) : nullptr;   // [TM][H1]

    const int tid = threadIdx.x;
    const int b0 = blockIdx.x * TM;
    const int B = a.B, T = a.T;
    const TrajPtrs& tp = a.tp;

    // head weights into LDS once, transposed: whs[j][k], row stride HL + 4
    const int ldw = HL + 4;
    for (int i = tid; i < HL * NH; i += WG) {
        const int k = i / NH, j = i - k * NH;
        float w = a.theta[a.net.wh_off + i];
        if (BF) w = bfr(w);
        whs[j * ldw + k] = w;
    }
    if (tid < 8) bhs[tid] = tid < NH ? a.theta[a.net.bh_off + tid] : 0.0f;

    // env state of this thread's environment (threads 0..TM-1)
    EnvState st{0u, 0.0f, 0.0f};
    const bool owner = tid < TM;
    const int b = b0 + tid;
    if (owner) {
        if (!REPLAY) {
            st.s0 = tp.s0[b];
            if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
        }
        if (ENV == ENV_MAZE) {
            for (int w = 0; w < 8; ++w) obs[tid * OBS_WORDS + w] = tp.walls[(size_t)w * B + b];
        }
    }
    if (ENV == ENV_MAZE && pre) {
        __syncthreads();
        maze_prefix<BF, WG>(a, TM, obs, a.theta + a.net.w_off[0], a.theta + a.net.b_off[0], pre, tid);
    }

    const int t_end = REPLAY ? T + a.bootstrap : T + 1;
    for (int t = 0; t < t_end; ++t) {
        const size_t tb = (size_t)t * B + b;
        // ---- observe -------------------------------------------------------
        if (owner) {
            if (REPLAY) {
                st.s0 = tp.tr_s0[tb];
                if (ENV == ENV_PENDULUM) { st.f0 = tp.tr_f0[tb]; st.f1 = tp.tr_f1[tb]; }
            } else {
                tp.tr_s0[tb] = st.s0;
                if (ENV == ENV_PENDULUM) { tp.tr_f0[tb] = st.f0; tp.tr_f1[tb] = st.f1; }
            }
            if (ENV == ENV_CATCH) {
                int bc, pc;
                catch_obs_cells(a.env, st.s0, bc, pc);
                obs[tid * OBS_WORDS + 0] = (uint32_t)bc;
                obs[tid * OBS_WORDS + 1] = (uint32_t)pc;
            } else if (ENV == ENV_PENDULUM) {
                float sn, cs;
                det_sincos(st.f0, sn, cs);
                obs[tid * OBS_WORDS + 0] = bits_from_f(cs);
                obs[tid * OBS_WORDS + 1] = bits_from_f(sn);
                obs[tid * OBS_WORDS + 2] = bits_from_f(st.f1);
            } else {
                obs[tid * OBS_WORDS + 8] = st.s0 & 0xffffu;
            }
        }
        __syncthreads();
        // ---- forward -------------------------------------------------------
        const bool keep = t < T && a.keep_acts;  // the bootstrap evaluation keeps no activations
        float* g0 = keep ? tp.act[0] + ((size_t)t * B + b0) * a.net.dims[1] : nullptr;
        run_first_layer<ENV, BF>(a, TM, obs, bufA, tid, g0, a.theta + a.net.w_off[0], pre);
        __syncthreads();
        float* cur = bufA;
        float* nxt = bufB;
        for (int l = 1; l < L; ++l) {
            float* gl = keep ? tp.act[l] + ((size_t)t * B + b0) * a.net.dims[l + 1] : nullptr;
            run_dense_layer<BF>(a, TM, l, cur, nxt, tid, gl);
            __syncthreads();
            float* tmp = cur; cur = nxt; nxt = tmp;
        }
        run_heads<WG>(cur, ldx, whs, ldw, bhs, heads, HL, NH, NHP, TM, tid);
        // the step's random draws do not depend on the network: the last lanes of the workgroup,
        // idle during the head chains, produce them now
        if (!REPLAY && t < T) {
            for (int e = WG - 1 - tid; e < TM; e += WG) {
                const u32x4 w = philox(a.seed, (uint32_t)(b0 + e), a.gstep + (uint64_t)t, DOM_ACTION);
                // the pendulum's noise is ready-made when the heads are: only z and tanh remain on the critical path
                rng[e * 4] = ENV == ENV_PENDULUM ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;
                rng[e * 4 + 1] = w.y;
            }
        }
        __syncthreads();
        // ---- sample, step, record -------------------------------------------
        if (owner) {
            const float4 h0 = ld4(heads + tid * NHP);
            const float4 h1 = NHP == 8 ? ld4(heads + tid * NHP + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const float hv[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
            float* hd = tp.tr_head + tb * NHP;
            *reinterpret_cast<float4*>(hd) = h0;
            if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = h1;
            const float val = last_head(hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], NH);
            tp.tr_val[tb] = val;
            if (!REPLAY && t < T) {
                const uint2 dr = *reinterpret_cast<const uint2*>(rng + tid * 4);   // action draw, words 0 and 1
                float r; int done;
                // the reset draw is only needed where an episode ends: the step runs with a placeholder
                // and the few lanes that finished an episode draw and reset afterwards
                if (ENV == ENV_PENDULUM) {
                    const float eps = f_from_bits(dr.x);
                    const float act = gaussian_action(hv[0], hv[1], eps);
                    tp.tr_eps[tb] = eps;
                    tp.tr_actf[tb] = act;
                    pendulum_step(a.env, st, act, 0u, 0u, r, done);
                    if (done) {
                        const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                        pendulum_reset(st, wr.x, wr.y);
                    }
                } else {
                    const int act = sample_categorical_any(hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], a.net.A, u01(dr.x));
                    tp.tr_act[tb] = (uint8_t)act;
                    if (ENV == ENV_CATCH) {
                        catch_step(a.env, st, act, 0u, r, done);
                        if (done) {
                            const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                            st.s0 = catch_reset(a.env, wr.x);
                        }
                    } else {
                        const uint32_t* wl = obs + tid * OBS_WORDS;
                        maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, r, done);
                    }
                }
                tp.tr_rew[tb] = r;
                tp.tr_done[tb] = (uint8_t)done;
            }
        }
        // the next observe phase writes obs words that only the first layer reads, and
        // two barriers separate that read from this point
    }
    if (!REPLAY && owner) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}


// ---------------------------------------------------------------------------
// Hidden layers on the matrix cores, weights streamed from L2: fp32 nets of two or more hidden layers that the
// weights-resident kernels (below and rollout_pinned.hip) do not take.  On gfx950 the fp32 MFMA instructions add their products one k at a time
// with a fused multiply-add, ascending in k, and chain through the accumulator operand -- measured bit-identical to the
// sequential fmaf chain on random, wide-range and integer inputs -- so starting the accumulator from the bias and feeding
// k in ascending order reproduces the canonical order exactly while running at matrix-core rate.
//
// A workgroup owns TM = 16 MT environments, eight of its wavefronts (two per SIMD) the layers; v_mfma_f32_16x16x4_f32:
// lane l feeds A[row l%16][k l/16] and B[k l/16][col l%16], accumulator register r is D[row 4 (l/16) + r][col l%16].
//
// What bounds it at the usual batches (a few tiles per compute unit or fewer) is latency.  Loads and stores of a wavefront
// complete in issue order and share a counter, so a load asked for behind the activation stores of the layer before is not
// seen until those are acknowledged; and with one layer's weights asked for when the layer starts, every layer of every
// step waits for L2 first.  So the work is divided: eight wavefronts compute and load weights but store nothing to memory;
// four more step the environments, draw the random numbers and copy the kept activations from LDS to memory, a layer
// behind.  A wavefront's weights are one stream across column tiles, layers and steps, two blocks of eight k-steps always in
// flight: every block is the same eight loads, so the wait before its use is for exactly that block, whatever the shapes.
// Biases, the first layer's weights where they fit (Catch boards, the maze's agent plane) and the maze's wall sums stay
// in LDS.
// The operands from LDS are asked for a block ahead as well.  Per step of the unroll, against one workgroup of eight
// wavefronts that did all of it: 512-256 net, 2000 environments 15.6 -> 12.3 us; 256-128-64, 1008: 8.5 -> 6.0 us; what is
// left is mostly the binary32 matrix rate of the compute units that have a tile (16 k cycles of 27 k; 4 k of 13 k).
// ---------------------------------------------------------------------------
constexpr int STW = 512;                // threads that compute
constexpr int STA = 256;                // threads beside them: environments, draws, records, activations
struct StreamArgs {
    RolloutArgs r;
    int w1_lds;                  // first-layer weights (maze: agent plane and goal row) in LDS
    int tseg;                    // REPLAY: time steps per workgroup (grid y)
    int tend;                    // time steps evaluated: T + 1 (with the bootstrap state) or T
};

// A wavefront's weight stream: its column tiles (wave, wave + 8, ...) of layer 1, then of layer 2, ..., then of layer 1 of
// the next step, each as K / 32 blocks of eight k-steps -- one float per lane and k-step.  The cursor is scalar throughout
// and runs two blocks ahead of the arithmetic.  The widths (powers of two) are packed into one word: picked from a struct
// or an array by a computed index they would live in scratch memory.
struct StreamCursor { int l, tile, k, w, K, N; };              // w: offset of W_l in theta; k: input the next block starts at
struct StreamNet {
    int L, w1;                                                 // offset of W_1 (layer 1: first to second hidden layer) in theta
    uint32_t lg;                                               // byte l - 1: log2 of the outputs of layer l (= inputs of layer l + 1)
    __device__ __forceinline__ int dim(int l) const { return 1 << ((lg >> (8 * (l - 1))) & 31u); }
    __device__ __forceinline__ void settle(StreamCursor& c, int wave) const
    {
        // on to the next tile that exists (a wavefront may have none in a narrow layer, but has one in some layer)
        while (16 * c.tile >= c.N) {
            c.w += c.K * c.N + c.N;
            c.l += 1; c.tile = wave;
            if (c.l == L) { c.l = 1; c.w = w1; }
            c.K = dim(c.l); c.N = dim(c.l + 1);
        }
    }
    __device__ __forceinline__ void advance(StreamCursor& c, int wave) const
    {
        c.k += 32;
        if (c.k == c.K) { c.k = 0; c.tile += 8; settle(c, wave); }
    }
};
typedef __amdgpu_buffer_rsrc_t rsrc_w;
typedef uint32_t u4v_w __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void stream_load(float (&d)[8], rsrc_w theta, const StreamCursor& c, int lane)
{
    const uint32_t lane_off = 4u * ((uint32_t)(lane >> 4) * (uint32_t)c.N + (uint32_t)(lane & 15));
    const uint32_t row = 4u * (uint32_t)(c.w + 16 * c.tile + c.k * c.N), step = 16u * (uint32_t)c.N;
#pragma unroll
    for (int u = 0; u < 8; ++u) d[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(theta, lane_off, row + u * step, 0));
}

// Layer l of the step for this wavefront's column tiles: X and Y in LDS.  wA, wB: the stream's two blocks in flight.
template <int MT, bool BF>
__device__ __forceinline__ void stream_layer(const StreamNet& n, rsrc_w theta, int l, const float* __restrict__ X, float* __restrict__ Y, int ldx,
                                             const float* __restrict__ bias, int wave, int lane, StreamCursor& cur, float (&wA)[8], float (&wB)[8])
{
    const int K = n.dim(l), N = n.dim(l + 1), kq = lane >> 4;
    const float* xp = X + (lane & 15) * ldx + kq;
    f4v acc[MT];
    float avA[8][MT], avB[8][MT];
    auto fetch = [&](float (&av)[8][MT], int k0) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int m = 0; m < MT; ++m) av[u][m] = xp[m * 16 * ldx + k0 + 4 * u];
        __builtin_amdgcn_sched_barrier(0);
    };
    auto block = [&](float (&w)[8], float (&av)[8][MT]) {
#pragma unroll
        for (int u = 0; u < 8; u += 2) round2<BF>(w[u], w[u + 1]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][m], w[u], acc[m], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        stream_load(w, theta, cur, lane);
        n.advance(cur, wave);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int tile = wave; 16 * tile < N; tile += 8) {
        const int col = 16 * tile + (lane & 15);
        const float bv = bias[col];
#pragma unroll
        for (int m = 0; m < MT; ++m) { acc[m][0] = bv; acc[m][1] = bv; acc[m][2] = bv; acc[m][3] = bv; }
        fetch(avA, 0);
        for (int k0 = 0; k0 < K; k0 += 64) {                          // K is a multiple of 64
            fetch(avB, k0 + 32);
            block(wA, avA);
            fetch(avA, k0 + 64 < K ? k0 + 64 : 0);
            block(wB, avB);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                float y0 = acc[m][r] > 0.0f ? acc[m][r] : 0.0f, y1 = acc[m][r + 1] > 0.0f ? acc[m][r + 1] : 0.0f;
                round2<BF>(y0, y1);
                Y[(16 * m + 4 * kq + r) * ldx + col] = y0;
                Y[(16 * m + 4 * kq + r + 1) * ldx + col] = y1;
            }
    }
}

template <int ENV, int MT, bool REPLAY, bool BF>
__global__ __launch_bounds__(STW + STA) void rollout_stream_kernel(const StreamArgs sa)
{
    const RolloutArgs& a = sa.r;
    constexpr int TM = 16 * MT;
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int ldx = a.ldx, NH = a.net.NH, NHP = a.net.NHP, L = a.net.L, HL = a.net.dims[L], H1 = a.net.dims[1], D = a.net.dims[0];
    const int n_cells = a.env.rows * a.env.cols;
    float* bufA = smem;
    float* bufB = bufA + TM * ldx;
    float* whs = bufB + TM * ldx;                 // [8][HL + 4] head weights, transposed
    float* bhs = whs + 8 * (HL + 4);              // [8] head biases
    float* heads = bhs + 8;                       // [TM][NHP]
    uint32_t* obs = reinterpret_cast<uint32_t*>(heads + TM * NHP);   // [TM][OBS_WORDS]
    uint32_t* rng = obs + TM * OBS_WORDS;                            // [TM][4] draws of the current step
    float* bs = reinterpret_cast<float*>(rng + TM * 4);              // biases of the hidden layers
    int nb = 0;
    for (int l = 1; l <= L; ++l) nb += a.net.dims[l];
    float* pre = bs + nb;                                            // maze: [TM][H1] wall sums
    float* w1s = ENV == ENV_MAZE ? pre + TM * H1 : pre;              // first-layer weights, or (maze) agent plane + goal row

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * TM;
    const int B = a.B, T = a.T;
    const int rows_left = B - b0;                                    // environments of this tile (whole groups of 16)
    const TrajPtrs& tp = a.tp;
    const int ldw = HL + 4;
    const float* w1g = a.theta + a.net.w_off[0];
    for (int i = tid; i < HL * NH; i += STW + STA) whs[(i % NH) * ldw + i / NH] = round1<BF>(a.theta[a.net.wh_off + i]);
    if (tid < 8) bhs[tid] = tid < NH ? a.theta[a.net.bh_off + tid] : 0.0f;
    {
        int off = 0;
        for (int l = 0; l < L; ++l) {
            for (int i = tid; i < a.net.dims[l + 1]; i += STW + STA) bs[off + i] = a.theta[a.net.b_off[l] + i];
            off += a.net.dims[l + 1];
        }
    }
    if (sa.w1_lds) {
        const f4v* src = reinterpret_cast<const f4v*>(w1g + (ENV == ENV_MAZE ? (size_t)n_cells * H1 : 0));
        f4v* dst = reinterpret_cast<f4v*>(w1s);
        const int n4 = (ENV == ENV_MAZE ? n_cells : D) * H1 / 4;
        constexpr int NTH = STW + STA;
        for (int i0 = 0; i0 < n4; i0 += 4 * NTH) {
            f4v v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int i = i0 + u * NTH + tid; v[u] = src[i < n4 ? i : 0]; }
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int i = i0 + u * NTH + tid; if (i < n4) { round4<BF>(v[u]); dst[i] = v[u]; } }
        }
        if (ENV == ENV_MAZE)
            for (int i = tid; i < H1; i += NTH) w1s[(size_t)n_cells * H1 + i] = round1<BF>(w1g[(size_t)(3 * n_cells - 1) * H1 + i]);
    }
    const bool aux = wave >= STW / 64;                               // a scalar branch: what follows stays in scalar registers
    const int at = tid - STW;
    EnvState st{0u, 0.0f, 0.0f};
    const bool mine = aux && at < TM;                                // this thread's environment (rows past B: any valid state)
    const bool owner = mine && at < rows_left;
    const int b = b0 + (owner ? at : 0);
    if (mine) {
        if (!REPLAY) {
            st.s0 = tp.s0[b];
            if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
        }
        if (ENV == ENV_MAZE) for (int w = 0; w < 8; ++w) obs[at * OBS_WORDS + w] = tp.walls[(size_t)w * B + b];
    }
    if (ENV == ENV_MAZE) {
        __syncthreads();
        maze_prefix<BF, STW + STA>(a, TM, obs, w1g, bs, pre, tid);
    }
    const int t_begin = REPLAY ? (int)blockIdx.y * sa.tseg : 0;
    const int t_end = REPLAY ? (t_begin + sa.tseg < sa.tend ? t_begin + sa.tseg : sa.tend) : T + 1;
    EnvState nx{0u, 0.0f, 0.0f};                                     // REPLAY: the next step's state, asked for a step ahead
    auto ask = [&](int t) {
        const size_t tb = (size_t)(t < t_end ? t : t_end - 1) * B + b;
        nx.s0 = tp.tr_s0[tb];
        if (ENV == ENV_PENDULUM) { nx.f0 = tp.tr_f0[tb]; nx.f1 = tp.tr_f1[tb]; }
    };
    auto observe = [&](int t) {
        if (REPLAY) { st = nx; ask(t + 1); }
        else if (owner) {
            const size_t tb = (size_t)t * B + b;
            tp.tr_s0[tb] = st.s0;
            if (ENV == ENV_PENDULUM) { tp.tr_f0[tb] = st.f0; tp.tr_f1[tb] = st.f1; }
        }
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            obs[at * OBS_WORDS + 0] = (uint32_t)bc;
            obs[at * OBS_WORDS + 1] = (uint32_t)pc;
        } else if (ENV == ENV_PENDULUM) {
            float sn, cs;
            det_sincos(st.f0, sn, cs);
            obs[at * OBS_WORDS + 0] = bits_from_f(round1<BF>(cs));
            obs[at * OBS_WORDS + 1] = bits_from_f(round1<BF>(sn));
            obs[at * OBS_WORDS + 2] = bits_from_f(round1<BF>(st.f1));
        } else {
            obs[at * OBS_WORDS + 8] = st.s0 & 0xffffu;
        }
    };
    // h_l of the step from LDS to memory, 16 bytes a thread
    auto copy_out = [&](int t, int l, const float* src) {
        const int N = a.net.dims[l + 1], c4 = N >> 2, n4 = (TM < rows_left ? TM : rows_left) * c4;
        f4v* dst = reinterpret_cast<f4v*>(tp.act[l] + ((size_t)t * B + b0) * N);
        for (int i0 = at; i0 < n4; i0 += 4 * STA) {
            f4v v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * STA < n4 ? i0 + u * STA : i0;
                v[u] = *reinterpret_cast<const f4v*>(src + (i / c4) * ldx + ((i % c4) << 2));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) if (i0 + u * STA < n4) dst[i0 + u * STA] = v[u];
        }
    };
    if (REPLAY && mine) ask(t_begin);
    if (mine) observe(t_begin);
    __syncthreads();

    if (!aux) {
        // ==== the layers ====================================================
        uint32_t lg = 0;
        int widest = 0;
        for (int l = 1; l <= L; ++l) {
            const int d = a.net.dims[l];
            lg |= (uint32_t)(31 - __builtin_clz((uint32_t)d)) << (8 * (l - 1));
            if (l > 1 && d > widest) widest = d;
        }
        const StreamNet net{L, a.net.w_off[1], lg};
        const rsrc_w theta = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.theta), 0, (uint32_t)a.net.P * 4u, 0x00020000);
        float wA[8], wB[8];
        // a wavefront without a tile in any layer follows the stream of one that has
        const int sw = 16 * wave < widest ? wave : 0;
        StreamCursor sc{1, sw, 0, net.w1, net.dim(1), net.dim(2)};
        net.settle(sc, sw);
        stream_load(wA, theta, sc, lane); net.advance(sc, sw);
        __builtin_amdgcn_sched_barrier(0);
        stream_load(wB, theta, sc, lane); net.advance(sc, sw);
        __builtin_amdgcn_sched_barrier(0);
        for (int t = t_begin; t < t_end; ++t) {
            const int cg = H1 >> 2, cgs = 31 - __builtin_clz((uint32_t)cg);
            constexpr int FB = 4;                                    // (environment, four columns) pieces in flight
            for (int i0 = tid; i0 < TM * cg; i0 += FB * STW) {
                f4v wv[FB][ENV == ENV_PENDULUM ? 3 : 2], bv[FB];
#pragma unroll
                for (int u = 0; u < FB; ++u) {
                    const int i = i0 + u * STW < TM * cg ? i0 + u * STW : i0, m = i >> cgs, c = (i & (cg - 1)) << 2;
                    const uint32_t* o = obs + m * OBS_WORDS;
                    if (ENV == ENV_PENDULUM) {
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            if (sa.w1_lds) wv[u][k] = *reinterpret_cast<const f4v*>(w1s + k * H1 + c);
                            else { wv[u][k] = *reinterpret_cast<const f4v*>(w1g + k * H1 + c); round4<BF>(wv[u][k]); }
                        }
                        bv[u] = *reinterpret_cast<const f4v*>(bs + c);
                    } else {
                        const int r0 = ENV == ENV_CATCH ? (int)o[0] : (int)o[8], r1 = ENV == ENV_CATCH ? (int)o[1] : n_cells;
                        if (sa.w1_lds) {
                            wv[u][0] = *reinterpret_cast<const f4v*>(w1s + r0 * H1 + c);
                            wv[u][1] = *reinterpret_cast<const f4v*>(w1s + r1 * H1 + c);
                        } else {
                            wv[u][0] = *reinterpret_cast<const f4v*>(w1g + (size_t)(ENV == ENV_CATCH ? r0 : n_cells + r0) * H1 + c);
                            wv[u][1] = *reinterpret_cast<const f4v*>(w1g + (size_t)(ENV == ENV_CATCH ? r1 : 3 * n_cells - 1) * H1 + c);
                            round4<BF>(wv[u][0]); round4<BF>(wv[u][1]);
                        }
                        bv[u] = ENV == ENV_MAZE ? *reinterpret_cast<const f4v*>(pre + m * H1 + c) : *reinterpret_cast<const f4v*>(bs + c);
                    }
                }
#pragma unroll
                for (int u = 0; u < FB; ++u) {
                    const int i = i0 + u * STW;
                    if (i < TM * cg) {
                        const int m = i >> cgs, c = (i & (cg - 1)) << 2;
                        f4v v = bv[u];
                        if (ENV == ENV_PENDULUM) {
                            const uint32_t* o = obs + m * OBS_WORDS;
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const float x = f_from_bits(o[k]);
#pragma unroll
                                for (int e = 0; e < 4; ++e) v[e] = fmaf(x, wv[u][k][e], v[e]);
                            }
                        } else {
                            v += wv[u][0];
                            v += wv[u][1];
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
                        round4<BF>(v);
                        *reinterpret_cast<f4v*>(bufA + m * ldx + c) = v;
                    }
                }
            }
            __syncthreads();
            float* cur = bufA;
            float* nxt = bufB;
            const float* bias = bs + H1;
            for (int l = 1; l < L; ++l) {
                stream_layer<MT, BF>(net, theta, l, cur, nxt, ldx, bias, wave, lane, sc, wA, wB);
                bias += net.dim(l + 1);
                __syncthreads();
                float* tmp = cur; cur = nxt; nxt = tmp;
            }
            run_heads<STW>(cur, ldx, whs, ldw, bhs, heads, HL, NH, NHP, TM, tid);
            __syncthreads();
            __syncthreads();                                         // the environments step
        }
        return;
    }
    // ==== environments, draws and records; the same barriers ====================
    for (int t = t_begin; t < t_end; ++t) {
        const bool keep = t < T && a.keep_acts;                      // the bootstrap evaluation keeps no activations
        if (!REPLAY && t < T) {                                      // the step's draws do not depend on the network
            for (int i = STA - 1 - at; i < (ENV == ENV_MAZE ? TM : 2 * TM); i += STA) {
                const int e = i < TM ? i : i - TM;
                const u32x4 w = philox(a.seed, (uint32_t)(b0 + e), a.gstep + (uint64_t)t, i < TM ? DOM_ACTION : DOM_RESET);
                const uint32_t w0 = (ENV == ENV_PENDULUM && i < TM) ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;
                *reinterpret_cast<uint2*>(rng + e * 4 + (i < TM ? 0 : 2)) = make_uint2(w0, w.y);
            }
        }
        __syncthreads();
        const float* cur = bufA;
        const float* nxt = bufB;
        for (int l = 1; l < L; ++l) {
            if (keep) copy_out(t, l - 1, cur);
            __syncthreads();
            const float* tmp = cur; cur = nxt; nxt = tmp;
        }
        if (keep) copy_out(t, L - 1, cur);
        __syncthreads();
        if (at >= 64 && at < 64 + TM && at - 64 < rows_left) {
            const int e = at - 64;
            const size_t te = (size_t)t * B + b0 + e;
            const float4 h0 = ld4(heads + e * NHP);
            const float4 h1 = NHP == 8 ? ld4(heads + e * NHP + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float* hd = tp.tr_head + te * NHP;
            *reinterpret_cast<float4*>(hd) = h0;
            if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = h1;
            tp.tr_val[te] = last_head(h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w, NH);
        }
        if (mine && !REPLAY && t < T) {
            const float4 h0 = ld4(heads + at * NHP);
            const float4 h1 = NHP == 8 ? ld4(heads + at * NHP + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const uint4 dr = *reinterpret_cast<const uint4*>(rng + at * 4);   // action draw, reset draw
            const size_t tb = (size_t)t * B + b;
            float r; int done;
            if (ENV == ENV_PENDULUM) {
                const float eps = f_from_bits(dr.x);
                const float act = gaussian_action(h0.x, h0.y, eps);
                pendulum_step(a.env, st, act, dr.z, dr.w, r, done);
                if (owner) { tp.tr_eps[tb] = eps; tp.tr_actf[tb] = act; }
            } else {
                const int act = sample_categorical_any(h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w, a.net.A, u01(dr.x));
                if (ENV == ENV_CATCH) catch_step(a.env, st, act, dr.z, r, done);
                else {
                    const uint32_t* wl = obs + at * OBS_WORDS;
                    maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, r, done);
                }
                if (owner) tp.tr_act[tb] = (uint8_t)act;
            }
            if (owner) { tp.tr_rew[tb] = r; tp.tr_done[tb] = (uint8_t)done; }
        }
        if (mine && t + 1 < t_end) observe(t + 1);
        __syncthreads();
    }
    if (!REPLAY && owner) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// ---------------------------------------------------------------------------
// Weights resident on chip.  For two-layer nets up to 256 x 256 the whole hidden-to-hidden matrix fits the register file
// of one compute unit: a CU has 4 SIMDs x 512 registers x 64 lanes x 4 B = 512 KB, W2 (256 x 256 fp32) is 256 KB, 128
// registers per lane over eight wavefronts.  Each lane loads, once per launch, exactly the B-operand values it will feed to
// the matrix cores -- W2[k][its columns] for its k phase -- and reuses them for all T+1 forward passes, so the acting loop
// reads no hidden-layer weight from memory at all.  The first layer's matrix (gathered by row) sits in LDS where it fits,
// the head matrix always.  The accumulation order is the canonical one.
//
// A step is a chain: the 256-wide layer on the matrix cores (8.2 k cycles for each 16 environments), then heads (2.1 k: 256
// dependent multiply-adds), sample, step, observe (1 k) and the next first layer.  The two kinds cannot overlap: a binary32
// MFMA and binary32 vector operations use the same units, and a wavefront that streams such MFMAs starves the vector work of
// the others on its SIMD (measured: 256 dependent operations beside such a stream end with it, whatever the priorities).
// What helps is two wavefronts per SIMD in the matrix layer (one alone left its gaps open: LDS, stores), nothing but the
// chain between the barriers, and no barrier inside it: one wavefront per group of 16 environments sums the heads, samples,
// steps and observes, the others meanwhile copy the activations out of LDS and make the next step's random draws; records
// go out beside the other wavefronts' MFMAs.  (Every wavefront taking two or four environments through the whole chain was
// slower: eight times the LDS reads for the head chains.)
// G groups of 16 environments per workgroup: 2 where one group each would need more compute units than there are.
// 256-256 pendulum, 8192 environments, T = 32: 25.4 k cycles a step with both operands of the head chains from LDS and the
// number of heads a run-time value (17 registers in scratch, whose reloads waited for the records' stores), 24.1 k now; Catch,
// 4096 environments, T = 20: 14.6 k and 14.1 k.  The registers that frees let a learner's workgroup share the unit: a
// decoupled step of the latter 416 -> 395 us.
// ---------------------------------------------------------------------------
constexpr int RES_WAVES = 8;

template <int ENV, int RW, int G, bool HOLD>
__global__ __launch_bounds__(64 * RES_WAVES) void rollout_resident_kernel(const RolloutArgs a, const int w1_lds)
{
    constexpr int NTHR = 64 * RES_WAVES, TM = 16 * G, EPW = TM / RES_WAVES, KS = RW / 4;
    constexpr int NT = RW / (16 * RES_WAVES);                      // column tiles of 16 per wavefront
    constexpr int LDX = RW + 4, LDW = RW + 4;
    constexpr int NE = 256 / RW < EPW ? 256 / RW : EPW, IT = EPW / NE;   // first layer: environments side by side, passes
    if (HOLD) asm volatile("" : : : "v159");                       // (see launch_resident_env)
    extern __shared__ float4 smem4[];
    float* X = reinterpret_cast<float*>(smem4);                    // [TM][LDX] first layer's outputs
    float* Y = X + TM * LDX;                                       // [TM][LDX] second layer's
    float* whs = Y + TM * LDX;                                     // [8][LDW] head weights, transposed
    float* b1s = whs + 8 * LDW;                                    // [RW] biases of the first layer
    uint32_t* rng = reinterpret_cast<uint32_t*>(b1s + RW);         // [2][TM][4] draws: the action's two words (pendulum: noise), the reset's
    uint32_t* obs = rng + 2 * TM * 4;                              // [TM][OBS_WORDS]: cells, features; maze: walls and the cell
    float* w1s = reinterpret_cast<float*>(obs + TM * OBS_WORDS);   // [D][RW] W1; maze: [TM][RW] wall sums
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH > 4 ? 8 : 4;   // actions, or mean and deviation, and the value
    const int D = a.net.dims[0], B = a.B, T = a.T;
    const int n_cells = a.env.rows * a.env.cols;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * TM, rows_left = B - b0;            // the last workgroup may have one group only
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];

    // what goes to LDS is asked for first, then this lane's share of W2, in matrix-core operand order; the former lands while
    // the latter streams in
    float wreg[KS][NT], bv[NT];
    {
        constexpr int NWH = (RW * 8 + NTHR - 1) / NTHR, W1B = 8;
        const f4v* w1src = reinterpret_cast<const f4v*>(w1g);
        f4v* w1dst = reinterpret_cast<f4v*>(w1s);
        const int n_w1 = ENV != ENV_MAZE && w1_lds ? D * RW / 4 : 0;
        float wv[NWH];
        f4v vw1[W1B];
#pragma unroll
        for (int u = 0; u < NWH; ++u) wv[u] = a.theta[a.net.wh_off + (tid + u * NTHR < RW * NH ? tid + u * NTHR : 0)];
        const float vb1 = a.theta[a.net.b_off[0] + (tid & (RW - 1))];
        if (ENV != ENV_MAZE) {
#pragma unroll
            for (int u = 0; u < W1B; ++u) vw1[u] = w1src[tid + u * NTHR < n_w1 ? tid + u * NTHR : 0];
        }
        __builtin_amdgcn_sched_barrier(0);
        const int col0 = wave * 16 * NT + NT * (lane & 15), kq = lane >> 4;
        load_nt<NT>(a.theta + a.net.b_off[1] + col0, bv);
#pragma unroll
        for (int s = 0; s < KS; ++s) load_nt<NT>(a.theta + a.net.w_off[1] + (size_t)(4 * s + kq) * RW + col0, wreg[s]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NWH; ++u) {
            const int i = tid + u * NTHR, kk = i / NH, j = i - kk * NH;
            if (i < RW * NH) whs[j * LDW + kk] = wv[u];
        }
        if (tid < RW) b1s[tid] = vb1;
        if (ENV != ENV_MAZE) {
#pragma unroll
            for (int u = 0; u < W1B; ++u) if (tid + u * NTHR < n_w1) w1dst[tid + u * NTHR] = vw1[u];
            for (int i0 = tid + W1B * NTHR; i0 < n_w1; i0 += W1B * NTHR) {
#pragma unroll
                for (int u = 0; u < W1B; ++u) vw1[u] = w1src[i0 + u * NTHR < n_w1 ? i0 + u * NTHR : 0];
#pragma unroll
                for (int u = 0; u < W1B; ++u) if (i0 + u * NTHR < n_w1) w1dst[i0 + u * NTHR] = vw1[u];
            }
        } else {
            for (int i = tid; i < TM * 8; i += NTHR) {
                const int m = i >> 3, w = i & 7;
                obs[m * OBS_WORDS + w] = tp.walls[(size_t)w * B + b0 + (m < rows_left ? m : 0)];
            }
            __syncthreads();
            maze_prefix<false, NTHR>(a, TM, obs, w1g, b1s, w1s, tid);
        }
    }
    // Wavefront g < G owns the environments of group g: lane e + 16 j sums heads j and j + 4 of environment e, lane e steps
    // it.  In the first layer every wavefront takes EPW rows.
    // A group that does not exist (B an odd multiple of 16, G = 2) stands in the state of the tile's first environment for the
    // whole unroll and shows that: every wavefront's first layer runs on all rows, so each needs an observation that is a
    // valid index into W1.
    const int m0 = EPW * wave;
    const bool live = m0 < rows_left, owner = wave < G && 16 * wave < rows_left;   // (of the wavefront)
    EnvState st{0u, 0.0f, 0.0f};
    {
        const int b = b0 + (owner ? 16 * wave + (lane & 15) : 0);
        st.s0 = tp.s0[b];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
    }
    const int c = (lane * 4) & (RW - 1);                           // first layer: this lane's columns
    f4v wp[3];                                                     // pendulum: three rows; maze: the goal's row
    if (ENV == ENV_PENDULUM) {
#pragma unroll
        for (int k = 0; k < 3; ++k) wp[k] = *reinterpret_cast<const f4v*>(w1g + k * RW + c);
    } else if (ENV == ENV_MAZE) wp[0] = *reinterpret_cast<const f4v*>(w1g + (size_t)(3 * n_cells - 1) * RW + c);
    const float hbias0 = a.theta[a.net.bh_off + ((lane >> 4) < NH ? lane >> 4 : 0)], hbias1 = a.theta[a.net.bh_off + ((lane >> 4) + 4 < NH ? (lane >> 4) + 4 : 0)];
    __syncthreads();
    const f4v b1v = *reinterpret_cast<const f4v*>(b1s + c);
    // Everything loaded so far has arrived before the loop starts: inside it a wait for a load would be a wait for every
    // older store of the wavefront as well (loads and stores complete in issue order).
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0)

    float sine = 0.0f;                                             // pendulum: of the angle as observed
    auto observe = [&](int lane) {
        if (wave >= G || lane >= 16) return;
        uint32_t* o = obs + (16 * wave + lane) * OBS_WORDS;
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            o[0] = (uint32_t)bc; o[1] = (uint32_t)pc;
        } else if (ENV == ENV_PENDULUM) {
            float cs;
            det_sincos(st.f0, sine, cs);
            o[0] = bits_from_f(cs); o[1] = bits_from_f(sine); o[2] = bits_from_f(st.f1);
        } else o[8] = st.s0 & 0xffffu;
    };
    auto draw = [&](int t, int lane) {                             // (one wavefront)
        if (lane >= 2 * TM) return;
        const int m = lane & (TM - 1);
        const bool reset = lane >= TM;
        const u32x4 w = philox(a.seed, (uint32_t)(b0 + m), a.gstep + (uint64_t)t, reset ? DOM_RESET : DOM_ACTION);
        const uint32_t w0 = (ENV == ENV_PENDULUM && !reset) ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;
        *reinterpret_cast<uint2*>(rng + ((t & 1) * TM + m) * 4 + (reset ? 2 : 0)) = make_uint2(w0, w.y);
    };
    f4v h1[IT];                                                    // first layer of the step that comes next
    // (lane: handed in, see the time loop)
    auto first = [&](int lane) {
        const int c = (lane * 4) & (RW - 1), sub = lane / (RW / 4);
        const uint32_t* o = obs + (m0 + (sub < NE ? sub : 0)) * OBS_WORDS;
#pragma unroll
        for (int it = 0; it < IT; ++it, o += NE * OBS_WORDS) {
            f4v v;
            if (ENV == ENV_PENDULUM) {
                v = b1v;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float x = f_from_bits(o[k]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = fmaf(x, wp[k][q], v[q]);
                }
            } else if (ENV == ENV_CATCH) {
                const int r0 = (int)o[0], r1 = (int)o[1];
                f4v x0, x1;
                if (w1_lds) { x0 = *reinterpret_cast<const f4v*>(w1s + r0 * RW + c); x1 = *reinterpret_cast<const f4v*>(w1s + r1 * RW + c); }
                else { x0 = *reinterpret_cast<const f4v*>(w1g + r0 * RW + c); x1 = *reinterpret_cast<const f4v*>(w1g + r1 * RW + c); }
                v = (b1v + x0) + x1;
            } else {
                const f4v x0 = *reinterpret_cast<const f4v*>(w1g + (size_t)(n_cells + (int)o[8]) * RW + c);
                v = (*reinterpret_cast<const f4v*>(w1s + (m0 + it * NE + (sub < NE ? sub : 0)) * RW + c) + x0) + wp[0];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = v[q] > 0.0f ? v[q] : 0.0f;
            h1[it] = v;
        }
        if (sub < NE) {
#pragma unroll
            for (int it = 0; it < IT; ++it) *reinterpret_cast<f4v*>(X + (m0 + it * NE + sub) * LDX + c) = h1[it];
        }
    };
    // Records, as stores without branches (what is not to be written has a descriptor of no bytes): they go between the MFMAs
    // of the next matrix layer, where the other wavefront of the SIMD covers them.  On their own, all wavefronts at once,
    // they took 0.6 to 0.9 k cycles of every step.
    auto rsrc = [&](const void* p, bool on) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, on ? 0x7fffffffu : 0u, 0x00020000); };
    auto store_h1 = [&](int t, int it, int lane) {                 // piece it of the first layer of step t
        const rsrc_w d = rsrc(tp.act[0] + ((size_t)t * B + b0 + m0) * RW, t < T && a.keep_acts && live);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v_w, h1[it]), d, lane / (RW / 4) < NE ? 16 * lane : -1, NE * RW * 4 * it, 0);
    };
    float hv0 = 0.0f, hv1 = 0.0f, rew = 0.0f, actf = 0.0f, eps = 0.0f;
    int act = 0, done = 0;
    auto store_state = [&](int t, int lane) {                      // what step t shows
        const size_t te = (size_t)t * B + b0 + 16 * wave;
        const int o4 = lane < 16 ? 4 * lane : -1;
        __builtin_amdgcn_raw_buffer_store_b32(st.s0, rsrc(tp.tr_s0 + te, true), o4, 0, 0);
        if (ENV == ENV_PENDULUM) {
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f0), rsrc(tp.tr_f0 + te, true), o4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(st.f1), rsrc(tp.tr_f1 + te, true), o4, 0, 0);
        }
    };
    auto store_heads = [&](int t, bool on, int lane) {
        const size_t te = (size_t)t * B + b0 + 16 * wave;
        const int e = lane & 15, j = lane >> 4;
        const rsrc_w d = rsrc(tp.tr_head + te * NHP, on);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(j < NH ? hv0 : 0.0f), d, 4 * (e * NHP + j), 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(j + 4 < NH ? hv1 : 0.0f), d, NHP == 8 ? 4 * (e * NHP + 4 + j) : -1, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(NH > 4 ? hv1 : hv0), rsrc(tp.tr_val + te, on), j == ((NH - 1) & 3) ? 4 * e : -1, 0, 0);
    };
    auto store_step = [&](int t, bool on, int lane) {              // what was done in step t
        const size_t te = (size_t)t * B + b0 + 16 * wave;
        const int o4 = lane < 16 ? 4 * lane : -1, o1 = lane < 16 ? lane : -1;
        if (ENV == ENV_PENDULUM) {
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(eps), rsrc(tp.tr_eps + te, on), o4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(actf), rsrc(tp.tr_actf + te, on), o4, 0, 0);
        } else __builtin_amdgcn_raw_buffer_store_b8((uint8_t)act, rsrc(tp.tr_act + te, on), o1, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(bits_from_f(rew), rsrc(tp.tr_rew + te, on), o4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)done, rsrc(tp.tr_done + te, on), o1, 0, 0);
    };
    observe(lane);
    if (wave == RES_WAVES - 1) draw(0, lane);
    __syncthreads();
    first(lane);
    __syncthreads();
    const int lane0 = lane;
    for (int t = 0; t <= T; ++t) {
        // everything derived from the lane is worked out again every step from a value the compiler cannot see through:
        // dozens of loop-invariant addresses would otherwise be kept in registers, on top of the weights, and spilled
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        const int col0 = wave * 16 * NT + NT * (lane & 15), kq = lane >> 4;
        // ---- the matrix layer ----
        {
            const float* xp = X + (lane & 15) * LDX + kq;
            f4v acc[G][NT];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int n = 0; n < NT; ++n) { acc[g][n][0] = bv[n]; acc[g][n][1] = bv[n]; acc[g][n][2] = bv[n]; acc[g][n][3] = bv[n]; }
            constexpr int PF = 8;                                  // LDS reads run this many steps ahead of their MFMAs
            float ap[PF][G];
#pragma unroll
            for (int u = 0; u < PF; ++u)
#pragma unroll
                for (int g = 0; g < G; ++g) ap[u][g] = xp[16 * g * LDX + 4 * u];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                float av[G];
#pragma unroll
                for (int g = 0; g < G; ++g) { av[g] = ap[s % PF][g]; if (s + PF < KS) ap[s % PF][g] = xp[16 * g * LDX + 4 * (s + PF)]; }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[g][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[g], wreg[s][n], acc[g][n], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (s % 2 == 0 && s / 2 < IT) store_h1(t, s / 2, lane);
                if (owner) {
                    if (s == 9) store_state(t, lane);
                    if (s == 11) store_heads(t - 1, t > 0, lane);
                    if (s == 13) store_step(t - 1, t > 0, lane);
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float o[NT];
#pragma unroll
                    for (int n = 0; n < NT; ++n) o[n] = acc[g][n][r] > 0.0f ? acc[g][n][r] : 0.0f;
                    store_nt<NT>(Y + (16 * g + 4 * kq + r) * LDX + col0, o);
                }
        }
        float wh[RW / 16];                                             // head weights of the row's head, input 16 s + lane (they never change)
        if (owner) {
            const int e = lane & 15, j = lane >> 4;
#pragma unroll
            for (int s = 0; s < RW / 16; ++s) wh[s] = whs[(j < NH ? j : 0) * LDW + 16 * s + e];
        }
        __syncthreads();
        asm volatile("" : "+v"(lane));
        hv0 = hbias0; hv1 = hbias1;
        if (owner) {
            // ---- head chains ----
            const int e = lane & 15;
            // The chain is bound by what one wavefront issues: a multiply-add four cycles, everything between them as much
            // again.  Of its operands the environment's activations are read 16 bytes at a time; the head's weights sit in
            // the lanes of the row, sixteen to a register, and reach the multiply-add as its row broadcast.  (Both read from
            // LDS: 2.6 k cycles for 256 inputs.)
            const f4v* x = reinterpret_cast<const f4v*>(Y + (16 * wave + e) * LDX);
            constexpr int S = RW / 8, PF = 4;                      // pieces of eight inputs; read this many ahead
            f4v xr[PF][2];
#pragma unroll
            for (int u = 0; u < PF; ++u) { xr[u][0] = x[2 * u]; xr[u][1] = x[2 * u + 1]; }
            float w2[NH > 4 ? RW / 16 : 1];
            if (NH > 4) {
#pragma unroll
                for (int s = 0; s < RW / 16; ++s) w2[NH > 4 ? s : 0] = whs[4 * LDW + 16 * s + e];
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const f4v x0 = xr[s % PF][0], x1 = xr[s % PF][1];
                __builtin_amdgcn_sched_barrier(0);
                if (s % 2 == 0) { chain8<0>(wh[s / 2], x0, x1, hv0); if (NH > 4) chain8<0>(w2[NH > 4 ? s / 2 : 0], x0, x1, hv1); }
                else { chain8<8>(wh[s / 2], x0, x1, hv0); if (NH > 4) chain8<8>(w2[NH > 4 ? s / 2 : 0], x0, x1, hv1); }
                __builtin_amdgcn_sched_barrier(0);
                if (s + PF < S) { xr[s % PF][0] = x[2 * (s + PF)]; xr[s % PF][1] = x[2 * (s + PF) + 1]; }
            }
            if (t < T) {
                // ---- sample, step, observe ----
                float h[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) h[q] = __shfl(hv0, e + 16 * q, 64);
#pragma unroll
                for (int q = 0; q < 4; ++q) h[4 + q] = NH > 4 ? __shfl(hv1, e + 16 * q, 64) : 0.0f;
                if (lane < 16) {
                    const uint4 d = *reinterpret_cast<const uint4*>(rng + ((t & 1) * TM + 16 * wave + e) * 4);
                    if (ENV == ENV_PENDULUM) {
                        eps = f_from_bits(d.x);
                        actf = gaussian_action(h[0], h[1], eps);
                        pendulum_step_sn(a.env, st, sine, actf, d.z, d.w, rew, done);
                    } else {
                        act = sample_categorical_any(h[0], h[1], h[2], h[3], h[4], h[5], h[6], h[7], a.net.A, u01(d.x));
                        if (ENV == ENV_CATCH) catch_step(a.env, st, act, d.z, rew, done);
                        else {
                            const uint32_t* wl = obs + (16 * wave + e) * OBS_WORDS;
                            maze_step(a.env, st, act, [wl](int cc) { return ((wl[cc >> 5] >> (cc & 31)) & 1u) != 0u; }, rew, done);
                        }
                    }
                }
                observe(lane);
            }
        }
        if (wave >= RES_WAVES / 2 && t < T) {
            // ---- meanwhile: the second layer's record, the next draws ----
            if (a.keep_acts) {
                const int at = (wave - RES_WAVES / 2) * 64 + lane, n4 = (TM < rows_left ? TM : rows_left) * (RW / 4);
                f4v* dst = reinterpret_cast<f4v*>(tp.act[1] + ((size_t)t * B + b0) * RW);
                constexpr int NC = TM * RW / 4 / 256;
                f4v v[NC];
#pragma unroll
                for (int u = 0; u < NC; ++u) { const int i = at + 256 * u; v[u] = *reinterpret_cast<const f4v*>(Y + (i / (RW / 4)) * LDX + 4 * (i % (RW / 4))); }
#pragma unroll
                for (int u = 0; u < NC; ++u) { const int i = at + 256 * u; if (i < n4) dst[i] = v[u]; }
            }
        }
        if (wave == RES_WAVES - 1 && t < T) draw(t + 1, lane);
        if (t == T) { if (owner) store_heads(t, true, lane); break; }
        __syncthreads();
        // ---- next first layer ----
        asm volatile("" : "+v"(lane));
        first(lane);
        __syncthreads();
    }
    if (owner && lane < 16) {
        const int b = b0 + 16 * wave + lane;
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// The same for 64-wide layers, four wavefronts and 16 environments, for the batches that rollout_small_ok leaves: a step is
// latency only (the layer on the matrix cores 1.0 k cycles, heads 0.8 k, sample and step 1.1 k of 3.5 k), and fewer wavefronts
// with everything they store where they compute it are quicker than the form above (T = 20, Catch: 64 environments, which
// rollout_small_kernel has now, 34 us against 40; 8192, which this has, 43).
template <int KS, int NT>
__device__ __forceinline__ void resident_m16(const float (&wreg)[KS][NT], const float* __restrict__ X, float* __restrict__ Y,
                                             int ldx, const float* __restrict__ bias, int N, int tid, float* __restrict__ gout)
{
    const int lane = tid & 63, wave = tid >> 6;
    const int col0 = wave * (N >> 2) + NT * (lane & 15), kq = lane >> 4;
    f4v acc[NT];
    {
        float bv[NT];
        load_nt<NT>(bias + col0, bv);
#pragma unroll
        for (int t = 0; t < NT; ++t) { acc[t][0] = bv[t]; acc[t][1] = bv[t]; acc[t][2] = bv[t]; acc[t][3] = bv[t]; }
    }
    const float* xp = X + (lane & 15) * ldx + kq;
    // the activation operand of step s + PF is read from LDS before the MFMAs of step s are issued: with one
    // wavefront per SIMD nothing else would hide the LDS latency
    constexpr int PF = 4;
    float ap[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u) ap[u] = xp[4 * u];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const float av = ap[s % PF];
        ap[s % PF] = xp[4 * (s + PF < KS ? s + PF : 0)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, wreg[s][t], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 4 * kq + r;
        float o[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) o[t] = acc[t][r] > 0.0f ? acc[t][r] : 0.0f;
        store_nt<NT>(Y + row * ldx + col0, o);
        if (gout) store_nt<NT>(gout + (size_t)row * N + col0, o);
    }
}

template <int ENV>
__global__ __launch_bounds__(WG) void rollout_resident64_kernel(const RolloutArgs a)
{
    constexpr int RK = 64, RN = 64, TM = 16;
    constexpr int KS = RK / 4, NT = RN / 64;                       // MFMA k-steps per forward pass, tiles per wavefront
    constexpr bool W1_IN_LDS = ENV != ENV_MAZE;
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    constexpr int HL = RN;
    const int ldx = a.ldx, NH = a.net.NH, NHP = a.net.NHP, D = a.net.dims[0];
    float* bufA = smem;
    float* bufB = bufA + TM * ldx;
    float* whs = bufB + TM * ldx;                 // [8][HL + 4] head weights, transposed
    float* bhs = whs + 8 * (HL + 4);              // [8] head biases
    float* heads = bhs + 8;                       // [TM][NHP]
    uint32_t* obs = reinterpret_cast<uint32_t*>(heads + TM * NHP);   // [TM][OBS_WORDS]
    uint32_t* rng = obs + TM * OBS_WORDS;                            // [TM][4] draws of the current step
    float* b1s = reinterpret_cast<float*>(rng + TM * 4);             // [RK], [RN] biases of the two hidden layers
    float* b2s = b1s + RK;
    float* w1s = b2s + RN;                                           // [D][RK] first-layer weights (maze: [TM][RK] prefix)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b0 = blockIdx.x * TM;
    const int B = a.B, T = a.T;
    const TrajPtrs& tp = a.tp;

    // The prologue's loads are issued in batches and land while the hidden-to-hidden matrix streams into the
    // registers: one load, one wait, one LDS store at a time would cost a memory round trip per 4 KB.
    constexpr int ldw = HL + 4;
    constexpr int NWH = HL * 8 / WG;                               // head-matrix elements per lane, at most
    constexpr int W1B = 8;                                         // 16-byte pieces of W1 per lane and batch
    static_assert(RK <= WG && RN <= WG, "one bias element per lane");
    const f4v* w1src = reinterpret_cast<const f4v*>(a.theta + a.net.w_off[0]);
    f4v* w1dst = reinterpret_cast<f4v*>(w1s);
    const int n_w1 = W1_IN_LDS ? D * RK / 4 : 0;
    float vwh[NWH];
    f4v vw1[W1B];
#pragma unroll
    for (int u = 0; u < NWH; ++u) {
        const int i = tid + u * WG;
        vwh[u] = a.theta[a.net.wh_off + (i < HL * NH ? i : 0)];     // unconditional: the stores below select
    }
    const float vbh = a.theta[a.net.bh_off + (tid < NH ? tid : 0)];
    const float vb1 = a.theta[a.net.b_off[0] + (tid < RK ? tid : 0)];
    const float vb2 = a.theta[a.net.b_off[1] + (tid < RN ? tid : 0)];
#pragma unroll
    for (int u = 0; u < W1B; ++u) {
        const int i = tid + u * WG;
        if (W1_IN_LDS) vw1[u] = w1src[i < n_w1 ? i : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
    const float* w1 = W1_IN_LDS ? w1s : a.theta + a.net.w_off[0];

    // this lane's share of W2, in matrix-core operand order
    float wreg[KS][NT];
    {
        const float* W2 = a.theta + a.net.w_off[1];
        const int col0 = wave * (RN >> 2) + NT * (lane & 15);
        const int kq = lane >> 4;
#pragma unroll
        for (int s = 0; s < KS; ++s) load_nt<NT>(W2 + (size_t)(4 * s + kq) * RN + col0, wreg[s]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NWH; ++u) {
        const int i = tid + u * WG;
        const int k = i / NH, j = i - k * NH;
        if (i < HL * NH) whs[j * ldw + k] = vwh[u];
    }
    if (tid < 8) bhs[tid] = tid < NH ? vbh : 0.0f;
    if (tid < RK) b1s[tid] = vb1;
    if (tid < RN) b2s[tid] = vb2;
#pragma unroll
    for (int u = 0; u < W1B; ++u) {
        const int i = tid + u * WG;
        if (i < n_w1) w1dst[i] = vw1[u];
    }
    for (int i0 = W1B * WG; i0 < n_w1; i0 += W1B * WG) {
#pragma unroll
        for (int u = 0; u < W1B; ++u) {
            const int i = i0 + tid + u * WG;
            vw1[u] = w1src[i < n_w1 ? i : 0];
        }
#pragma unroll
        for (int u = 0; u < W1B; ++u) {
            const int i = i0 + tid + u * WG;
            if (i < n_w1) w1dst[i] = vw1[u];
        }
    }

    EnvState st{0u, 0.0f, 0.0f};
    const bool owner = tid < TM;
    const int b = b0 + tid;
    if (owner) {
        st.s0 = tp.s0[b];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
        if (ENV == ENV_MAZE) {
            for (int w = 0; w < 8; ++w) obs[tid * OBS_WORDS + w] = tp.walls[(size_t)w * B + b];
        }
    }
    if (ENV == ENV_MAZE) {
        __syncthreads();
        maze_prefix<false, WG>(a, TM, obs, w1, b1s, w1s, tid);
    }

    // Everything loaded so far (weights, the envs' states) has arrived before the loop starts.  Inside the
    // loop the acting path then only stores to memory, and no step waits for an earlier step's stores: a
    // wait for a load would be a wait for every older store of the wavefront as well.
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0)

    for (int t = 0; t <= T; ++t) {
        const size_t tb = (size_t)t * B + b;
        if (owner) {
            tp.tr_s0[tb] = st.s0;
            if (ENV == ENV_PENDULUM) { tp.tr_f0[tb] = st.f0; tp.tr_f1[tb] = st.f1; }
            if (ENV == ENV_CATCH) {
                int bc, pc;
                catch_obs_cells(a.env, st.s0, bc, pc);
                obs[tid * OBS_WORDS + 0] = (uint32_t)bc;
                obs[tid * OBS_WORDS + 1] = (uint32_t)pc;
            } else if (ENV == ENV_PENDULUM) {
                float sn, cs;
                det_sincos(st.f0, sn, cs);
                obs[tid * OBS_WORDS + 0] = bits_from_f(cs);
                obs[tid * OBS_WORDS + 1] = bits_from_f(sn);
                obs[tid * OBS_WORDS + 2] = bits_from_f(st.f1);
            } else {
                obs[tid * OBS_WORDS + 8] = st.s0 & 0xffffu;
            }
        }
        __syncthreads();
        const bool keep = t < T && a.keep_acts;
        float* g0 = keep ? tp.act[0] + ((size_t)t * B + b0) * RK : nullptr;
        first_layer<ENV, TM * RK / 1024, false>(a, obs, bufA, ldx, tid, g0, w1, b1s, ENV == ENV_MAZE ? w1s : nullptr);
        __syncthreads();
        float* g1 = keep ? tp.act[1] + ((size_t)t * B + b0) * RN : nullptr;
        resident_m16<KS, NT>(wreg, bufA, bufB, ldx, b2s, RN, tid, g1);
        __syncthreads();
        heads_pipe<4, HL>(bufB, ldx, whs, ldw, bhs, heads, NH, NHP, TM, tid);
        // the step's random draws do not depend on the network: the last lanes of the workgroup,
        // idle during the head chains, produce them now -- the action draw of every env and the draw
        // that places the next episode, which then costs nothing where an episode ends
        if (t < T) {
            for (int i = WG - 1 - tid; i < (ENV == ENV_MAZE ? TM : 2 * TM); i += WG) {
                const int e = i < TM ? i : i - TM;
                const u32x4 w = philox(a.seed, (uint32_t)(b0 + e), a.gstep + (uint64_t)t, i < TM ? DOM_ACTION : DOM_RESET);
                // the pendulum's noise is ready-made when the heads are: only z and tanh remain on the critical path
                const uint32_t w0 = (ENV == ENV_PENDULUM && i < TM) ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;
                *reinterpret_cast<uint2*>(rng + e * 4 + (i < TM ? 0 : 2)) = make_uint2(w0, w.y);
            }
        }
        __syncthreads();
        // the record of the head outputs is written by the second wavefront, which has nothing else to do here:
        // the lanes that sample and step the envs are the critical path of the whole workgroup (handing the rest
        // of the step's record -- state, action, reward, episode end -- to idle lanes through LDS as well was
        // measured: no further gain)
        if (tid >= 64 && tid < 64 + TM) {
            const int e = tid - 64;
            const size_t te = (size_t)t * B + b0 + e;
            const float4 h0 = ld4(heads + e * NHP);
            const float4 h1 = NHP == 8 ? ld4(heads + e * NHP + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float* hd = tp.tr_head + te * NHP;
            *reinterpret_cast<float4*>(hd) = h0;
            if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = h1;
            tp.tr_val[te] = last_head(h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w, NH);
        }
        if (owner) {
            const float4 h0 = ld4(heads + tid * NHP);
            const float4 h1 = NHP == 8 ? ld4(heads + tid * NHP + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const float hv[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
            if (t < T) {
                const uint4 dr = *reinterpret_cast<const uint4*>(rng + tid * 4);   // action draw, reset draw
                float r; int done;
                if (ENV == ENV_PENDULUM) {
                    const float eps = f_from_bits(dr.x);
                    const float act = gaussian_action(hv[0], hv[1], eps);
                    tp.tr_eps[tb] = eps;
                    tp.tr_actf[tb] = act;
                    pendulum_step(a.env, st, act, dr.z, dr.w, r, done);
                } else {
                    const int act = sample_categorical_any(hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], a.net.A, u01(dr.x));
                    tp.tr_act[tb] = (uint8_t)act;
                    if (ENV == ENV_CATCH) {
                        catch_step(a.env, st, act, dr.z, r, done);
                    } else {
                        const uint32_t* wl = obs + tid * OBS_WORDS;
                        maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, r, done);
                    }
                }
                tp.tr_rew[tb] = r;
                tp.tr_done[tb] = (uint8_t)done;
            }
        }
    }
    if (owner) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// ---------------------------------------------------------------------------
// One hidden layer of at most 64 units on a Catch board or the pendulum's three features: the
// whole agent fits one lane.  Lane b keeps its env's state and the H hidden activations in
// registers, gathers its two first-layer rows (or takes three fmas per unit) from an LDS copy
// of W1, runs the NH head chains with the head matrix broadcast from LDS, draws its own random
// numbers, samples, steps and records -- no exchange between lanes, so no barrier inside the
// time loop, and every vector instruction works for 64 envs.  The arithmetic per env is the
// same canonical chain as in rollout_kernel.  No hidden activations are kept: the update of
// such nets rebuilds the layer from the state.  Bound by what the wavefronts issue.  Catch 10 x 5, 32 units, 262144
// environments, T = 16: 72.8 us with the heads as multiply-adds on operands from LDS, 55.9 on the matrix instruction and
// with four wavefronts per SIMD.
// ---------------------------------------------------------------------------
template <int ENV, int H, bool REPLAY>
__global__ __launch_bounds__(WG, H == 32 ? 4 : 2) void rollout_lane_kernel(const RolloutArgs a)
{
    constexpr int LDW = H + 4;                                    // row stride of W1 in LDS
    extern __shared__ float4 smem4[];
    float* w1s = reinterpret_cast<float*>(smem4);                 // [D][LDW]
    constexpr int NH = ENV == ENV_CATCH ? 4 : 3, NHP = 4;          // actions, or mean and deviation, and the value
    const int D = a.net.dims[0];
    float* b1s = w1s + D * LDW;                                   // [H]
    float* whs = b1s + H;                                         // [H][4] head weights, k-major, columns >= NH zero
    const int tid = threadIdx.x;
    // the parameters come into LDS in batches of eight loads per thread: one load, one wait, one store at a time
    // would be a memory round trip per KB
    {
        const float vb1 = a.theta[a.net.b_off[0] + (tid < H ? tid : 0)];
        constexpr int NW = (H * 4 + WG - 1) / WG;
        float vwh[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int i = q * WG + tid, k = i >> 2, j = i & 3;
            vwh[q] = a.theta[a.net.wh_off + ((i < H * 4 && j < NH) ? k * NH + j : 0)];
        }
        const float* w1g = a.theta + a.net.w_off[0];
        const int n = D * H;
        for (int i0 = 0; i0 < n; i0 += 8 * WG) {
            float pw[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) { const int i = i0 + q * WG + tid; pw[q] = w1g[i < n ? i : 0]; }
#pragma unroll
            for (int q = 0; q < 8; ++q) { const int i = i0 + q * WG + tid; if (i < n) w1s[(i / H) * LDW + i % H] = pw[q]; }
        }
        if (tid < H) b1s[tid] = vb1;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int i = q * WG + tid, j = i & 3;
            if (i < H * 4) whs[i] = j < NH ? vwh[q] : 0.0f;
        }
    }
    __syncthreads();

    const int B = a.B, T = a.T;
    const int b = blockIdx.x * WG + tid;
    if (b >= B) return;
    const TrajPtrs& tp = a.tp;
    float wh[H];                                                  // head weights of this lane's head, tid % 4
#pragma unroll
    for (int k = 0; k < H; ++k) wh[k] = whs[4 * k + (tid & 3)];
    f4v bh;
#pragma unroll
    for (int j = 0; j < 4; ++j) bh[j] = j < NH ? a.theta[a.net.bh_off + j] : 0.0f;
    EnvState st{0u, 0.0f, 0.0f};
    if (!REPLAY) {
        st.s0 = tp.s0[b];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
    }
    const int t_end = REPLAY ? T + a.bootstrap : T + 1;
    for (int t = 0; t < t_end; ++t) {
        const size_t tb = (size_t)t * B + b;
        if (REPLAY) {
            st.s0 = tp.tr_s0[tb];
            if (ENV == ENV_PENDULUM) { st.f0 = tp.tr_f0[tb]; st.f1 = tp.tr_f1[tb]; }
        } else {
            tp.tr_s0[tb] = st.s0;
            if (ENV == ENV_PENDULUM) { tp.tr_f0[tb] = st.f0; tp.tr_f1[tb] = st.f1; }
        }
        // the action draw does not depend on the network: issued first, used last
        u32x4 dr{0u, 0u, 0u, 0u};
        if (!REPLAY && t < T) dr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_ACTION);
        // ---- first layer -------------------------------------------------------
        float h[H];
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            const float* r0 = w1s + bc * LDW;
            const float* r1 = w1s + pc * LDW;
#pragma unroll
            for (int j = 0; j < H; j += 4) {
                const float4 bb = ld4(b1s + j), w0 = ld4(r0 + j), w1 = ld4(r1 + j);
                h[j] = (bb.x + w0.x) + w1.x; h[j + 1] = (bb.y + w0.y) + w1.y;
                h[j + 2] = (bb.z + w0.z) + w1.z; h[j + 3] = (bb.w + w0.w) + w1.w;
            }
        } else {
            float sn, cs;
            det_sincos(st.f0, sn, cs);
            const float x[3] = {cs, sn, st.f1};
#pragma unroll
            for (int j = 0; j < H; j += 4) {
                const float4 bb = ld4(b1s + j);
                float v[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float4 w = ld4(w1s + k * LDW + j);
                    v[0] = fmaf(x[k], w.x, v[0]); v[1] = fmaf(x[k], w.y, v[1]);
                    v[2] = fmaf(x[k], w.z, v[2]); v[3] = fmaf(x[k], w.w, v[3]);
                }
                h[j] = v[0]; h[j + 1] = v[1]; h[j + 2] = v[2]; h[j + 3] = v[3];
            }
        }
        // ---- heads: NH chains over k, ascending.  v_mfma_f32_4x4x1 multiplies the heads (rows, lane % 4) with four lanes'
        // environments (columns): register r of a lane is head r of its own environment, one instruction of eight cycles
        // an input where four multiply-adds took sixteen and an LDS read ----
        f4v hv = bh;
#pragma unroll
        for (int k = 0; k < H; ++k) hv = __builtin_amdgcn_mfma_f32_4x4x1f32(wh[k], h[k] > 0.0f ? h[k] : 0.0f, hv, 0, 0, 0);
        *reinterpret_cast<f4v*>(tp.tr_head + tb * NHP) = hv;
        tp.tr_val[tb] = hv[NH - 1];
        if (!REPLAY && t < T) {
            float r; int done;
            if (ENV == ENV_PENDULUM) {
                float eps, act;
                sample_gaussian(hv[0], hv[1], dr.x, dr.y, eps, act);
                tp.tr_eps[tb] = eps;
                tp.tr_actf[tb] = act;
                pendulum_step(a.env, st, act, 0u, 0u, r, done);
                if (done) {
                    const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                    pendulum_reset(st, wr.x, wr.y);
                }
            } else {
                const int act = sample_categorical_any(hv[0], hv[1], hv[2], 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 3, u01(dr.x));
                tp.tr_act[tb] = (uint8_t)act;
                catch_step(a.env, st, act, 0u, r, done);
                if (done) {
                    const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                    st.s0 = catch_reset(a.env, wr.x);
                }
            }
            tp.tr_rew[tb] = r;
            tp.tr_done[tb] = (uint8_t)done;
        }
    }
    if (!REPLAY) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// One-hidden-layer nets the lane kernel takes: width 32 or 64 on Catch or the pendulum, fp32, no kept activations -- and
// enough environments that a lane each fills the chip; with fewer a row of 16 lanes per environment (rollout_one.hip) is
// done sooner.  T = 16, a lane against 16 lanes, Catch 10 x 5 and the pendulum: width 32, 8192 environments 23.6 us against
// 16.5, 33.5 against 20.6; 16384 24.1 against 23.3, 35.2 against 29.4; 24576 24.7 against 29.8, 38.0 against 41.4.  Width 64:
// 16384 36.8 against 27.2, 48.3 against 34.6; 32768 37.6 against 46.4, 50.1 against 62.2.
static int rollout_lane_width(const anakin* h)
{
    const NetShape& n = h->net;
    if (n.bf16 || n.L != 1 || h->env.kind == ENV_MAZE || !one_layer_fused(h)) return 0;
    if (h->mode & (ANAKIN_MODE_CANONICAL_ACTING | ANAKIN_MODE_STREAM_WEIGHTS)) return 0;
    if ((n.dims[1] == 32 && h->B >= 24576) || (n.dims[1] == 64 && h->B >= 32768)) return n.dims[1];
    return 0;
}

template <int ENV, int H, bool REPLAY>
static hipError_t launch_lane(anakin* h, const RolloutArgs& a)
{
    const size_t lds = ((size_t)h->net.dims[0] * (H + 4) + H + H * 4) * 4;
    ProfScope prof(h, REPLAY ? "replay_forward" : "rollout");
    hipLaunchKernelGGL((rollout_lane_kernel<ENV, H, REPLAY>), dim3((h->B + WG - 1) / WG), dim3(WG), lds, h->stream, a);
    return hipGetLastError();
}

// which resident shape (if any) fits this net: 0 none, else the width (64, 128, 256)
int rollout_resident_width(const NetShape& net)
{
    if (net.bf16 || net.L != 2 || net.dims[1] != net.dims[2]) return 0;
    const int w = net.dims[1];
    return (w == 64 || w == 128 || w == 256) ? w : 0;
}
// LDS of the weights-resident kernel with G groups of 16 environments, with and without the first layer's weights
static size_t resident_lds_bytes(const NetShape& net, int env_kind, int G, bool w1)
{
    const size_t w = net.dims[1];
    size_t words = (size_t)2 * G * 16 * (w + 4) + 8 * (w + 4) + w + (size_t)16 * G * (8 + OBS_WORDS);
    if (env_kind == ENV_MAZE) words += (size_t)16 * G * w;
    else if (w1) words += (size_t)net.dims[0] * w;
    return words * 4;
}
// environments per workgroup: two groups of 16 as soon as one group each would not fit the chip's compute units at once
int rollout_resident_tile(const NetShape& net, int env_kind, int B)
{
    const int w = rollout_resident_width(net);
    if (w == 64) {
        // the 64-wide form always keeps W1 (maze: the tile's wall sums) and both biases in LDS: a board too large for that streams
        const size_t lds = rollout_lds_bytes(net, EnvDims{}, 16, nullptr) + (size_t)(2 + (env_kind == ENV_MAZE ? 16 : net.dims[0])) * w * 4;
        return lds <= 160 * 1024 ? 16 : 0;
    }
    return w ? (B > 16 * 256 ? 32 : 16) : 0;
}

// LDS of the streaming matrix-core kernel without / with the first layer's weights
static size_t stream_lds_bytes(const NetShape& net, const EnvDims& env, int TM, bool w1)
{
    size_t words = rollout_lds_bytes(net, env, TM, nullptr) / 4;
    for (int l = 1; l <= net.L; ++l) words += net.dims[l];
    if (env.kind == ENV_MAZE) words += (size_t)TM * net.dims[1];
    if (w1) words += (size_t)(env.kind == ENV_MAZE ? env.rows * env.cols + 1 : net.dims[0]) * net.dims[1];
    return words * 4;
}
// Environments per workgroup of the streaming matrix-core kernel, 0 where it does not apply: the largest of 16, 32 and 64
// that fits LDS and still leaves a workgroup per compute unit (an environment more per tile is an environment less that
// waits for another workgroup, but the weight stream is shared by the tile).
int rollout_pick_tile_mfma(const NetShape& net, const EnvDims& env, int B)
{
    if (net.L < 2) return 0;
    for (int l = 1; l < net.L; ++l) if (net.dims[l] % 64) return 0;     // blocks of 64 inputs
    int best = 0;
    for (int tm = 16; tm <= 64; tm *= 2) {
        if (stream_lds_bytes(net, env, tm, false) > 160 * 1024) break;
        if (!best || (B + tm - 1) / tm >= 256) best = tm;
    }
    return best;
}

size_t rollout_lds_bytes(const NetShape& net, const EnvDims&, int TM, int* ldx_out)
{
    int hmax = 0;
    for (int l = 1; l <= net.L; ++l) hmax = net.dims[l] > hmax ? net.dims[l] : hmax;
    const int ldx = hmax + 4;
    if (ldx_out) *ldx_out = ldx;
    size_t words = (size_t)2 * TM * ldx + (size_t)8 * (net.dims[net.L] + 4) + 8 + (size_t)TM * net.NHP + (size_t)TM * (OBS_WORDS + 4);
    return words * 4;
}

int rollout_pick_tile(const NetShape& net, int B)
{
    int lo = 16, hi = 256;
    for (int l = 1; l <= net.L; ++l) {
        const int N = net.dims[l];
        const int mn = 1024 / N > 1 ? 1024 / N : 1;      // RM >= 1
        const int mx = 16 * 1024 / N;                    // RM <= 16
        if (mn > lo) lo = mn;
        if (mx < hi) hi = mx;
    }
    // a tile also has to fit LDS: two activation buffers of the widest layer plus the transposed head matrix (a
    // 1024-wide last layer with 16 envs is 2 KB over; the caller then gets "no rollout tile fits" at create)
    auto fits = [&](int tm) { return tm >= lo && tm <= hi && B % tm == 0 && rollout_lds_bytes(net, EnvDims{}, tm, nullptr) <= 160 * 1024; };   // what one workgroup can be given on gfx950
    int best = 0;
    for (int tm = 16; tm <= 256; tm *= 2) {
        if (!fits(tm)) continue;
        if (!best) best = tm;                            // smallest valid tile
        if (B / tm >= 2048) best = tm;                   // largest tile that still leaves eight workgroups per CU
    }
    if (best && B / best < 256) {                        // small batches: fill the chip first
        for (int tm = 16; tm <= 256; tm *= 2)
            if (fits(tm) && B / tm >= 256) best = tm;
    }
    return best;
}

template <int ENV, bool BF, bool REPLAY>
static hipError_t launch_one(anakin* h, const RolloutArgs& args, int TM)
{
    size_t lds = rollout_lds_bytes(h->net, h->env, TM, nullptr);
    RolloutArgs a = args;
    if (ENV == ENV_MAZE) {
        // the wall sums of the tile stay in LDS where they fit beside the activations (all but the widest layers)
        const size_t pre = (size_t)TM * h->net.dims[1] * 4;
        a.maze_prefix = lds + pre <= 160 * 1024 ? 1 : 0;
        if (a.maze_prefix) lds += pre;
    }
    auto kern = rollout_kernel<ENV, BF, REPLAY>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, REPLAY ? "replay_forward" : "rollout");
    hipLaunchKernelGGL(kern, dim3(h->B / TM), dim3(WG), lds, h->stream, a, TM);
    return hipGetLastError();
}

void fill_rollout_args(anakin* h, RolloutArgs& a);

// environments per workgroup of the replay: with the steps spread over workgroups as well every size can fill the chip, so
// the one that ends first -- the longest share of steps per compute unit times the rows of a step, and about eight rows'
// time that a step costs at any size
static int replay_tile(const anakin* h, int tend)
{
    int best = 16;
    long best_cost = 0;
    for (int tm = 16; tm <= 64 && stream_lds_bytes(h->net, h->env, tm, false) <= 160 * 1024; tm *= 2) {
        const int tiles = (h->B + tm - 1) / tm, tseg = replay_segment(tiles, tend);
        const long wgs = (long)tiles * ((tend + tseg - 1) / tseg), cost = (wgs + 255) / 256 * tseg * (tm + 8);
        if (!best_cost || cost <= best_cost) { best = tm; best_cost = cost; }
    }
    return best;
}

template <int ENV, bool REPLAY, bool BF>
static hipError_t launch_stream(anakin* h, const RolloutArgs& args, int TM)
{
    StreamArgs a;
    a.r = args;
    a.w1_lds = stream_lds_bytes(h->net, h->env, TM, true) <= 160 * 1024 ? 1 : 0;
    const size_t lds = stream_lds_bytes(h->net, h->env, TM, a.w1_lds != 0);
    const int tiles = (h->B + TM - 1) / TM;
    a.tend = args.T + (args.bootstrap ? 1 : 0);
    a.tseg = replay_segment(tiles, a.tend);
    auto kern = TM == 16 ? rollout_stream_kernel<ENV, 1, REPLAY, BF> : TM == 32 ? rollout_stream_kernel<ENV, 2, REPLAY, BF> : rollout_stream_kernel<ENV, 4, REPLAY, BF>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, REPLAY ? "replay_forward" : "rollout");
    hipLaunchKernelGGL(kern, dim3(tiles, REPLAY ? (a.tend + a.tseg - 1) / a.tseg : 1), dim3(STW + STA), lds, h->stream, a);
    return hipGetLastError();
}

template <int ENV, int RW, int G, bool HOLD = false>
static hipError_t launch_resident(anakin* h, const RolloutArgs& a)
{
    const int w1 = h->env.kind != ENV_MAZE && resident_lds_bytes(h->net, h->env.kind, G, true) <= 160 * 1024;
    const size_t lds = resident_lds_bytes(h->net, h->env.kind, G, w1 != 0);
    auto kern = rollout_resident_kernel<ENV, RW, G, HOLD>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, "rollout");
    hipLaunchKernelGGL(kern, dim3((h->B + 16 * G - 1) / (16 * G)), dim3(64 * RES_WAVES), lds, h->stream, a, w1);
    return hipGetLastError();
}

template <int ENV>
static hipError_t launch_resident64(anakin* h, const RolloutArgs& a)
{
    constexpr int TM = 16, RW = 64;
    size_t lds = rollout_lds_bytes(h->net, h->env, TM, nullptr);
    lds += (size_t)2 * RW * 4;                                     // the hidden layers' biases
    lds += (size_t)(ENV == ENV_MAZE ? TM : h->net.dims[0]) * RW * 4;
    auto kern = rollout_resident64_kernel<ENV>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, "rollout");
    hipLaunchKernelGGL(kern, dim3(h->B / TM), dim3(WG), lds, h->stream, a);
    return hipGetLastError();
}

// Layers of 128 take 104 to 145 registers, so that two workgroups share a compute unit (boards; unrolls of 16 with one, two to a
// unit: Catch, 65536 environments 527 / 417 us, 16 x 16 maze, 12288 178 / 142; where there is one per unit anyway the same).
// Beside a learner it takes 160, whatever the code needs, while its workgroups have a unit each: with fewer a replay (240
// for its two wavefronts per SIMD) finds room beside it, and as both are bound by the matrix cores and the actor is the longer
// chain, the step takes longer.  Decoupled steps without / with: Catch 8192 environments, T = 20 302 / 262 us, T = 40 575 / 487,
// 2048, T = 40 196 / 165, 3072, T = 20 136 / 138.5; maze 4080, T = 20 249 / 238, 8192 354 / 372; the pendulum, which leaves no
// room in either form, within 3 %.  More workgroups than units: Catch 10240, T = 20 347 / 370, 16384 472 / 540.
template <int ENV>
static hipError_t launch_resident_env(anakin* h, const RolloutArgs& a, int width, int tm, bool beside)
{
    if (width == 256) return tm == 32 ? launch_resident<ENV, 256, 2>(h, a) : launch_resident<ENV, 256, 1>(h, a);
    if (width == 128) {
        if (beside && (h->B + tm - 1) / tm <= 256) return tm == 32 ? launch_resident<ENV, 128, 2, true>(h, a) : launch_resident<ENV, 128, 1, true>(h, a);
        return tm == 32 ? launch_resident<ENV, 128, 2>(h, a) : launch_resident<ENV, 128, 1>(h, a);
    }
    return launch_resident64<ENV>(h, a);
}

// Which kernel acts, of those that hold the weights on chip (nets of one layer have theirs, launch_forward).
// beside: the learner runs at the same time (the actor of a decoupled step)
enum class Actor { PINNED, WIDE, SMALL, RESIDENT, OTHER };
static Actor pick_actor(const anakin* h, bool beside)
{
    if (h->mode & (ANAKIN_MODE_CANONICAL_ACTING | ANAKIN_MODE_STREAM_WEIGHTS)) return Actor::OTHER;
    // Each of its workgroups has a compute unit to itself: beside a learner it takes half of them at most (decoupled steps,
    // 256-256, T = 16: 256 environments 130 -> 101 us, 512 129.5 -> 119.5, but 1024 130.5 -> 171.6 on all units; 256-512:
    // 247 -> 144, 246 -> 181, 246 -> 248).
    // Where the pinned kernel, four times as many environments to a unit, could have the net, a quarter (128-256, T = 16, wide and
    // pinned beside a learner: 256 environments on Catch 89 and 99 us, the pendulum 92 and 106, the 8 x 8 maze 94 and 104; 512 100
    // and 96, 103 and 104, 108 and 103).
    if (h->wide > 0 && (!beside || h->B / (4 * h->wide) <= (h->pinned.NB > 0 ? 64 : 128))) return Actor::WIDE;
    if (h->pinned.NB > 0) return Actor::PINNED;
    // Beside the learner of a small board net a few of its workgroups cost more than they save (decoupled Catch, T = 20: 512
    // environments 57.6 -> 59.2 us, 1024 66.4 -> 67.9, but 2048 83.6 -> 82.1, 4096 110.2 -> 104.3; pendulum 1024 71.0 -> 64.1,
    // 4096 102.8 -> 96.7).
    if (rollout_small_ok(h) && (!beside || h->env.kind == ENV_PENDULUM || h->B > 1024)) return Actor::SMALL;
    return h->TM_res > 0 ? Actor::RESIDENT : Actor::OTHER;
}

// Whether the V-trace launch of a decoupled step is kept off the units that the actor works on (launch_scan_loss): the 256-wide
// actor of Catch is the only one that leaves registers for its wavefronts (215 of 256 for each of two per SIMD; 233 and 243 on
// mazes and the pendulum) and is slowed by them, and while it has at most 160 workgroups there are units enough without it.
// Decoupled steps of 256-256, beside the actor / off its units: Catch 1536 environments, T = 8 116 / 105 us, T = 20 186 / 186,
// 2048, T = 8 122 / 124, T = 20 222 / 220, T = 40 382 / 362, T = 64 583 / 563, 2560, T = 8 152 / 148, T = 40 534 / 534, but 3584,
// T = 40 667 / 672, 4080 715 / 741; maze 2048, T = 20 293 / 298, 3072 388 / 402; pendulum 4080, T = 40 659 / 668.  Behind the actors
// of other nets as well it loses or nothing: 128-128 2048, T = 20 107 / 112, 256-128-64 195 / 200, bf16 256-256 3072 153 / 161.
// lds: what the V-trace workgroup has then; the actor's 43 KB and W1, where that fits, have to leave less.
bool vtrace_off_the_actor(const anakin* h, size_t lds)
{
    if (h->env.kind != ENV_CATCH || rollout_resident_width(h->net) != 256 || pick_actor(h, true) != Actor::RESIDENT || h->B > 16 * 160) return false;
    const size_t w1 = resident_lds_bytes(h->net, ENV_CATCH, 1, true), actor = w1 <= 160 * 1024 ? w1 : resident_lds_bytes(h->net, ENV_CATCH, 1, false);
    return actor + lds > 160 * 1024;
}

template <bool REPLAY>
static hipError_t launch_forward(anakin* h, const RolloutArgs& a, bool beside = false)
{
    const bool bf = h->net.bf16 != 0;
    if (const int lw = rollout_lane_width(h)) {
        if (a.keep_acts == 0) {
            if (h->env.kind == ENV_CATCH) return lw == 32 ? launch_lane<ENV_CATCH, 32, REPLAY>(h, a) : launch_lane<ENV_CATCH, 64, REPLAY>(h, a);
            return lw == 32 ? launch_lane<ENV_PENDULUM, 32, REPLAY>(h, a) : launch_lane<ENV_PENDULUM, 64, REPLAY>(h, a);
        }
    }
    if (rollout_one_ok(h)) return launch_rollout_one(h, a, REPLAY);
    if (!REPLAY) {
        const int w = rollout_resident_width(h->net);
        switch (pick_actor(h, beside)) {
            case Actor::PINNED: return launch_pinned(h, a);
            case Actor::WIDE:   return launch_wide(h, a);
            case Actor::SMALL:  return launch_small(h, a);
            case Actor::RESIDENT:
                switch (h->env.kind) {
                    case ENV_CATCH:    return launch_resident_env<ENV_CATCH>(h, a, w, h->TM_res, beside);
                    case ENV_PENDULUM: return launch_resident_env<ENV_PENDULUM>(h, a, w, h->TM_res, beside);
                    default:           return launch_resident_env<ENV_MAZE>(h, a, w, h->TM_res, beside);
                }
            case Actor::OTHER: break;
        }
    }
    if (h->TM_mfma > 0 && !(h->mode & ANAKIN_MODE_CANONICAL_ACTING)) {
        const int TM = REPLAY ? replay_tile(h, a.T + (a.bootstrap ? 1 : 0)) : h->TM_mfma;
        switch (h->env.kind) {
            case ENV_CATCH:    return bf ? launch_stream<ENV_CATCH, REPLAY, true>(h, a, TM) : launch_stream<ENV_CATCH, REPLAY, false>(h, a, TM);
            case ENV_PENDULUM: return bf ? launch_stream<ENV_PENDULUM, REPLAY, true>(h, a, TM) : launch_stream<ENV_PENDULUM, REPLAY, false>(h, a, TM);
            default:           return bf ? launch_stream<ENV_MAZE, REPLAY, true>(h, a, TM) : launch_stream<ENV_MAZE, REPLAY, false>(h, a, TM);
        }
    }
    switch (h->env.kind) {
        case ENV_CATCH:    return bf ? launch_one<ENV_CATCH, true, REPLAY>(h, a, h->TM) : launch_one<ENV_CATCH, false, REPLAY>(h, a, h->TM);
        case ENV_PENDULUM: return bf ? launch_one<ENV_PENDULUM, true, REPLAY>(h, a, h->TM) : launch_one<ENV_PENDULUM, false, REPLAY>(h, a, h->TM);
        default:           return bf ? launch_one<ENV_MAZE, true, REPLAY>(h, a, h->TM) : launch_one<ENV_MAZE, false, REPLAY>(h, a, h->TM);
    }
}

hipError_t launch_rollout(anakin* h)
{
    RolloutArgs a;
    fill_rollout_args(h, a);
    return launch_forward<false>(h, a);
}

// the actor of a decoupled step: parameters from the behaviour copy, no hidden activations kept
hipError_t launch_rollout_behaviour(anakin* h)
{
    RolloutArgs a;
    fill_rollout_args(h, a);
    a.theta = at<const float>(h, h->lay.theta_b);
    a.keep_acts = 0;
    return launch_forward<false>(h, a, true);
}

// the learner's forward pass over the stored unroll with the current parameters: hidden activations
// for the backward pass, head outputs and values into the learner's own buffers
hipError_t launch_replay_forward(anakin* h, bool bootstrap)
{
    RolloutArgs a;
    fill_rollout_args(h, a);
    a.bootstrap = bootstrap ? 1 : 0;
    a.tp.tr_head = at<float>(h, h->lay.head_new);
    a.tp.tr_val = at<float>(h, h->lay.val_new);
    const int samples = (h->T + a.bootstrap) * h->B;
    if (replay_resident_ok(h, samples)) return launch_replay_resident(h, a, samples);
    return launch_forward<true>(h, a);
}

}  // namespace ank
