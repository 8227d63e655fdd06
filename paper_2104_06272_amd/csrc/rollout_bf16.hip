// Acting for bf16 networks on the matrix cores (paper figure 2 top; section 2.1
// loop).  Same persistent structure as the fp32 kernels: a workgroup of eight
// wavefronts owns 64 environments for the whole unroll, env state in registers,
// activations in LDS (bf16), trajectory and hidden activations to HBM.  It takes the nets
// whose hidden matrices do not fit the registers (the others: rollout_bf16_pinned.hip) and all
// replays.
//
// Numerics (bf16 workload): weights and layer inputs are bfloat16, products are
// exact in fp32, accumulation is fp32 inside v_mfma_f32_32x32x16_bf16, bias and
// ReLU are applied in fp32 and the result is rounded to bfloat16 for the next
// layer; head outputs stay fp32.  The accumulation order inside the bf16 MFMA
// is the hardware's, so head outputs agree with a sequential fp32 chain only
// to rounding; sampling and env stepping downstream are exact functions of the
// head outputs the kernel stores.
//
// The first layer is a gather-sum over the 0/1 observation in fp32.  For the
// maze the wall plane and the goal never change, so their contribution (bias +
// wall rows + goal row) is computed once per launch, on the matrix cores, and
// then lives in registers for the whole unroll; each step adds the agent row.
// Hidden activations go to HBM sample-packed (see learn_bf16.hip): layers of
// different widths from registers, where the accumulator layout of the MFMA holds
// four consecutive samples of one column, half of a packed group; equal layers and
// the first one from LDS, by transposing reads.
//
// Weights of the hidden layers are read from L2 in operand tiles (one KiB per
// wavefront load, see internal.h), four 16-input steps ahead or more; two
// wavefronts per SIMD cover the rest of the latency.
//
// Operand layout of v_mfma_f32_32x32x16_bf16 (verified on gfx950): lane l feeds
// A[row l%32][k 8*(l/32) .. +7] and B[k 8*(l/32) .. +7][col l%32]; accumulator
// register r of lane l is D[row 8*(r/4) + 4*(l/32) + r%4][col l%32].
#include "acting_bf16.h"

namespace ank {

constexpr int BTM = 64;                 // envs per workgroup

// Hidden layer on the matrix cores: Y[64][N] = relu(X[64][K] W + b), X and Y bf16 in LDS.
// Wavefront w computes columns [32*NT*w, 32*NT*(w+1)); wavefronts past N stay idle.
// gP: sample-packed copy of Y in HBM (null: not kept), g8: first sample group of this tile.
template <int NT>
__device__ __forceinline__ void bf16_layer(const uint16_t* __restrict__ X, uint16_t* __restrict__ Y, int ldx,
                                           const uint16_t* __restrict__ Wt, const float* __restrict__ bias,
                                           int K, int N, int wave, int lane, uint16_t* __restrict__ gP, size_t g8,
                                           uint32_t* __restrict__ gM)
{
    const int l32 = lane & 31, kg = lane >> 5;
    const int n0 = wave * 32 * NT;
    if (n0 >= N) return;
    f16v acc[2][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float b = bias[n0 + 32 * t + l32];
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[0][t][r] = b; acc[1][t][r] = b; }
    }
    const uint16_t* xa = X + l32 * ldx + 8 * kg;
    const int KS = K >> 4;                                       // 16-input steps: 8, 16 or 32
    const uint16_t* wb = Wt + ((size_t)(n0 >> 5) * KS << 9) + lane * 8;
    constexpr int U = 4;                                         // steps per prefetch block
    bf8 w0[U][NT], w1[U][NT];
    auto load = [&](bf8 (&d)[U][NT], int s) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) d[u][t] = *reinterpret_cast<const bf8*>(wb + ((size_t)(t * KS + s + u) << 9));
    };
    auto compute = [&](const bf8 (&d)[U][NT], int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bf8 a0 = *reinterpret_cast<const bf8*>(xa + 16 * (s + u));
            const bf8 a1 = *reinterpret_cast<const bf8*>(xa + 32 * ldx + 16 * (s + u));
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[0][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, d[u][t], acc[0][t], 0, 0, 0);
                acc[1][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, d[u][t], acc[1][t], 0, 0, 0);
            }
        }
    };
    // the scheduling barriers keep every block of loads ahead of the MFMAs of the block before it
    load(w0, 0);
    for (int s = 0; s < KS; s += 2 * U) {
        load(w1, s + U);
        __builtin_amdgcn_sched_barrier(0);
        compute(w0, s);
        if (s + 2 * U < KS) load(w0, s + 2 * U);
        __builtin_amdgcn_sched_barrier(0);
        compute(w1, s + U);
    }
    // register group r/4 of lane (l32, kg) holds rows 8*(r/4) + 4*kg + 0..3 of column l32
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = n0 + 32 * t + l32;
            uint32_t mk = 0u;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int row = mt * 32 + 8 * g + 4 * kg;
                const uint32_t p01 = pack_bf16x2(relu(acc[mt][t][4 * g]), relu(acc[mt][t][4 * g + 1]));
                const uint32_t p23 = pack_bf16x2(relu(acc[mt][t][4 * g + 2]), relu(acc[mt][t][4 * g + 3]));
                Y[(row + 0) * ldx + col] = (uint16_t)p01; Y[(row + 1) * ldx + col] = (uint16_t)(p01 >> 16);
                Y[(row + 2) * ldx + col] = (uint16_t)p23; Y[(row + 3) * ldx + col] = (uint16_t)(p23 >> 16);
                if (gP) {
                    // written once, read by the update: streaming stores leave the weights in L2
                    u32v2 pv; pv[0] = p01; pv[1] = p23;
                    __builtin_nontemporal_store(pv, reinterpret_cast<u32v2*>(gP + ((g8 + mt * 4 + g) * N + col) * 8 + 4 * kg));
                    mk |= (nonzero_flags_pk(p01) << (2 * g)) | (nonzero_flags_pk(p23) << (2 * g + 1));
                }
            }
            if (gP) __builtin_nontemporal_store(mk, gM + relu_mask_index((g8 >> 2) + mt, kg, N, col));
        }
}

// One piece of an activation tile X[64][..] on its way to HBM, sample-packed: lanes 0..31 take columns n0 .. n0 + 31 of the
// samples 16 gp + 0..7 of half mt, lanes 32..63 of the next eight.  The transposing read gives a lane four rows of one column
// (a group of 16 lanes reads 4 rows x 16 columns, lane s row s / 4 and columns 4 (s % 4) ..).  The ReLU flags of the piece go
// into m0 (rows 0..3 of each eight) and m1 (rows 4..7), to be shifted by twice the lane's half.
__device__ __forceinline__ u32v4 read_piece(const uint16_t* __restrict__ X, int ldx, int n0, int mt, int gp, int lane)
{
    typedef short s4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s4v* lds_s4;
    const int kg = lane >> 5, s = lane & 15, gq = (lane >> 4) & 1;
    const uint16_t* x = X + (32 * mt + 16 * gp + 8 * kg + (s >> 2)) * ldx + n0 + 16 * gq + 4 * (s & 3);
    const u32v2 lo = __builtin_bit_cast(u32v2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(x)));
    const u32v2 hi = __builtin_bit_cast(u32v2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(x + 4 * ldx)));
    u32v4 v;
    v[0] = lo[0]; v[1] = lo[1]; v[2] = hi[0]; v[3] = hi[1];
    return v;
}
// Memory is addressed through buffer descriptors, one per tile and array: what is not to be written has a descriptor of no
// bytes.  A branch around the stores would hide from the compiler how many operations are behind a load of the weight stream,
// and its waits would be for newer loads than the one that is needed.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t store_rsrc(const void* p, bool on) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, on ? 0x7fffffffu : 0u, 0x00020000); }
constexpr int NT_STORE = 2;             // streaming: written once, read by the update; the weights stay in L2
// dst: the packed activations of the tile's first sample group; flags: the ReLU words of its first stage
__device__ __forceinline__ void store_piece(const u32v4 v, int n0, int mt, int gp, int lane, int N, rsrc_t dst, uint32_t& m0, uint32_t& m1)
{
    const int l32 = lane & 31, kg = lane >> 5;
    __builtin_amdgcn_raw_buffer_store_b128(v, dst, 16 * (kg * N + l32), 16 * ((4 * mt + 2 * gp) * N + n0), NT_STORE);
    m0 |= (nonzero_flags_pk(v[0]) << (4 * gp)) | (nonzero_flags_pk(v[1]) << (4 * gp + 1));
    m1 |= (nonzero_flags_pk(v[2]) << (4 * gp)) | (nonzero_flags_pk(v[3]) << (4 * gp + 1));
}
// the ReLU words of a half of the tile, from the flags of its two pieces: each half of the lanes has two of the four groups of
// eight samples of both words, and writes one word
__device__ __forceinline__ void store_flags(int n0, int mt, int lane, int N, rsrc_t flags, uint32_t m0, uint32_t m1)
{
    const int l32 = lane & 31, kg = lane >> 5;
    const u32v2 w = __builtin_bit_cast(u32v2, __builtin_amdgcn_permlane32_swap(m0 << (2 * kg), m1 << (2 * kg), false, false));
    __builtin_amdgcn_raw_buffer_store_b32(w[0] | w[1], flags, 4 * (kg * N + l32), 4 * (2 * mt * N + n0), NT_STORE);
}
// 32 NT columns of an activation tile to HBM at once
template <int NT>
__device__ __forceinline__ void store_tile(const uint16_t* X, int ldx, int n0, int lane, int N, rsrc_t dst, rsrc_t flags)
{
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            uint32_t m0 = 0u, m1 = 0u;
            const u32v4 v0 = read_piece(X, ldx, n0 + 32 * t, mt, 0, lane), v1 = read_piece(X, ldx, n0 + 32 * t, mt, 1, lane);
            store_piece(v0, n0 + 32 * t, mt, 0, lane, N, dst, m0, m1);
            store_piece(v1, n0 + 32 * t, mt, 1, lane, N, dst, m0, m1);
            store_flags(n0 + 32 * t, mt, lane, N, flags, m0, m1);
        }
}

// The same layer for nets whose hidden layers all have this width H.  What bounds it: the weights' way from L2 (512 columns:
// 512 KB a layer, 54 B per cycle and compute unit when all of them stream: 9.7 k cycles) and the matrix cores (8.2 k), so
// nothing may stand in the way of either:
// - The stream of a wavefront runs RING k steps ahead, through layers and time steps without a break: the next layer's
//   first weights are asked for during this one, the first layer's during the last of the step before.  (Eight steps ahead
//   were no quicker and took registers that the maze's prefix needs.)
// - Loads and stores of a wavefront complete in issue order, so a load behind a store waits for its acknowledgement.  Biases
//   are in LDS (read from memory they waited for the first layer's stores, 2 k cycles); the layer's inputs go to HBM from
//   LDS, a piece a step, beside the MFMAs.
// - The weights are the A operand (rows: outputs), the activations the B operand (columns: environments): a lane ends up
//   with four consecutive outputs of one environment, one 8-byte LDS store (as the other operand order: four 2-byte ones,
//   2.2 k cycles of a 512-wide layer's 3.5 k between its last MFMA and the barrier).
// 3 layers of 512 units, 16 x 16 maze, 16384 environments, 33 passes: 793 -> 669 us, 45.1 -> 37.9 k cycles a pass.  Of these
// the two streamed layers take 27.8 k (MFMAs 16.4 k; without the stores 25.5 k, without the weights' loads as well 20.6 k).
constexpr int RING = 4;
template <int NT, int H>
__device__ __forceinline__ void bf16_layer_stream(const uint16_t* __restrict__ X, uint16_t* __restrict__ Y, int ldx,
                                                  const uint16_t* __restrict__ Wt, const uint16_t* __restrict__ Wt_next,
                                                  const float* __restrict__ bias, int wave, int lane, rsrc_t dst, rsrc_t flags, bf8 (&w)[RING][NT])
{
    constexpr int KS = H / 16, PN = 4 * NT;                        // k steps; pieces of X to store, one a step
    static_assert(KS % RING == 0 && PN < KS, "whole turns of the ring; the pieces fit");
    const int l32 = lane & 31, kg = lane >> 5;
    const int n0 = wave * 32 * NT;
    if (n0 >= H) return;
    f16v acc[2][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 b = *reinterpret_cast<const float4*>(bias + n0 + 32 * t + 8 * g + 4 * kg);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) { acc[mt][t][4 * g] = b.x; acc[mt][t][4 * g + 1] = b.y; acc[mt][t][4 * g + 2] = b.z; acc[mt][t][4 * g + 3] = b.w; }
        }
    const uint16_t* xa = X + l32 * ldx + 8 * kg;
    const size_t wave_off = ((size_t)(n0 >> 5) * KS << 9) + lane * 8;
    bf8 av[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) av[0][mt] = *reinterpret_cast<const bf8*>(xa + 32 * mt * ldx);
    uint32_t m0 = 0u, m1 = 0u;
    u32v4 piece;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) av[(s + 1) & 1][mt] = *reinterpret_cast<const bf8*>(xa + 32 * mt * ldx + 16 * (s + 1));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[s % RING][t], av[s & 1][mt], acc[mt][t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            w[s % RING][t] = *reinterpret_cast<const bf8*>((s + RING < KS ? Wt : Wt_next) + wave_off + ((size_t)(t * KS + (s + RING) % KS) << 9));
        // pieces of X: tile of 32 columns, half of the samples, 16 of its 32; read a step before it is stored
        if (s >= 1 && s <= PN) {
            const int pc = s - 1;
            store_piece(piece, n0 + 32 * (pc / 4), (pc / 2) % 2, pc % 2, lane, H, dst, m0, m1);
            if (pc % 2 == 1) {
                store_flags(n0 + 32 * (pc / 4), (pc / 2) % 2, lane, H, flags, m0, m1);
                m0 = 0u; m1 = 0u;
            }
        }
        if (s < PN) piece = read_piece(X, ldx, n0 + 32 * (s / 4), (s / 2) % 2, s % 2, lane);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                u32v2 v;
                v[0] = pack_bf16x2(relu(acc[mt][t][4 * g]), relu(acc[mt][t][4 * g + 1]));
                v[1] = pack_bf16x2(relu(acc[mt][t][4 * g + 2]), relu(acc[mt][t][4 * g + 3]));
                *reinterpret_cast<u32v2*>(Y + (32 * mt + l32) * ldx + n0 + 32 * t + 8 * g + 4 * kg) = v;
            }
}

// the first weights of the stream
template <int NT, int H>
__device__ __forceinline__ void bf16_ring_fill(const uint16_t* __restrict__ Wt, int wave, int lane, bf8 (&w)[RING][NT])
{
    constexpr int KS = H / 16;
    const int n0 = wave * 32 * NT;
    if (n0 >= H) return;
    const uint16_t* wb = Wt + ((size_t)(n0 >> 5) * KS << 9) + lane * 8;
#pragma unroll
    for (int s = 0; s < RING; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) w[s][t] = *reinterpret_cast<const bf8*>(wb + ((size_t)(t * KS + s) << 9));
}

__device__ __forceinline__ void run_bf16_layer(const uint16_t* X, uint16_t* Y, int ldx, const uint16_t* Wt, const float* bias,
                                               int K, int N, int wave, int lane, uint16_t* gP, size_t g8, uint32_t* gM)
{
    if (N >= 512) bf16_layer<2>(X, Y, ldx, Wt, bias, K, N, wave, lane, gP, g8, gM);
    else bf16_layer<1>(X, Y, ldx, Wt, bias, K, N, wave, lane, gP, g8, gM);
}

// H1: width of the first hidden layer (128, 256 or 512).  Thread (pair of columns cp, env slice eq)
// owns columns 2*cp, 2*cp+1 of the first layer for EPT = H1/16 consecutive environments.
// REPLAY: the learner's pass over a stored unroll (decoupled acting and learning): states from the stored
// snapshots, head outputs and values to tp.tr_head / tp.tr_val (pointed at the learner's buffers), nothing
// sampled or stepped.
template <int ENV, int H1, bool UNI, bool REPLAY>
__global__ __launch_bounds__(BWG) void rollout_bf16_kernel(const RolloutBf16Args a)
{
    extern __shared__ uint4 smem4[];
    uint16_t* bufA = reinterpret_cast<uint16_t*>(smem4);
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH > 4 ? 8 : 4;   // actions, or mean and deviation, and the value
    const int ldx = a.ldx, L = a.net.L, HL = UNI ? H1 : a.net.dims[a.net.L];
    const int D = a.net.dims[0];
    const int ldh = HL + 8;
    uint16_t* bufB = bufA + BTM * ldx;
    uint16_t* whs = bufB + BTM * ldx;                            // [8][HL + 8] head weights, rows >= NH zero
    float* hp = reinterpret_cast<float*>(whs + 8 * ldh);         // [4][64][8] partial head sums per quarter of HL
    uint32_t* obs = reinterpret_cast<uint32_t*>(hp + 4 * BTM * 8);
    uint32_t* rng = obs + BTM * BOBS;
    float* bs = reinterpret_cast<float*>(rng + BTM * 2);         // UNI: [L - 1][H1] biases of the layers behind the first

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b0 = blockIdx.x * BTM;
    const int B = a.B, T = a.T;
    const TrajPtrs& tp = a.tp;
    const uint16_t* w1 = a.w + a.net.w_off[0];
    constexpr int EPT = H1 / 16;
    const int cp = tid % (H1 / 2), eq = tid / (H1 / 2);
    const int c = 2 * cp, e0 = eq * EPT;

    EnvState st{0u, 0.0f, 0.0f};
    const bool owner = tid < BTM;
    const int b = b0 + tid;
    float hb[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) hb[j] = j < NH ? a.theta[a.net.bh_off + j] : 0.0f;
    if (owner) {
        if (!REPLAY) {
            st.s0 = tp.s0[b];
            if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b]; st.f1 = tp.f1[b]; }
        }
        if (ENV == ENV_MAZE) for (int w = 0; w < 8; ++w) obs[tid * BOBS + w] = tp.walls[(size_t)w * B + b];
    }
    for (int i = tid; i < 8 * ldh; i += BWG) {
        const int k = i / ldh, j = i - k * ldh;
        whs[i] = (k < NH && j < HL) ? a.wt[a.net.wh_off + (size_t)k * HL + j] : (uint16_t)0;
    }
    if (UNI) for (int i = tid; i < (L - 1) * H1; i += BWG) bs[i] = a.theta[a.net.b_off[1 + i / H1] + i % H1];
    __syncthreads();
    // first-layer constants of this thread: the bias, plus -- for the maze -- the contribution of the wall
    // plane and of the goal cell, which never change: prefix[64][H1] = b1 + Walls[64][cells] W1[cells][H1]
    // on the matrix cores, handed over in the LDS of the two activation buffers, which are not in use yet (64 rows of
    // ldx floats are exactly both): workgroups that replay other time steps of the same environments have their own
    float pre[ENV == ENV_MAZE ? EPT : 1][2];
    const float bias0 = a.theta[a.net.b_off[0] + c], bias1 = a.theta[a.net.b_off[0] + c + 1];
    if (ENV == ENV_MAZE) {
        float* prefix = reinterpret_cast<float*>(smem4);         // [64][ldx]
        const int n = a.env.rows * a.env.cols;
        const int l32 = lane & 31, kg = lane >> 5;
        constexpr int NT1 = H1 >= 512 ? 2 : 1;
        const int n0 = wave * 32 * NT1;
        if (n0 < H1) {
            f16v acc[2][NT1];
#pragma unroll
            for (int t4 = 0; t4 < NT1; ++t4) {
                const float bb = a.theta[a.net.b_off[0] + n0 + 32 * t4 + l32];
#pragma unroll
                for (int r = 0; r < 16; ++r) { acc[0][t4][r] = bb; acc[1][t4][r] = bb; }
            }
            const int KS = D >> 4;
            const uint16_t* wb = a.wt + a.net.w_off[0] + ((size_t)(n0 >> 5) * KS << 9) + lane * 8;   // operand tiles of W1
            for (int k0 = 0; k0 < n; k0 += 16) {
                bf8 av[2];
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const int cell = k0 + 8 * kg;
                    const uint32_t bits = (obs[(mt * 32 + l32) * BOBS + (cell >> 5)] >> (cell & 31)) & 0xffu;
#pragma unroll
                    for (int q = 0; q < 8; ++q) av[mt][q] = ((bits >> q) & 1u) ? (__bf16)1.0f : (__bf16)0.0f;
                }
#pragma unroll
                for (int t4 = 0; t4 < NT1; ++t4) {
                    const bf8 bv = *reinterpret_cast<const bf8*>(wb + ((size_t)(t4 * KS + (k0 >> 4)) << 9));
                    acc[0][t4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[0], bv, acc[0][t4], 0, 0, 0);
                    acc[1][t4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[1], bv, acc[1][t4], 0, 0, 0);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t4 = 0; t4 < NT1; ++t4)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = mt * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
                        prefix[row * ldx + n0 + 32 * t4 + l32] = acc[mt][t4][r];
                    }
        }
        __syncthreads();
        const uint32_t goal = *reinterpret_cast<const uint32_t*>(w1 + (size_t)(3 * n - 1) * H1 + c);
        const float g0 = bf2f((uint16_t)(goal & 0xffffu)), g1 = bf2f((uint16_t)(goal >> 16));
#pragma unroll
        for (int m = 0; m < EPT; ++m) {
            const float2 p = *reinterpret_cast<const float2*>(prefix + (e0 + m) * ldx + c);
            pre[ENV == ENV_MAZE ? m : 0][0] = p.x + g0;
            pre[ENV == ENV_MAZE ? m : 0][1] = p.y + g1;
        }
    }
    float wp[3][2] = {{0, 0}, {0, 0}, {0, 0}};                   // pendulum: the three rows of W1
    if (ENV == ENV_PENDULUM) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t ww = *reinterpret_cast<const uint32_t*>(w1 + (size_t)k * H1 + c);
            wp[k][0] = bf2f((uint16_t)(ww & 0xffffu)); wp[k][1] = bf2f((uint16_t)(ww >> 16));
        }
    }

    constexpr int NTU = H1 >= 512 ? 2 : 1;
    bf8 ring[RING][NTU];                                         // UNI: the weight stream's next k steps
    if (UNI && L > 1) bf16_ring_fill<NTU, H1>(a.wt + a.net.w_off[1], __builtin_amdgcn_readfirstlane(wave), lane, ring);
    const int tid_outer = tid;
    const int t_begin = REPLAY ? (int)blockIdx.y * a.tseg : 0;
    const int t_end = REPLAY ? (t_begin + a.tseg < a.tend ? t_begin + a.tseg : a.tend) : T + 1;
    for (int t = t_begin; t < t_end; ++t) {
        // everything derived from the thread index is recomputed every step from a value the compiler
        // cannot see through: dozens of loop-invariant addresses would otherwise be kept in registers
        // across the whole time loop, on top of the 2 * EPT prefix values, and spilled
        int tid_step = tid_outer;
        asm volatile("" : "+v"(tid_step));
        const int tid = tid_step, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int cp = tid % (H1 / 2), eq = tid / (H1 / 2);
        const int c = 2 * cp, e0 = eq * EPT;
        const bool owner = tid < BTM;
        const int b = b0 + tid;
        const size_t tb = (size_t)t * B + b;
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
                obs[tid * BOBS + 0] = (uint32_t)bc; obs[tid * BOBS + 1] = (uint32_t)pc;
            } else if (ENV == ENV_PENDULUM) {
                float sn, cs;
                det_sincos(st.f0, sn, cs);
                obs[tid * BOBS + 0] = bits_from_f(bf16_to_f(bf16_bits(cs)));
                obs[tid * BOBS + 1] = bits_from_f(bf16_to_f(bf16_bits(sn)));
                obs[tid * BOBS + 2] = bits_from_f(bf16_to_f(bf16_bits(st.f1)));
            } else {
                obs[tid * BOBS + 8] = st.s0 & 0xffffu;
            }
        }
        __syncthreads();
        const bool keep = t < T && a.keep_acts;
        const size_t g8 = ((size_t)t * B + b0) >> 3;             // first sample group of this tile
        // where layer l (from 0, all of them H1 wide, or the first) is kept; the flags of a narrower first layer are not
        auto tile_rsrc = [&](int l) { return store_rsrc(reinterpret_cast<const uint16_t*>(tp.act[l]) + g8 * H1 * 8, keep); };
        auto flag_rsrc = [&](int l) { return store_rsrc(tp.mask[l] + relu_mask_index(g8 >> 2, 0, H1, 0), keep && (l > 0 || H1 >= 512)); };
        // the last wavefront draws this step's random numbers while it waits for its weight rows
        if (!REPLAY && wave == 7 && t < T) {
            const u32x4 w = philox(a.seed, (uint32_t)(b0 + lane), a.gstep + (uint64_t)t, DOM_ACTION);
            rng[lane * 2] = ENV == ENV_PENDULUM ? bits_from_f(gaussian_noise(w.x, w.y)) : w.x;   // the noise is ready when the heads are
            rng[lane * 2 + 1] = w.y;
        }
        // ---- first layer: fp32 gather-sum / three fmas, rounded to bf16 ----------
        {
            const int n = a.env.rows * a.env.cols;
            uint32_t r0[ENV == ENV_PENDULUM ? 1 : EPT], r1[ENV == ENV_CATCH ? EPT : 1];
            if (ENV != ENV_PENDULUM) {
                // all weight-row loads of this thread in flight before the first is used
#pragma unroll
                for (int m = 0; m < EPT; ++m) {
                    const int row0 = ENV == ENV_CATCH ? (int)obs[(e0 + m) * BOBS + 0] : n + (int)obs[(e0 + m) * BOBS + 8];
                    r0[ENV == ENV_PENDULUM ? 0 : m] = *reinterpret_cast<const uint32_t*>(w1 + (size_t)row0 * H1 + c);
                    if (ENV == ENV_CATCH)
                        r1[ENV == ENV_CATCH ? m : 0] = *reinterpret_cast<const uint32_t*>(w1 + (size_t)obs[(e0 + m) * BOBS + 1] * H1 + c);
                }
            }
#pragma unroll
            for (int m0 = 0; m0 < EPT; m0 += 8) {
                float v[8][2];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int m = m0 + q;
                    float vx = ENV == ENV_MAZE ? pre[ENV == ENV_MAZE ? m : 0][0] : bias0;
                    float vy = ENV == ENV_MAZE ? pre[ENV == ENV_MAZE ? m : 0][1] : bias1;
                    if (ENV == ENV_PENDULUM) {
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            const float x = f_from_bits(obs[(e0 + m) * BOBS + k]);
                            vx = fmaf(x, wp[k][0], vx); vy = fmaf(x, wp[k][1], vy);
                        }
                    } else {
                        const uint32_t g = r0[ENV == ENV_PENDULUM ? 0 : m];
                        vx += bf2f((uint16_t)(g & 0xffffu)); vy += bf2f((uint16_t)(g >> 16));
                        if (ENV == ENV_CATCH) {
                            const uint32_t g1 = r1[ENV == ENV_CATCH ? m : 0];
                            vx += bf2f((uint16_t)(g1 & 0xffffu)); vy += bf2f((uint16_t)(g1 >> 16));
                        }
                    }
                    v[q][0] = relu(vx); v[q][1] = relu(vy);
                }
                uint32_t px[4], py[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    px[q] = pack_bf16x2(v[2 * q][0], v[2 * q + 1][0]);
                    py[q] = pack_bf16x2(v[2 * q][1], v[2 * q + 1][1]);
                    // rows m0+2q and m0+2q+1 of the LDS tile, both columns as one 4-byte store
                    *reinterpret_cast<uint32_t*>(bufA + (e0 + m0 + 2 * q) * ldx + c) = (px[q] & 0xffffu) | (py[q] << 16);
                    *reinterpret_cast<uint32_t*>(bufA + (e0 + m0 + 2 * q + 1) * ldx + c) = (px[q] >> 16) | (py[q] & 0xffff0000u);
                }
            }
        }
        __syncthreads();
        uint16_t* cur = bufA;
        uint16_t* nxt = bufB;
        if (UNI) {
#pragma unroll 1
            for (int l = 1; l < L; ++l) {
                bf16_layer_stream<NTU, H1>(cur, nxt, ldx, a.wt + a.net.w_off[l], a.wt + a.net.w_off[l + 1 < L ? l + 1 : 1], bs + (l - 1) * H1,
                                           wave, lane, tile_rsrc(l - 1), flag_rsrc(l - 1), ring);
                __syncthreads();
                uint16_t* tmp = cur; cur = nxt; nxt = tmp;
            }
        } else {
            if (keep && wave < H1 / 64) store_tile<2>(bufA, ldx, 64 * wave, lane, H1, tile_rsrc(0), flag_rsrc(0));
            for (int l = 1; l < L; ++l) {
                const int K = a.net.dims[l], N = a.net.dims[l + 1];
                run_bf16_layer(cur, nxt, ldx, a.wt + a.net.w_off[l], a.theta + a.net.b_off[l], K, N, wave, lane,
                               keep ? reinterpret_cast<uint16_t*>(tp.act[l]) : nullptr, g8, tp.mask[l]);
                __syncthreads();
                uint16_t* tmp = cur; cur = nxt; nxt = tmp;
            }
        }
        // ---- heads: wavefront (tile, quarter) sums one quarter of the last layer for 32 envs ----
        {
            const int l32 = lane & 31, kg = lane >> 5;
            const int tile = wave & 1, kq = wave >> 1, kq_len = HL >> 2;
            f16v acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
            const uint16_t* xa = cur + (tile * 32 + l32) * ldx + kq * kq_len + 8 * kg;
            const uint16_t* wbs = whs + (l32 & 7) * ldh + kq * kq_len + 8 * kg;
            const bool real = l32 < 8;
            // one base address, recomputed every step, and constant offsets from it: sixteen loop-invariant
            // addresses would otherwise be kept (and spilled) across the time loop
            int hp_base = (kq * BTM + tile * 32 + 4 * kg) * 8 + l32;
            asm volatile("" : "+v"(hp_base));
            for (int k0 = 0; k0 < kq_len; k0 += 16) {
                const bf8 av = *reinterpret_cast<const bf8*>(xa + k0);
                bf8 bvv = *reinterpret_cast<const bf8*>(wbs + k0);
                if (!real) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) bvv[q] = (__bf16)0.0f;
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bvv, acc, 0, 0, 0);
            }
            if (real) {
#pragma unroll
                for (int r = 0; r < 16; ++r) hp[hp_base + (8 * (r >> 2) + (r & 3)) * 8] = acc[r];
            }
        }
        __syncthreads();
        if (UNI && keep) {
            // the last layer to HBM, by the wavefronts that do not sample; the last one takes the first's share
            const rsrc_t dst = tile_rsrc(L - 1), flags = flag_rsrc(L - 1);
            if (wave > 0 && wave * 32 * NTU < H1) store_tile<NTU>(cur, ldx, wave * 32 * NTU, lane, H1, dst, flags);
            if (wave == 7) store_tile<NTU>(cur, ldx, 0, lane, H1, dst, flags);
        }
        if (owner) {
            float hv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            float4 hq[4][2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                hq[q][0] = *reinterpret_cast<const float4*>(hp + (q * BTM + tid) * 8);
                hq[q][1] = NH > 4 ? *reinterpret_cast<const float4*>(hp + (q * BTM + tid) * 8 + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < NH) {
                    float s = hb[j];
#pragma unroll
                    for (int q = 0; q < 4; ++q) s += j % 4 == 0 ? hq[q][j / 4].x : j % 4 == 1 ? hq[q][j / 4].y : j % 4 == 2 ? hq[q][j / 4].z : hq[q][j / 4].w;
                    hv[j] = s;
                }
            float* hd = tp.tr_head + tb * NHP;
            *reinterpret_cast<float4*>(hd) = make_float4(hv[0], hv[1], hv[2], hv[3]);
            if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = make_float4(hv[4], hv[5], hv[6], hv[7]);
            const float val = last_head(hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], NH);
            tp.tr_val[tb] = val;
            if (!REPLAY && t < T) {
                const uint2 dr = *reinterpret_cast<const uint2*>(rng + tid * 2);
                float r; int done;
                if (ENV == ENV_PENDULUM) {
                    const float eps = f_from_bits(dr.x);
                    const float act = gaussian_action(hv[0], hv[1], eps);
                    tp.tr_eps[tb] = eps; tp.tr_actf[tb] = act;
                    pendulum_step(a.env, st, act, 0u, 0u, r, done);
                    if (done) {
                        const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                        pendulum_reset(st, wr.x, wr.y);
                    }
                } else {
                    const int act = sample_categorical_any(hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], ENV == ENV_CATCH ? 3 : 4, u01(dr.x));
                    tp.tr_act[tb] = (uint8_t)act;
                    if (ENV == ENV_CATCH) {
                        catch_step(a.env, st, act, 0u, r, done);
                        if (done) {
                            const u32x4 wr = philox(a.seed, (uint32_t)b, a.gstep + (uint64_t)t, DOM_RESET);
                            st.s0 = catch_reset(a.env, wr.x);
                        }
                    } else {
                        const uint32_t* wl = obs + tid * BOBS;
                        maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, r, done);
                    }
                }
                tp.tr_rew[tb] = r;
                tp.tr_done[tb] = (uint8_t)done;
            }
        }
    }
    if (!REPLAY && owner) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// can this net act on the bf16 matrix-core path?
bool rollout_bf16_ok(const NetShape& net, const EnvDims& env, int B)
{
    if (!net.bf16 || B % BTM) return false;
    if (env.kind == ENV_MAZE && (env.rows * env.cols) % 16) return false;   // wall plane in whole 16-cell steps
    for (int l = 1; l <= net.L; ++l) {
        const int n = net.dims[l];
        if (n != 128 && n != 256 && n != 512) return false;     // 1, 2 or 4 tiles of 32 columns per wavefront, 64-input prefetch blocks
    }
    return true;
}

void fill_rollout_args(anakin* h, RolloutArgs& a);

// what: 0 the acting unroll, 1 the actor of a decoupled step (behaviour copies of the parameters, no activations
// kept), 2 the learner's replay of the stored unroll with the current parameters
void fill_bf16_args(anakin* h, int what, RolloutBf16Args& a)
{
    RolloutArgs base;
    fill_rollout_args(h, base);
    const Layout& L = h->lay;
    a.env = base.env; a.net = base.net; a.tp = base.tp; a.theta = base.theta;
    a.w = at<const uint16_t>(h, L.w_bf16); a.wt = at<const uint16_t>(h, L.wt_bf16);
    a.keep_acts = 1;
    if (what == 1) {
        a.theta = at<const float>(h, L.theta_b); a.w = at<const uint16_t>(h, L.w_bf16_b); a.wt = at<const uint16_t>(h, L.wt_bf16_b);
        a.keep_acts = 0;
    } else if (what == 2) {
        a.tp.tr_head = at<float>(h, L.head_new); a.tp.tr_val = at<float>(h, L.val_new);
    }
    a.B = h->B; a.T = h->T; a.seed = h->seed; a.gstep = h->gstep;
    a.tend = a.tseg = h->T + 1;
    int hmax = 0;
    for (int l = 1; l <= h->net.L; ++l) hmax = h->net.dims[l] > hmax ? h->net.dims[l] : hmax;
    a.ldx = hmax + 8;
}

template <bool REPLAY>
static hipError_t launch_bf16_forward(anakin* h, int what, bool bootstrap = true)
{
    RolloutBf16Args a;
    fill_bf16_args(h, what, a);
    a.tend = h->T + (bootstrap ? 1 : 0);
    a.tseg = REPLAY ? replay_segment(h->B / BTM, a.tend) : a.tend;
    const int HL = h->net.dims[h->net.L], H1 = h->net.dims[1];
    const size_t lds = (size_t)2 * BTM * a.ldx * 2 + (size_t)8 * (HL + 8) * 2 + (size_t)4 * BTM * 8 * 4 + (size_t)BTM * (BOBS + 2) * 4 + (size_t)(h->net.L - 1) * H1 * 4;
    auto launch = [&](auto kern) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        ProfScope prof(h, REPLAY ? "replay_forward" : "rollout");
        hipLaunchKernelGGL(kern, dim3(h->B / BTM, REPLAY ? (a.tend + a.tseg - 1) / a.tseg : 1), dim3(BWG), lds, h->stream, a);
        return hipGetLastError();
    };
    bool uni = true;                                             // every hidden layer H1 wide: the weight stream runs across layers
    for (int l = 2; l <= h->net.L; ++l) uni = uni && h->net.dims[l] == H1;
#define ANK_BF16_W(ENVK, W) (uni ? launch(rollout_bf16_kernel<ENVK, W, true, REPLAY>) : launch(rollout_bf16_kernel<ENVK, W, false, REPLAY>))
#define ANK_BF16_CASE(ENVK) (H1 == 128 ? ANK_BF16_W(ENVK, 128) : H1 == 256 ? ANK_BF16_W(ENVK, 256) : ANK_BF16_W(ENVK, 512))
    switch (h->env.kind) {
        case ENV_CATCH:    return ANK_BF16_CASE(ENV_CATCH);
        case ENV_PENDULUM: return ANK_BF16_CASE(ENV_PENDULUM);
        default:           return ANK_BF16_CASE(ENV_MAZE);
    }
#undef ANK_BF16_CASE
#undef ANK_BF16_W
}

hipError_t launch_rollout_bf16(anakin* h) { return pinned_bf16_ok(h) ? launch_pinned_bf16(h, 0) : launch_bf16_forward<false>(h, 0); }
hipError_t launch_rollout_bf16_behaviour(anakin* h) { return pinned_bf16_ok(h) ? launch_pinned_bf16(h, 1) : launch_bf16_forward<false>(h, 1); }
hipError_t launch_replay_bf16(anakin* h, bool bootstrap) { return launch_bf16_forward<true>(h, 2, bootstrap); }

}  // namespace ank
