// Acting for bf16 nets with the hidden matrices in registers, 32 or 64 environments per workgroup.
//
// A step of the unroll is a chain of short phases; what bounds it at anything but the largest nets is their latency, and
// with weights streamed from L2 (rollout_bf16.hip) every layer also waits for them, behind the activation stores of the
// layer before (loads and stores of a wavefront complete in issue order): 4.2 us a step for a 128-128 net, whose matrix
// work is 0.2.  Here nothing is loaded inside the loop: each of eight wavefronts keeps up to four blocks of 128 inputs x
// 32 outputs (32 registers each; the host cuts the net into them, and a block's layer, inputs and outputs are scalars), the
// first layer's rows are in LDS where they fit.  Stores to memory of a layer's outputs, the records and the random draws
// are made by whichever wavefronts wait for another phase: outputs behind the next barrier, records beside the heads,
// draws beside the environment steps.  The row stride of the activations is a constant, so that the transposing two-byte
// stores of an accumulator tile have immediate offsets (with a variable one a tile's epilogue took 1080 cycles, now 450).
// The arithmetic and its order are those of the streaming kernel: the same bits.
//
// An unroll, streaming -> here: pendulum 128-128, 1024 environments, T = 32 137 -> 67 us; 256-256, 8192, T = 20 132 -> 68;
// 256-256-256, 4096 177 -> 89; Catch 512-128, 8192 187 -> 97; maze 512-256, 4096 192 -> 143; with 64 environments per
// workgroup: 128-128, 65536, T = 16 283 -> 188, 256-256-256, 16384, T = 20 194 -> 171.
#include <type_traits>
#include "acting_bf16.h"

namespace ank {

struct PinnedBf16Plan {
    static constexpr int WAVES = 8, MAX_BLOCKS = 4;
    enum : uint32_t { VALID = 1u, START = 2u, END = 4u };          // first / last block of its 32 outputs
    static constexpr int LAYER = 3, LGN = 5, TILE = 9, KBLOCK = 14;   // bits: layer (2), log2 of its outputs (4), output / 32 (5), input / 128 (2)
    int NB;                                                        // blocks per wavefront (0: does not fit)
    uint32_t block[WAVES][MAX_BLOCKS];
};
struct PinnedBf16Args {
    RolloutBf16Args r;
    PinnedBf16Plan p;
    int w1_lds;                                                    // first-layer rows (maze: the agent plane) in LDS
};
typedef const __attribute__((address_space(4))) PinnedBf16Args* kernarg_bf16;

// stores the packed outputs pk of a finished layer (the block word pend; 0: nothing to store) and their ReLU masks
template <int MT>
__device__ __forceinline__ void pinned_bf16_flush(uint32_t& pend, const uint32_t (&pk)[MT][8], float* a1, float* a2, float* a3, uint32_t* m1, uint32_t* m2, uint32_t* m3, size_t g8, int lane)
{
    if (!pend) return;
    const int l = (pend >> PinnedBf16Plan::LAYER) & 3, N = 1 << ((pend >> PinnedBf16Plan::LGN) & 15), kg = lane >> 5, col = 32 * ((pend >> PinnedBf16Plan::TILE) & 31) + (lane & 31);
    float* act = a3;
    uint32_t* mask = m3;
    if (l == 2) { act = a2; mask = m2; }
    if (l == 1) { act = a1; mask = m1; }
    uint16_t* o = reinterpret_cast<uint16_t*>(act) + (g8 * N + col) * 8 + 4 * kg;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        uint32_t mk = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u32v2 pv; pv[0] = pk[mt][2 * g]; pv[1] = pk[mt][2 * g + 1];
            __builtin_nontemporal_store(pv, reinterpret_cast<u32v2*>(o + (size_t)(mt * 4 + g) * N * 8));
            mk |= (nonzero_flags_pk(pv[0]) << (2 * g)) | (nonzero_flags_pk(pv[1]) << (2 * g + 1));
        }
        __builtin_nontemporal_store(mk, mask + relu_mask_index((g8 >> 2) + mt, kg, N, col));
    }
    pend = 0u;
}

template <int ENV, int H1, int LDX, int MT, int NB>
__global__ __launch_bounds__(BWG, 2) void rollout_bf16_pinned_kernel(const PinnedBf16Args q)
{
    constexpr int TM = 32 * MT;
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH <= 4 ? 4 : 8;
    constexpr int EPT = H1 == 512 ? 32 : TM * H1 / 1024;           // environments per thread in the first layer
    constexpr int GE = EPT < 8 ? EPT : 8;                          // of them, as many as share a packed group
    constexpr int FTHR = TM / EPT * (H1 / 2);                      // threads it takes
    const RolloutBf16Args& a = q.r;
    extern __shared__ uint4 smem4[];
    uint16_t* bufs = reinterpret_cast<uint16_t*>(smem4);           // [2][TM][LDX]: layer l's outputs in buffer l % 2
    const int L = a.net.L, HL = a.net.dims[a.net.L], D = a.net.dims[0], ldh = HL + 8;
    uint16_t* whs = bufs + 2 * TM * LDX;                           // [8][HL + 8] head weights, rows >= NH zero
    float* hp = reinterpret_cast<float*>(whs + 8 * ldh);           // [4][TM][8] partial head sums per quarter of HL
    uint32_t* obs = reinterpret_cast<uint32_t*>(hp + 4 * TM * 8);  // [TM][BOBS]
    uint32_t* rng = obs + TM * BOBS;                               // [2][TM][4] draws: the action's two words (pendulum: noise), the reset's
    uint16_t* w1s = reinterpret_cast<uint16_t*>(rng + 2 * TM * 4); // first-layer rows
    const int tid0 = threadIdx.x, lane0 = tid0 & 63, wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
    const int b0 = blockIdx.x * TM, B = a.B, T = a.T, n_cells = a.env.rows * a.env.cols;
    const TrajPtrs& tp = a.tp;
    const uint16_t* w1 = a.w + a.net.w_off[0];

    // ---- this wavefront's blocks of the hidden matrices, in matrix-core operand order ----
    bf8 w[NB][8];
    float bv[NB];
    uint32_t blk[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const uint32_t d = q.p.block[wave][i];
        blk[i] = d;
        const int l = (d >> PinnedBf16Plan::LAYER) & 3, ct = (d >> PinnedBf16Plan::TILE) & 31, kb = (d >> PinnedBf16Plan::KBLOCK) & 3;
        if (d & PinnedBf16Plan::VALID) {
            const uint16_t* src = a.wt + a.net.w_off[l] + ((size_t)(ct * (a.net.dims[l] >> 4) + 8 * kb) << 9) + lane0 * 8;
#pragma unroll
            for (int u = 0; u < 8; ++u) w[i][u] = *reinterpret_cast<const bf8*>(src + (u << 9));
            bv[i] = a.theta[a.net.b_off[l] + 32 * ct + (lane0 & 31)];
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) w[i][u] = bf8{};
            bv[i] = 0.0f;
        }
    }
    // the last wavefront owns the environments, one per lane
    const bool owner = wave == 7 && (MT == 2 || lane0 < TM);
    EnvState st{0u, 0.0f, 0.0f};
    if (owner) {
        st.s0 = tp.s0[b0 + lane0];
        if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b0 + lane0]; st.f1 = tp.f1[b0 + lane0]; }
        if (ENV == ENV_MAZE) for (int v = 0; v < 8; ++v) obs[lane0 * BOBS + v] = tp.walls[(size_t)v * B + b0 + lane0];
    }
    for (int i = tid0; i < 8 * ldh; i += BWG) {
        const int k = i / ldh, j = i - k * ldh;
        whs[i] = (k < NH && j < HL) ? a.wt[a.net.wh_off + (size_t)k * HL + j] : (uint16_t)0;
    }
    if (q.w1_lds) {
        const uint4* src = reinterpret_cast<const uint4*>(w1 + (ENV == ENV_MAZE ? (size_t)n_cells * H1 : 0));
        uint4* dst = reinterpret_cast<uint4*>(w1s);
        const int n8 = (ENV == ENV_MAZE ? n_cells : D) * H1 / 8;
#pragma unroll 1
        for (int i = tid0; i < n8; i += BWG) dst[i] = src[i];
    }
    float hb[NH];
#pragma unroll
    for (int j = 0; j < NH; ++j) hb[j] = a.theta[a.net.bh_off + j];
    auto draw = [&](int t, int lane) __attribute__((always_inline)) {   // (one wavefront)
#pragma unroll
        for (int e = 0; e < (ENV == ENV_MAZE ? 1 : 2) * TM; e += 64) {  // (the maze's reset draws nothing)
            const int m = (e + lane) & (TM - 1);
            const bool reset = e + lane >= TM;
            if (ENV == ENV_MAZE && reset) break;
            const u32x4 v = philox(a.seed, (uint32_t)(b0 + m), a.gstep + (uint64_t)t, reset ? DOM_RESET : DOM_ACTION);
            const uint32_t v0 = (ENV == ENV_PENDULUM && !reset) ? bits_from_f(gaussian_noise(v.x, v.y)) : v.x;
            u32v2 o; o[0] = v0; o[1] = v.y;
            *reinterpret_cast<u32v2*>(rng + ((t & 1) * TM + m) * 4 + (reset ? 2 : 0)) = o;
        }
    };
    float sine = 0.0f;
    auto observe = [&](int lane) __attribute__((always_inline)) {
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            obs[lane * BOBS + 0] = (uint32_t)bc; obs[lane * BOBS + 1] = (uint32_t)pc;
        } else if (ENV == ENV_PENDULUM) {
            float cs;
            det_sincos(st.f0, sine, cs);
            obs[lane * BOBS + 0] = bits_from_f(bf16_to_f(bf16_bits(cs)));
            obs[lane * BOBS + 1] = bits_from_f(bf16_to_f(bf16_bits(sine)));
            obs[lane * BOBS + 2] = bits_from_f(bf16_to_f(bf16_bits(st.f1)));
        } else obs[lane * BOBS + 8] = st.s0 & 0xffffu;
    };
    if (owner) observe(lane0);
    if (wave == 6) draw(0, lane0);
    __syncthreads();
    // ---- first-layer constants of this thread (columns c, c + 1 of environments e0 ..), as in rollout_bf16_kernel ----
    const int c0 = 2 * (tid0 % (H1 / 2)), e00 = tid0 / (H1 / 2) * EPT;
    const bool first_thread = FTHR == BWG || tid0 < FTHR;
    float pre[ENV == ENV_MAZE ? EPT : 1][2];
    const float bias0 = a.theta[a.net.b_off[0] + c0], bias1 = a.theta[a.net.b_off[0] + c0 + 1];
    if (ENV == ENV_MAZE) {
        // 32 rows of the wall sums at a time, through the two activation buffers
        float* prefix = reinterpret_cast<float*>(smem4);           // [32][H1 + 4]
        const int l32 = lane0 & 31, kg = lane0 >> 5;
        constexpr int NT1 = H1 >= 512 ? 2 : 1;
        const int n0 = wave * 32 * NT1;
        const int KS = D >> 4;
        const uint16_t* wb = a.wt + a.net.w_off[0] + ((size_t)(n0 >> 5) * KS << 9) + lane0 * 8;   // operand tiles of W1
        const uint32_t goal = *reinterpret_cast<const uint32_t*>(w1 + (size_t)(3 * n_cells - 1) * H1 + c0);
        const float g0 = bf2f((uint16_t)(goal & 0xffffu)), g1 = bf2f((uint16_t)(goal >> 16));
#pragma unroll 1
        for (int mt = 0; mt < MT; ++mt) {
            if (n0 < H1) {
                f16v acc[NT1];
#pragma unroll
                for (int t4 = 0; t4 < NT1; ++t4) {
                    const float bb = a.theta[a.net.b_off[0] + n0 + 32 * t4 + l32];
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[t4][r] = bb;
                }
#pragma unroll 1
                for (int k0 = 0; k0 < n_cells; k0 += 16) {
                    bf8 av;
                    const int cell = k0 + 8 * kg;
                    const uint32_t bits = (obs[(mt * 32 + l32) * BOBS + (cell >> 5)] >> (cell & 31)) & 0xffu;
#pragma unroll
                    for (int u = 0; u < 8; ++u) av[u] = ((bits >> u) & 1u) ? (__bf16)1.0f : (__bf16)0.0f;
#pragma unroll
                    for (int t4 = 0; t4 < NT1; ++t4) {
                        const bf8 wv = *reinterpret_cast<const bf8*>(wb + ((size_t)(t4 * KS + (k0 >> 4)) << 9));
                        acc[t4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, wv, acc[t4], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int t4 = 0; t4 < NT1; ++t4)
#pragma unroll
                    for (int r = 0; r < 16; ++r) prefix[(8 * (r >> 2) + 4 * kg + (r & 3)) * (H1 + 4) + n0 + 32 * t4 + l32] = acc[t4][r];
            }
            __syncthreads();
#pragma unroll
            for (int m = 0; m < EPT; ++m)
                if (first_thread && (e00 + m) / 32 == mt) {
                    const float2 p = *reinterpret_cast<const float2*>(prefix + ((e00 + m) & 31) * (H1 + 4) + c0);
                    pre[ENV == ENV_MAZE ? m : 0][0] = p.x + g0;
                    pre[ENV == ENV_MAZE ? m : 0][1] = p.y + g1;
                }
            __syncthreads();
        }
    }
    float wp[3][2] = {{0, 0}, {0, 0}, {0, 0}};                     // pendulum: the three rows of W1
    if (ENV == ENV_PENDULUM) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t ww = *reinterpret_cast<const uint32_t*>(w1 + (size_t)k * H1 + c0);
            wp[k][0] = bf2f((uint16_t)(ww & 0xffffu)); wp[k][1] = bf2f((uint16_t)(ww >> 16));
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0): nothing loaded before the loop is waited for inside it

    float hv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float rew = 0.0f, actf = 0.0f, eps = 0.0f;
    int act = 0, done = 0;
    for (int t = 0; t <= T; ++t) {
        // everything derived from the thread index is worked out again every step from a value the compiler cannot see
        // through: dozens of loop-invariant addresses would otherwise be kept in registers, and spilled
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const bool keep = t < T && a.keep_acts;
        const size_t g8 = ((size_t)t * B + b0) >> 3;               // first sample group of this tile
        // ---- first layer: fp32 gather-sum / three fmas, rounded to bf16 ----
        if (first_thread) {
            const int c = 2 * (tid % (H1 / 2)), e0 = tid / (H1 / 2) * EPT;
            uint16_t* actP = keep ? reinterpret_cast<uint16_t*>(tp.act[0]) : nullptr;
            // weight rows of RB environments asked for before the first is used (two sets of loads: a pointer that may be LDS
            // or memory would make flat ones)
            constexpr int RB = EPT < 16 ? EPT : EPT == 16 ? 16 : 8;
            uint32_t r0[ENV == ENV_PENDULUM ? 1 : RB], r1[ENV == ENV_CATCH ? RB : 1];
            auto rows = [&](const uint16_t* base, int m1) __attribute__((always_inline)) {
                uint32_t cell[RB][2];
#pragma unroll
                for (int m = 0; m < RB; ++m) {
                    const uint32_t* o = obs + (e0 + m1 + m) * BOBS;
                    if (ENV == ENV_CATCH) { const uint2 v = *reinterpret_cast<const uint2*>(o); cell[m][0] = v.x; cell[m][1] = v.y; }
                    else cell[m][0] = o[8];
                }
#pragma unroll
                for (int m = 0; m < RB; ++m) {
                    r0[ENV == ENV_PENDULUM ? 0 : m] = *reinterpret_cast<const uint32_t*>(base + cell[m][0] * (uint32_t)H1 + c);
                    if (ENV == ENV_CATCH) r1[ENV == ENV_CATCH ? m : 0] = *reinterpret_cast<const uint32_t*>(base + cell[m][1] * (uint32_t)H1 + c);
                }
            };
            uint32_t mkx[2] = {0u, 0u}, mky[2] = {0u, 0u};         // ReLU masks of whole 32-sample stages (H1 = 512)
#pragma unroll
            for (int m0 = 0; m0 < EPT; m0 += GE) {
                if (ENV != ENV_PENDULUM && m0 % RB == 0) {
                    if (q.w1_lds) rows(w1s, m0);
                    else rows(w1 + (ENV == ENV_MAZE ? (size_t)n_cells * H1 : 0), m0);
                }
                float v[GE][2];
#pragma unroll
                for (int u = 0; u < GE; ++u) {
                    const int m = m0 + u;
                    float vx = ENV == ENV_MAZE ? pre[ENV == ENV_MAZE ? m : 0][0] : bias0;
                    float vy = ENV == ENV_MAZE ? pre[ENV == ENV_MAZE ? m : 0][1] : bias1;
                    if (ENV == ENV_PENDULUM) {
                        const float4 f = *reinterpret_cast<const float4*>(obs + (e0 + m) * BOBS);
                        const float x[3] = {f.x, f.y, f.z};
#pragma unroll
                        for (int k = 0; k < 3; ++k) { vx = fmaf(x[k], wp[k][0], vx); vy = fmaf(x[k], wp[k][1], vy); }
                    } else {
                        const uint32_t g = r0[ENV == ENV_PENDULUM ? 0 : m % RB];
                        vx += bf2f((uint16_t)(g & 0xffffu)); vy += bf2f((uint16_t)(g >> 16));
                        if (ENV == ENV_CATCH) {
                            const uint32_t g1 = r1[ENV == ENV_CATCH ? m % RB : 0];
                            vx += bf2f((uint16_t)(g1 & 0xffffu)); vy += bf2f((uint16_t)(g1 >> 16));
                        }
                    }
                    v[u][0] = relu(vx); v[u][1] = relu(vy);
                }
                uint32_t px[GE / 2], py[GE / 2];
#pragma unroll
                for (int u = 0; u < GE / 2; ++u) {
                    px[u] = pack_bf16x2(v[2 * u][0], v[2 * u + 1][0]);
                    py[u] = pack_bf16x2(v[2 * u][1], v[2 * u + 1][1]);
                    *reinterpret_cast<uint32_t*>(bufs + (e0 + m0 + 2 * u) * LDX + c) = (px[u] & 0xffffu) | (py[u] << 16);
                    *reinterpret_cast<uint32_t*>(bufs + (e0 + m0 + 2 * u + 1) * LDX + c) = (px[u] >> 16) | (py[u] & 0xffff0000u);
                }
                if (actP) {
                    uint16_t* dst = actP + ((g8 + ((e0 + m0) >> 3)) * H1 + c) * 8 + (GE == 8 ? 0 : e0 & 4);   // columns c, c + 1 of a group of eight samples
                    if constexpr (GE == 8) {
                        u32v4 x4, y4;
#pragma unroll
                        for (int u = 0; u < 4; ++u) { x4[u] = px[u]; y4[u] = py[u]; }
                        __builtin_nontemporal_store(x4, reinterpret_cast<u32v4*>(dst));
                        __builtin_nontemporal_store(y4, reinterpret_cast<u32v4*>(dst + 8));
                    } else {
                        u32v2 x2, y2;
#pragma unroll
                        for (int u = 0; u < 2; ++u) { x2[u] = px[u]; y2[u] = py[u]; }
                        __builtin_nontemporal_store(x2, reinterpret_cast<u32v2*>(dst));
                        __builtin_nontemporal_store(y2, reinterpret_cast<u32v2*>(dst + 8));
                    }
                    if constexpr (EPT == 32) {
#pragma unroll
                        for (int k2 = 0; k2 < 2; ++k2) {
                            mkx[k2] |= (nonzero_flags_pk(px[2 * k2]) << (m0 >> 2)) | (nonzero_flags_pk(px[2 * k2 + 1]) << ((m0 >> 2) + 1));
                            mky[k2] |= (nonzero_flags_pk(py[2 * k2]) << (m0 >> 2)) | (nonzero_flags_pk(py[2 * k2 + 1]) << ((m0 >> 2) + 1));
                        }
                    }
                }
            }
            if (actP && EPT == 32) {
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                    u32v2 mv; mv[0] = mkx[k2]; mv[1] = mky[k2];
                    __builtin_nontemporal_store(mv, reinterpret_cast<u32v2*>(tp.mask[0] + relu_mask_index((g8 >> 2) + (e0 >> 5), k2, H1, c)));
                }
            }
        }
        // ---- hidden layers: this wavefront's blocks ----
        int passed = 0;                                            // barriers passed in this step: layer l reads behind the l-th
        f16v acc[MT];
        int xi = 0;
        uint32_t pk[MT][8], pend = 0u;                             // a finished layer's packed outputs, stored to memory behind the barrier
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) asm volatile("" : "=v"(acc[mt]));
        const int l32 = lane & 31, kg = lane >> 5;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            uint32_t d = blk[i];
            asm volatile("" : "+s"(d));
            if (!(d & PinnedBf16Plan::VALID)) continue;
            const int l = (d >> PinnedBf16Plan::LAYER) & 3;
            if (d & PinnedBf16Plan::START) {
                float b = bv[i];
                xi = ((l - 1) & 1) * TM * LDX + l32 * LDX + 8 * kg;
                asm volatile("" : "+v"(b), "+v"(xi));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[mt][r] = b;
                while (passed < l) { __syncthreads(); ++passed; }
                pinned_bf16_flush<MT>(pend, pk, tp.act[1], tp.act[2], tp.act[3], tp.mask[1], tp.mask[2], tp.mask[3], g8, lane);
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                bf8 x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = *reinterpret_cast<const bf8*>(bufs + xi + mt * 32 * LDX + 16 * u);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[u], w[i][u], acc[mt], 0, 0, 0);
            }
            xi += 128;
            if (d & PinnedBf16Plan::END) {
                uint16_t* y = bufs + (l & 1) * TM * LDX + 4 * kg * LDX + 32 * ((d >> PinnedBf16Plan::TILE) & 31) + l32;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const uint32_t p01 = pack_bf16x2(relu(acc[mt][4 * g]), relu(acc[mt][4 * g + 1]));
                        const uint32_t p23 = pack_bf16x2(relu(acc[mt][4 * g + 2]), relu(acc[mt][4 * g + 3]));
                        uint16_t* o = y + (mt * 32 + 8 * g) * LDX;
                        o[0] = (uint16_t)p01; o[LDX] = (uint16_t)(p01 >> 16); o[2 * LDX] = (uint16_t)p23; o[3 * LDX] = (uint16_t)(p23 >> 16);
                        pk[mt][2 * g] = p01; pk[mt][2 * g + 1] = p23;
                    }
                if (keep) pend = d;
            }
        }
        while (passed < L) { __syncthreads(); ++passed; }
        // ---- heads: each of wavefronts 2 to 5 sums one quarter of the last layer for all environments; the records go beside it ----
        asm volatile("" : "+v"(tid));
        if (wave >= 2 && wave < 6) {
            const int l32 = tid & 31, kg = (tid & 63) >> 5, kq = wave - 2;
            auto quarter = [&](auto n) __attribute__((always_inline)) {
                constexpr int S = decltype(n)::value;              // steps of 16 inputs
                const uint16_t* wbs = whs + (l32 & 7) * ldh + 16 * S * kq + 8 * kg;   // (columns past the eighth: not used)
                bf8 hw[S];
#pragma unroll
                for (int s = 0; s < S; ++s) hw[s] = *reinterpret_cast<const bf8*>(wbs + 16 * s);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const uint16_t* xa = bufs + ((L - 1) & 1) * TM * LDX + (mt * 32 + l32) * LDX + 16 * S * kq + 8 * kg;
                    bf8 xv[S];
#pragma unroll
                    for (int s = 0; s < S; ++s) xv[s] = *reinterpret_cast<const bf8*>(xa + 16 * s);
                    f16v hacc;
#pragma unroll
                    for (int r = 0; r < 16; ++r) hacc[r] = 0.0f;
#pragma unroll
                    for (int s = 0; s < S; ++s) hacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[s], hw[s], hacc, 0, 0, 0);
                    if (l32 < 8) {
                        float* o = hp + (kq * TM + mt * 32 + 4 * kg) * 8 + l32;
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[(8 * (r >> 2) + (r & 3)) * 8] = hacc[r];
                    }
                }
            };
            if (HL == 128) quarter(std::integral_constant<int, 2>());
            else if (HL == 256) quarter(std::integral_constant<int, 4>());
            else quarter(std::integral_constant<int, 8>());
        } else if (owner) {
            kernarg_bf16 k = (kernarg_bf16)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(k));
            const size_t tb = (size_t)t * B + b0 + (tid & 63);
            k->r.tp.tr_s0[tb] = st.s0;
            if (ENV == ENV_PENDULUM) { k->r.tp.tr_f0[tb] = st.f0; k->r.tp.tr_f1[tb] = st.f1; }
            if (t > 0) {
                const size_t tq = tb - B;
                if (ENV == ENV_PENDULUM) { k->r.tp.tr_eps[tq] = eps; k->r.tp.tr_actf[tq] = actf; }
                else k->r.tp.tr_act[tq] = (uint8_t)act;
                k->r.tp.tr_rew[tq] = rew;
                k->r.tp.tr_done[tq] = (uint8_t)done;
                float* hd = k->r.tp.tr_head + tq * NHP;
                *reinterpret_cast<float4*>(hd) = make_float4(hv[0], hv[1], hv[2], hv[3]);
                if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = make_float4(hv[4], 0.0f, 0.0f, 0.0f);
                k->r.tp.tr_val[tq] = hv[NH - 1];
            }
        }
        pinned_bf16_flush<MT>(pend, pk, tp.act[1], tp.act[2], tp.act[3], tp.mask[1], tp.mask[2], tp.mask[3], g8, lane);
        __syncthreads();
        if (wave == 6 && t < T) draw(t + 1, tid & 63);
        if (owner) {
            const int lane = tid & 63;
            float4 part[4][NHP / 4];
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int u = 0; u < NHP / 4; ++u) part[p][u] = *reinterpret_cast<const float4*>(hp + (p * TM + lane) * 8 + 4 * u);
            const uint4 dr = *reinterpret_cast<const uint4*>(rng + ((t & 1) * TM + lane) * 4);
#pragma unroll
            for (int j = 0; j < NH; ++j) {
                float s = hb[j];
#pragma unroll
                for (int p = 0; p < 4; ++p) s += j % 4 == 0 ? part[p][j / 4].x : j % 4 == 1 ? part[p][j / 4].y : j % 4 == 2 ? part[p][j / 4].z : part[p][j / 4].w;
                hv[j] = s;
            }
            if (t < T) {
                if (ENV == ENV_PENDULUM) {
                    eps = f_from_bits(dr.x);
                    actf = gaussian_action(hv[0], hv[1], eps);
                    pendulum_step_sn(a.env, st, sine, actf, dr.z, dr.w, rew, done);
                } else {
                    act = sample_categorical_any(hv[0], hv[1], hv[2], hv[3], 0.0f, 0.0f, 0.0f, 0.0f, NH - 1, u01(dr.x));
                    if (ENV == ENV_CATCH) catch_step(a.env, st, act, dr.z, rew, done);
                    else {
                        const uint32_t* wl = obs + lane * BOBS;
                        maze_step(a.env, st, act, [wl](int c) { return ((wl[c >> 5] >> (c & 31)) & 1u) != 0u; }, rew, done);
                    }
                }
                observe(lane);
            }
        }
        __syncthreads();
    }
    if (owner) {
        const size_t tb = (size_t)T * B + b0 + lane0;
        float* hd = tp.tr_head + tb * NHP;
        *reinterpret_cast<float4*>(hd) = make_float4(hv[0], hv[1], hv[2], hv[3]);
        if (NHP == 8) *reinterpret_cast<float4*>(hd + 4) = make_float4(hv[4], 0.0f, 0.0f, 0.0f);
        tp.tr_val[tb] = hv[NH - 1];
        tp.s0[b0 + lane0] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b0 + lane0] = st.f0; tp.f1[b0 + lane0] = st.f1; }
    }
}

// Shares the blocks out: 32 outputs at a time to the wavefront with the fewest blocks of that layer on its SIMD, then the fewest at all
static bool pinned_bf16_share(const NetShape& net, PinnedBf16Plan& p)
{
    p = PinnedBf16Plan{};
    int load[PinnedBf16Plan::WAVES] = {0}, nb = 0;
    for (int l = 1; l < net.L; ++l) {
        const int K = net.dims[l], N = net.dims[l + 1], len = K / 128;
        int simd[4] = {0}, here[PinnedBf16Plan::WAVES] = {0};
        for (int tile = 0; tile < N / 32; ++tile) {
            int best = -1, best_key = 0;
            for (int w = 0; w < PinnedBf16Plan::WAVES; ++w) {
                const int key = ((simd[w & 3] * 16 + here[w]) * 2 + (w >= 2 && w < 6 ? 1 : 0)) * 16 + load[w];   // (2 to 5 have the heads)
                if (load[w] + len <= PinnedBf16Plan::MAX_BLOCKS && (best < 0 || key < best_key)) { best = w; best_key = key; }
            }
            if (best < 0) return false;
            for (int i = 0; i < len; ++i)
                p.block[best][load[best]++] = PinnedBf16Plan::VALID | (i == 0 ? PinnedBf16Plan::START : 0u) | (i == len - 1 ? PinnedBf16Plan::END : 0u) |
                                              (uint32_t)l << PinnedBf16Plan::LAYER | (uint32_t)__builtin_ctz(N) << PinnedBf16Plan::LGN |
                                              (uint32_t)tile << PinnedBf16Plan::TILE | (uint32_t)i << PinnedBf16Plan::KBLOCK;
            ++simd[best & 3]; ++here[best];
            if (load[best] > nb) nb = load[best];
        }
    }
    p.NB = nb <= 2 ? 2 : 4;
    return true;
}

static size_t pinned_bf16_lds(const NetShape& net, const EnvDims& env, int TM, int ldx, int* w1_lds)
{
    const int HL = net.dims[net.L], H1 = net.dims[1];
    size_t lds = (size_t)2 * TM * ldx * 2 + (size_t)8 * (HL + 8) * 2 + (size_t)4 * TM * 8 * 4 + (size_t)TM * BOBS * 4 + (size_t)2 * TM * 4 * 4;
    const size_t w1 = (size_t)(env.kind == ENV_MAZE ? env.rows * env.cols : net.dims[0]) * H1 * 2;
    *w1_lds = env.kind != ENV_PENDULUM && lds + w1 <= 160 * 1024 ? 1 : 0;
    return lds + (*w1_lds ? w1 : 0);
}

// 32 environments per workgroup while that leaves at most one workgroup per compute unit, 64 beyond (Catch 128-128, 65536
// environments: 253 us with 32, 188 with 64)
static int pinned_bf16_groups(int B) { return B <= 32 * 256 ? 1 : 2; }

// Nets whose blocks fit the registers.  Not the maze with a 512-wide first layer and 64 environments per workgroup: a thread's
// wall sums then take 64 registers beside the weights', and spill (512-128, 16384 environments: 211 us against 193 streaming).
bool pinned_bf16_ok(const anakin* h)
{
    PinnedBf16Plan p;
    if (h->mode & ANAKIN_MODE_STREAM_WEIGHTS) return false;
    if (h->env.kind == ENV_MAZE && h->net.dims[1] == 512 && pinned_bf16_groups(h->B) == 2) return false;
    return pinned_bf16_share(h->net, p);
}

// what: 0 the acting unroll, 1 the actor of a decoupled step
hipError_t launch_pinned_bf16(anakin* h, int what)
{
    PinnedBf16Args q;
    pinned_bf16_share(h->net, q.p);
    fill_bf16_args(h, what, q.r);
    const int MT = pinned_bf16_groups(h->B), H1 = h->net.dims[1];
    const int ldx = q.r.ldx <= 264 ? 264 : 520;
    const size_t lds = pinned_bf16_lds(h->net, h->env, 32 * MT, ldx, &q.w1_lds);
    auto launch = [&](auto kern) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        ProfScope prof(h, "rollout");
        hipLaunchKernelGGL(kern, dim3(h->B / (32 * MT)), dim3(BWG), lds, h->stream, q);
        return hipGetLastError();
    };
#define ANK_BF16_NB(ENVK, W, X, M) (q.p.NB == 2 ? launch(rollout_bf16_pinned_kernel<ENVK, W, X, M, 2>) : launch(rollout_bf16_pinned_kernel<ENVK, W, X, M, 4>))
#define ANK_BF16_M(ENVK, W, X) (MT == 1 ? ANK_BF16_NB(ENVK, W, X, 1) : ANK_BF16_NB(ENVK, W, X, 2))
#define ANK_BF16_X(ENVK, W) (ldx == 264 ? ANK_BF16_M(ENVK, W, 264) : ANK_BF16_M(ENVK, W, 520))
#define ANK_BF16_E(ENVK) (H1 == 128 ? ANK_BF16_X(ENVK, 128) : H1 == 256 ? ANK_BF16_X(ENVK, 256) : ANK_BF16_M(ENVK, 512, 520))
    switch (h->env.kind) {
        case ENV_CATCH:    return ANK_BF16_E(ENV_CATCH);
        case ENV_PENDULUM: return ANK_BF16_E(ENV_PENDULUM);
        default:           return ANK_BF16_E(ENV_MAZE);
    }
#undef ANK_BF16_E
#undef ANK_BF16_X
#undef ANK_BF16_M
#undef ANK_BF16_NB
}

}  // namespace ank
