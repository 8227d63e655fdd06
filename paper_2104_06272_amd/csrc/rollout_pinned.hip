// Acting with the hidden matrices in the register file, for nets of layers of different widths (or more than two).
//
// At these batches (at most one tile of 16 environments per compute unit) a step of the unroll is one dependent chain:
// first layer, matrix layers, heads, sample, step, observe.  What bounds it is the chain's latency: the fp32 matrix
// instruction (16 environments x 16 outputs x 4 inputs in 32 cycles, sequential along the inputs as the canonical order
// demands, and it chains at full rate), LDS round trips of 130 cycles, 4 to 8 cycles for every other instruction of a
// wavefront.  With the weights streamed from L2 each layer waited for memory as well, and a wavefront that streams has to
// leave stores to others (loads and stores complete in issue order).  So
//  - four wavefronts, one per SIMD, hold the hidden matrices (up to 24 blocks of 128 inputs x 16 outputs, 196 KB) and do
//    nothing but the layers between the barriers; where a layer has 32 outputs for each of them, two tiles share the
//    operand reads.  The host cuts the net into blocks (PinnedPlan); a block is 32 registers whose place in the code is
//    fixed and whose layer, inputs and outputs are scalars.
//  - four more own four environments each, a row of 16 lanes per environment: they sum the heads (lane j of the row head j;
//    the row's 16 inputs are handed round by the DPP row broadcast, so a step of the chain is one instruction), sample, step
//    and write the first layer's outputs, without a barrier or an exchange through LDS in between.
//  - records, random draws and copies of the activations are made by whichever kind waits for the other.
// (A form with v_mfma_f32_4x4x1 and tiles of four environments has the same instruction latency per input -- 12.6 to 15
// cycles against 8 or 16 -- and was slower where a layer has 64 outputs, 111 us against 106 on the net below.)
// An unroll against the streaming kernel: Catch 13 x 7, 256-128-64, 1008 environments, T = 24 150 -> 106 us; maze 9 x 13,
// 128-64, 1040, T = 23 89 -> 55; 128-128-128, 1024, T = 16 98 -> 66; pendulum 64-64-64, 2048, T = 20 79 -> 56.
// BF: bf16 nets that the bf16 matrix instructions do not take: weights, activations and features rounded to bfloat16, the
// arithmetic the same (pendulum 128-128, 48 environments, T = 20, vector ALU -> here: 509 -> 63 us).
#include <type_traits>
#include <string.h>
#include "acting.h"

namespace ank {


constexpr int PTM = 16;                                            // environments per workgroup
constexpr int PCW = PinnedPlan::WAVES;                           // wavefronts that compute the hidden layers, one per SIMD
constexpr int PTHR = 64 * PCW + 256;                               // and four more that own four environments each
struct PinnedArgs {
    RolloutArgs r;
    PinnedPlan p;
    int w1_lds;                  // first-layer rows (maze: agent plane and goal row) in LDS
    int xo[MAX_LAYERS];          // LDS offset of layer l's outputs, in floats: [16][dims + 4]
    int o_wh, o_b1, o_rng, o_obs, o_pre, o_w1;
};
typedef const __attribute__((address_space(4))) PinnedArgs* kernarg;

template <int ENV, int NB, bool BF>
__global__ __launch_bounds__(PTHR, 2) void rollout_pinned_kernel(const PinnedArgs q)
{
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH <= 4 ? 4 : 8;
    constexpr int PF = 8;                                          // LDS reads run this many steps ahead of their MFMAs
    constexpr int HREG = 128;                      // head inputs whose weights fit the owners' registers
    const RolloutArgs& a = q.r;
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int L = a.net.L, H1 = a.net.dims[1], HL = a.net.dims[L], D = a.net.dims[0], B = a.B, T = a.T;
    const int n_cells = a.env.rows * a.env.cols;
    float* whs = smem + q.o_wh;                                    // [NH][HL + 4] head weights, transposed (HL > HREG)
    float* b1s = smem + q.o_b1;                                    // [H1] biases of the first layer
    uint32_t* rng = reinterpret_cast<uint32_t*>(smem + q.o_rng);   // [2][16][4] draws
    uint32_t* obs = reinterpret_cast<uint32_t*>(smem + q.o_obs);   // maze: [16][OBS_WORDS], walls
    float* pre = smem + q.o_pre;                                   // maze: [16][H1] wall sums
    float* w1s = smem + q.o_w1;                                    // first-layer rows
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * PTM;

    const int ldw = HL + 4;
    // what goes to LDS; every wavefront asks for what it keeps in registers first
    auto fill = [&]() __attribute__((always_inline)) {
        if (HL > HREG)
            for (int i = tid; i < HL * NH; i += PTHR) whs[(i % NH) * ldw + i / NH] = round1<BF>(a.theta[a.net.wh_off + i]);
        for (int i = tid; i < H1; i += PTHR) b1s[i] = a.theta[a.net.b_off[0] + i];
        if (q.w1_lds) {
            const f4v* src = reinterpret_cast<const f4v*>(w1g + (ENV == ENV_MAZE ? (size_t)n_cells * H1 : 0));
            f4v* dst = reinterpret_cast<f4v*>(w1s);
            const int n4 = (ENV == ENV_MAZE ? n_cells : D) * H1 / 4;
            for (int i0 = 0; i0 < n4; i0 += 4 * PTHR) {
                f4v v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { const int i = i0 + u * PTHR + tid; v[u] = src[i < n4 ? i : 0]; }
#pragma unroll
                for (int u = 0; u < 4; ++u) { const int i = i0 + u * PTHR + tid; if (i < n4) { round4<BF>(v[u]); dst[i] = v[u]; } }
            }
            if (ENV == ENV_MAZE)
                for (int i = tid; i < H1; i += PTHR) w1s[(size_t)n_cells * H1 + i] = round1<BF>(w1g[(size_t)(3 * n_cells - 1) * H1 + i]);
        }
        if (ENV == ENV_MAZE) {
            for (int i = tid; i < PTM * 8; i += PTHR) obs[(i >> 3) * OBS_WORDS + (i & 7)] = tp.walls[(size_t)(i & 7) * B + b0 + (i >> 3)];
            __syncthreads();
            maze_prefix<BF, PTHR>(a, PTM, obs, w1g, b1s, pre, tid);
        }
    };
    const int lane0 = lane;
    // the draws of step t for all environments of the workgroup: the action's two words (pendulum: noise), the reset's
    auto draw = [&](int t, int lane) __attribute__((always_inline)) {
        if (lane >= 2 * PTM) return;
        const int m = lane & (PTM - 1);
        const bool reset = lane >= PTM;
        const u32x4 v = philox(a.seed, (uint32_t)(b0 + m), a.gstep + (uint64_t)t, reset ? DOM_RESET : DOM_ACTION);
        const uint32_t v0 = (ENV == ENV_PENDULUM && !reset) ? bits_from_f(gaussian_noise(v.x, v.y)) : v.x;
        *reinterpret_cast<uint2*>(rng + ((t & 1) * PTM + m) * 4 + (reset ? 2 : 0)) = make_uint2(v0, v.y);
    };

    if (wave < PCW) {
        // ==== the hidden layers ====================================================
        float w[NB][32], bv[NB];                                   // this wavefront's blocks, in matrix-core operand order
        uint32_t blk[NB], place[NB];
        const __amdgpu_buffer_rsrc_t theta = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.theta), 0, (uint32_t)a.net.P * 4u, 0x00020000);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const uint32_t d = q.p.block[wave][i][0];
            blk[i] = d; place[i] = q.p.block[wave][i][1];
            const int l = (d >> PinnedPlan::LAYER) & 3, N = a.net.dims[l + 1], col = 16 * ((d >> PinnedPlan::TILE) & 31) + (lane & 15);
            if (d & PinnedPlan::VALID) {
                const int k0 = 128 * ((d >> PinnedPlan::KBLOCK) & 3), n = d & PinnedPlan::HALF ? 16 : 32;
                const uint32_t off = 4u * (uint32_t)((lane >> 4) * N + col);
#pragma unroll
                for (int u = 0; u < 32; ++u) w[i][u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(theta, off, 4 * (a.net.w_off[l] + (k0 + (u < n ? 4 * u : 0)) * N), 0));
#pragma unroll
                for (int u = 0; u < 32; u += 2) round2<BF>(w[i][u], w[i][u + 1]);
                bv[i] = a.theta[a.net.b_off[l] + col];
            } else {
#pragma unroll
                for (int u = 0; u < 32; ++u) w[i][u] = 0.0f;
                bv[i] = 0.0f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        fill();
        if (wave == 0) draw(0, lane);
        __syncthreads();
        __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt(0): inside the loop a wait for a load would be one for every older store
        for (int t = 0; t <= T; ++t) {
            // everything derived from the lane is worked out again from a value the compiler cannot see through: dozens of
            // loop-invariant addresses would otherwise be kept in registers, on top of the weights, and spilled
            int lane = lane0;
            asm volatile("" : "+v"(lane));
            int passed = 0;                                        // barriers passed in this step: layer l reads behind the l-th
            f4v acc[2];
            float x[PF];                                           // ring of operands read ahead
            int xi = 0, yi = 0, ldy = 0;                           // LDS places of the next operand and of the outputs, distance of output rows
            // (set to whatever is there: a wavefront's first block always starts outputs, but to the compiler these would
            // be values of the step before)
            asm volatile("" : "=v"(acc[0]), "=v"(acc[1]));
#pragma unroll
            for (int u = 0; u < PF; ++u) asm volatile("" : "=v"(x[u]));
            auto start = [&](uint32_t d, uint32_t e, float b0, float b1) __attribute__((always_inline)) {
                const int l = (d >> PinnedPlan::LAYER) & 3, ldx = (1 << ((d >> PinnedPlan::LGK) & 15)) + 4;
                ldy = (1 << ((d >> PinnedPlan::LGN) & 15)) + 4;
                xi = 4 * (e & 0xffffu) + (int)__umul24((unsigned)lane & 15u, (unsigned)ldx) + (lane >> 4);
                yi = 4 * (e >> PinnedPlan::YOFF) + (int)__umul24((unsigned)(lane >> 4), 4u * (unsigned)ldy) + (lane & 15);
                asm volatile("" : "+v"(xi), "+v"(yi), "+v"(b0), "+v"(b1));   // worked out here, not behind the barrier (nor kept across steps)
                acc[0][0] = b0; acc[0][1] = b0; acc[0][2] = b0; acc[0][3] = b0;
                acc[1][0] = b1; acc[1][1] = b1; acc[1][2] = b1; acc[1][3] = b1;
                __builtin_amdgcn_sched_barrier(0);
                while (passed < l) { __syncthreads(); ++passed; }
#pragma unroll
                for (int u = 0; u < PF; ++u) x[u] = smem[xi + 4 * u];
            };
            auto end = [&](int j) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; r += 2) {
                    float a0 = acc[j][r] > 0.0f ? acc[j][r] : 0.0f, a1 = acc[j][r + 1] > 0.0f ? acc[j][r + 1] : 0.0f;
                    round2<BF>(a0, a1);
                    smem[yi + r * ldy + 16 * j] = a0; smem[yi + (r + 1) * ldy + 16 * j] = a1;
                }
            };
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                uint32_t d = blk[i], e = place[i];
                asm volatile("" : "+s"(d), "+s"(e));
                const bool pair = i + 1 < NB && i % 2 == 0 && (d & PinnedPlan::PAIR);
                if (!(d & PinnedPlan::VALID) || (i % 2 == 1 && (d & PinnedPlan::PAIR))) continue;   // (done with the one before)
                if (d & PinnedPlan::START) start(d, e, bv[i], bv[i + 1 < NB ? i + 1 : i]);
                auto steps = [&](auto two, auto from, auto to) __attribute__((always_inline)) {
#pragma unroll
                    for (int s = decltype(from)::value; s < decltype(to)::value; ++s) {
                        const float av = x[s % PF];
                        x[s % PF] = smem[xi + 4 * (s + PF)];             // (past these outputs' last input: what follows in LDS, not used)
                        __builtin_amdgcn_sched_barrier(0);
                        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, w[i][s], acc[0], 0, 0, 0);
                        if (decltype(two)::value) acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, w[i + 1 < NB ? i + 1 : i][s], acc[1], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                typedef std::integral_constant<int, 0> c0;
                typedef std::integral_constant<int, 16> c16;
                typedef std::integral_constant<int, 32> c32;
                if (pair) {
                    steps(std::true_type(), c0(), c16());
                    if (!(d & PinnedPlan::HALF)) steps(std::true_type(), c16(), c32());
                } else {
                    steps(std::false_type(), c0(), c16());
                    if (!(d & PinnedPlan::HALF)) steps(std::false_type(), c16(), c32());
                }
                xi += 128;
                if (d & PinnedPlan::END) {
                    end(0);
                    if (pair) end(1);
                }
            }
            while (passed < L) { __syncthreads(); ++passed; }
            // ---- while the environments step: the next draws, the activations' record (h_1 is recorded by its owners) ----
            asm volatile("" : "+v"(lane));
            if (t < T) {
                kernarg k = (kernarg)__builtin_amdgcn_kernarg_segment_ptr();
                asm volatile("" : "+s"(k));
                if (wave == 0) draw(t + 1, lane);
                if (a.keep_acts)
                    for (int l = 1; l < L; ++l) {
                        const int N = k->r.net.dims[l + 1], s4 = 29 - __builtin_clz((uint32_t)N);
                        f4v* dst = reinterpret_cast<f4v*>(k->r.tp.act[l] + ((size_t)t * B + b0) * N);
                        const float* src = smem + k->xo[l];
#pragma unroll 2
                        for (int i = 64 * wave + lane; i < (PTM << s4); i += 64 * PCW) dst[i] = *reinterpret_cast<const f4v*>(src + (i >> s4) * (N + 4) + 4 * (i & ((1 << s4) - 1)));
                    }
            }
        }
        return;
    }

    // ==== environments: row r of 16 lanes is environment r of the wavefront's four ==================
    const int row0 = 4 * (wave - PCW);
    float hw[HREG];                                                // lane j: weights of head j
#pragma unroll
    for (int u = 0; u < HREG; ++u) hw[u] = 0.0f;
    {
        const float* src = a.theta + a.net.wh_off + ((lane & 15) < NH ? lane & 15 : 0);
        if (HL <= HREG) {
#pragma unroll
            for (int u = 0; u < 64; ++u) hw[u] = src[u * NH];
        }
        if (HL == HREG) {
#pragma unroll
            for (int u = 64; u < HREG; ++u) hw[u] = src[u * NH];
        }
    }
#pragma unroll
    for (int u = 0; u < HREG; u += 2) round2<BF>(hw[u], hw[u + 1]);
    EnvState st{0u, 0.0f, 0.0f};
    st.s0 = tp.s0[b0 + row0 + (lane >> 4)];
    if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b0 + row0 + (lane >> 4)]; st.f1 = tp.f1[b0 + row0 + (lane >> 4)]; }
    const float hbias = a.theta[a.net.bh_off + ((lane & 15) < NH ? lane & 15 : 0)];
    __builtin_amdgcn_sched_barrier(0);
    fill();
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0)

    const int lg1 = 31 - __builtin_clz((uint32_t)H1);
    float* X1 = smem + q.xo[0];
    float sine = 0.0f, hv = 0.0f, rew = 0.0f, actf = 0.0f, eps = 0.0f;
    int act = 0, done = 0;
    // observe and first layer of this wavefront's four environments
    auto first = [&](int lane) __attribute__((always_inline)) {
        const int row = row0 + (lane >> 4), i16 = lane & 15;
        float* x1 = X1 + (int)__umul24((unsigned)row, (unsigned)(H1 + 4));
        // NP pieces of four columns, 64 columns apart: all loads, then all stores (which might be the same memory, for all the
        // compiler knows: one piece at a time is one LDS round trip each, 400 cycles)
        auto out = [&](int c0, f4v v) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
            round4<BF>(v);
            *reinterpret_cast<f4v*>(x1 + c0) = v;
        };
        auto gather = [&](auto n, int c0, const float* base, const float* r0, const float* r1) __attribute__((always_inline)) {
            constexpr int NP = decltype(n)::value;
            f4v v[NP], u0[NP], u1[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                v[p] = *reinterpret_cast<const f4v*>(base + c0 + 64 * p);
                u0[p] = *reinterpret_cast<const f4v*>(r0 + c0 + 64 * p);
                u1[p] = *reinterpret_cast<const f4v*>(r1 + c0 + 64 * p);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!q.w1_lds) {                                       // (rows in LDS are rounded already)
#pragma unroll
                for (int p = 0; p < NP; ++p) { round4<BF>(u0[p]); round4<BF>(u1[p]); }
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) { v[p] += u0[p]; v[p] += u1[p]; out(c0 + 64 * p, v[p]); }
        };
        auto features = [&](auto n, int c0, const float (&f)[3]) __attribute__((always_inline)) {
            constexpr int NP = decltype(n)::value;
            f4v v[NP], u[NP][3];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                v[p] = *reinterpret_cast<const f4v*>(b1s + c0 + 64 * p);
#pragma unroll
                for (int k = 0; k < 3; ++k) u[p][k] = *reinterpret_cast<const f4v*>(w1s + k * H1 + c0 + 64 * p);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[p][e] = fmaf(f[k], u[p][k][e], v[p][e]);
                out(c0 + 64 * p, v[p]);
            }
        };
        auto all = [&](auto piece) __attribute__((always_inline)) {
            if (H1 == 64) piece(std::integral_constant<int, 1>(), 4 * i16);
            else if (H1 == 128) piece(std::integral_constant<int, 2>(), 4 * i16);
            else {
#pragma unroll 1
                for (int c0 = 4 * i16; c0 < H1; c0 += ENV == ENV_PENDULUM ? 128 : 256) piece(std::integral_constant<int, ENV == ENV_PENDULUM ? 2 : 4>(), c0);
            }
        };
        // (two separate sets of loads: a pointer that may be either would make flat loads)
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            if (q.w1_lds) all([&](auto n, int c0) __attribute__((always_inline)) { gather(n, c0, b1s, w1s + (bc << lg1), w1s + (pc << lg1)); });
            else all([&](auto n, int c0) __attribute__((always_inline)) { gather(n, c0, b1s, w1g + (bc << lg1), w1g + (pc << lg1)); });
        } else if (ENV == ENV_MAZE) {
            const int cell = (int)(st.s0 & 0xffffu);
            if (q.w1_lds) all([&](auto n, int c0) __attribute__((always_inline)) { gather(n, c0, pre + (row << lg1), w1s + (cell << lg1), w1s + (n_cells << lg1)); });
            else all([&](auto n, int c0) __attribute__((always_inline)) { gather(n, c0, pre + (row << lg1), w1g + ((size_t)(n_cells + cell) << lg1), w1g + ((size_t)(3 * n_cells - 1) << lg1)); });
        } else {
            float f[3];
            det_sincos(st.f0, sine, f[0]);
            f[0] = round1<BF>(f[0]); f[1] = round1<BF>(sine); f[2] = round1<BF>(st.f1);
            all([&](auto n, int c0) __attribute__((always_inline)) { features(n, c0, f); });
        }
    };
    first(lane);

    for (int t = 0; t <= T; ++t) {
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        kernarg k = (kernarg)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(k));
        const int i16 = lane & 15, r16 = lane >> 4;
        __syncthreads();
        // ---- while the layers run: records of the step before and of this step's state, h_1, this step's draws ----
        {
            const int b = b0 + row0 + r16;
            const size_t tb = (size_t)t * B + b;
            if (i16 == 0) {
                k->r.tp.tr_s0[tb] = st.s0;
                if (ENV == ENV_PENDULUM) { k->r.tp.tr_f0[tb] = st.f0; k->r.tp.tr_f1[tb] = st.f1; }
                if (t > 0) {
                    const size_t tq = tb - B;
                    if (ENV == ENV_PENDULUM) { k->r.tp.tr_eps[tq] = eps; k->r.tp.tr_actf[tq] = actf; }
                    else k->r.tp.tr_act[tq] = (uint8_t)act;
                    k->r.tp.tr_rew[tq] = rew;
                    k->r.tp.tr_done[tq] = (uint8_t)done;
                }
            }
            if (t > 0) {
                if (i16 < NHP) k->r.tp.tr_head[(tb - B) * NHP + i16] = i16 < NH ? hv : 0.0f;
                if (i16 == NH - 1) k->r.tp.tr_val[tb - B] = hv;
            }
            if (t < T && a.keep_acts) {
                const float* x1 = X1 + (row0 + r16) * (H1 + 4);
#pragma unroll 1
                for (int c0 = 4 * i16; c0 < H1; c0 += 64) *reinterpret_cast<f4v*>(k->r.tp.act[0] + tb * H1 + c0) = *reinterpret_cast<const f4v*>(x1 + c0);
            }
        }
        // ---- heads: row r of lanes, lane j of it head j ----
        asm volatile("" : "+v"(lane));
        hv = hbias;
        int xi = q.xo[L - 1] + (int)__umul24((unsigned)(row0 + (lane >> 4)), (unsigned)(HL + 4)) + (lane & 15), di = ((t & 1) * PTM + row0 + (lane >> 4)) * 4;
        asm volatile("" : "+v"(xi), "+v"(di));                     // worked out here, not behind the barriers
        __builtin_amdgcn_sched_barrier(0);
        for (int l = 1; l < L; ++l) __syncthreads();
        const uint4 dr = *reinterpret_cast<const uint4*>(rng + di);
        if (HL <= HREG) {
            float xh[HREG / 16];
#pragma unroll
            for (int u = 0; u < HREG / 16; ++u) xh[u] = smem[xi + (16 * u < HL ? 16 * u : 0)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < HREG / 16; ++u)
                if (16 * u < HL)
                    chain16(xh[u], f4v{hw[16 * u], hw[16 * u + 1], hw[16 * u + 2], hw[16 * u + 3]}, f4v{hw[16 * u + 4], hw[16 * u + 5], hw[16 * u + 6], hw[16 * u + 7]},
                            f4v{hw[16 * u + 8], hw[16 * u + 9], hw[16 * u + 10], hw[16 * u + 11]}, f4v{hw[16 * u + 12], hw[16 * u + 13], hw[16 * u + 14], hw[16 * u + 15]}, hv);
        } else {
            const f4v* wr = reinterpret_cast<const f4v*>(whs + ((lane & 15) < NH ? lane & 15 : 0) * ldw);
            float xa = smem[xi], xb;
            f4v wa[4], wb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) wa[u] = wr[u];
#pragma unroll 1
            for (int k0 = 0; k0 < HL; k0 += 32) {
                xb = smem[xi + k0 + 16];
#pragma unroll
                for (int u = 0; u < 4; ++u) wb[u] = wr[k0 / 4 + 4 + u];
                __builtin_amdgcn_sched_barrier(0);
                chain16(xa, wa[0], wa[1], wa[2], wa[3], hv);
                const int kn = k0 + 32 < HL ? k0 + 32 : 0;
                xa = smem[xi + kn];
#pragma unroll
                for (int u = 0; u < 4; ++u) wa[u] = wr[kn / 4 + u];
                __builtin_amdgcn_sched_barrier(0);
                chain16(xb, wb[0], wb[1], wb[2], wb[3], hv);
            }
        }
        if (t == T) break;
        // ---- sample, step; all lanes of a row do the same ----
        row_step<ENV>(a.env, st, sine, hv, dr, obs + (row0 + (lane >> 4)) * OBS_WORDS, eps, actf, act, rew, done);
        asm volatile("" : "+v"(lane));
        first(lane);
    }
    const int i16 = lane & 15, b = b0 + row0 + (lane >> 4);
    const size_t tb = (size_t)T * B + b;
    if (i16 < NHP) tp.tr_head[tb * NHP + i16] = i16 < NH ? hv : 0.0f;
    if (i16 == NH - 1) tp.tr_val[tb] = hv;
    if (i16 == 0) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// LDS of a workgroup; offsets in floats
static size_t pinned_lds(const NetShape& net, const EnvDims& env, PinnedArgs& q)
{
    const int H1 = net.dims[1], HL = net.dims[net.L], cells = env.rows * env.cols;
    int off = 0;
    for (int l = 0; l < net.L; ++l) { q.xo[l] = off; off += PTM * (net.dims[l + 1] + 4); }
    q.o_wh = off; off += 8 * (HL + 4);
    q.o_b1 = off; off += H1;
    q.o_rng = off; off += 2 * PTM * 4;
    q.o_obs = off; off += env.kind == ENV_MAZE ? PTM * OBS_WORDS : 0;
    q.o_pre = off; off += env.kind == ENV_MAZE ? PTM * H1 : 0;
    q.o_w1 = off;
    const int w1 = (env.kind == ENV_MAZE ? cells + 1 : net.dims[0]) * H1;
    q.w1_lds = (size_t)(off + w1) * 4 <= 160 * 1024 ? 1 : 0;
    if (q.w1_lds) off += w1;
    return (size_t)off * 4;
}

// Shares the blocks out, 16 outputs at a time or, where a layer has enough of them, 32 (a pair of blocks at even places,
// which read their inputs once): to the wavefront with the fewest blocks of that layer, then the fewest at all
static bool pinned_share(const NetShape& net, const int* xo, PinnedPlan& p)
{
    memset(&p, 0, sizeof p);
    int load[PCW] = {0}, nb = 0;
    for (int l = 1; l < net.L; ++l) {
        const int K = net.dims[l], N = net.dims[l + 1], len = (K + 127) / 128, step = N / 16 >= 2 * PCW ? 2 : 1;
        int here[PCW] = {0};
        for (int tile = 0; tile < N / 16; tile += step) {
            int best = -1;
            for (int w = 0; w < PCW; ++w) {
                const int first = step == 2 ? (load[w] + 1) / 2 * 2 : load[w];
                if (first + step * len <= PinnedPlan::MAX_BLOCKS && (best < 0 || here[w] * 64 + load[w] < here[best] * 64 + load[best])) best = w;
            }
            if (best < 0) return false;
            if (step == 2) load[best] = (load[best] + 1) / 2 * 2;
            for (int i = 0; i < len * step; ++i) {
                const int kb = i / step, tl = tile + i % step;
                uint32_t* b = p.block[best][load[best]++];
                b[0] = PinnedPlan::VALID | (kb == 0 ? PinnedPlan::START : 0u) | (kb == len - 1 ? PinnedPlan::END : 0u) | (K == 64 ? PinnedPlan::HALF : 0u) | (step == 2 ? PinnedPlan::PAIR : 0u) |
                       (uint32_t)l << PinnedPlan::LAYER | (uint32_t)__builtin_ctz(K) << PinnedPlan::LGK | (uint32_t)__builtin_ctz(N) << PinnedPlan::LGN |
                       (uint32_t)tl << PinnedPlan::TILE | (uint32_t)kb << PinnedPlan::KBLOCK;
                b[1] = (uint32_t)(xo[l - 1] / 4) << PinnedPlan::XOFF | (uint32_t)((xo[l] + 16 * tl) / 4) << PinnedPlan::YOFF;
            }
            here[best] += len * step;
            if (load[best] > nb) nb = load[best];
        }
    }
    p.NB = nb <= 4 ? 4 : 6;
    return true;
}

// Which nets act with this kernel: two or more layers of 64 to 512 units whose blocks fit 4 x 6 (but rollout_wide.hip's
// wide_before_pinned), and at most one tile of 16 environments per compute unit -- beyond that the streaming kernel takes more environments per tile and shares its weight
// stream among them (256-128-64, 8192 environments: 220 us against 208 here, 64-64-64 99 against 109).  Two equal layers
// keep the kernels that have their width as a constant: eight wavefronts share their one matrix layer, four here
// (pendulum, 128-128: 89 us against 97; Catch, 64-64: 31.7 against 32.6).
void rollout_pinned_plan(const NetShape& net, const EnvDims& env, int B, PinnedPlan& p)
{
    memset(&p, 0, sizeof p);
    if (net.L < 2 || B > PTM * 256 || rollout_resident_tile(net, env.kind, B)) return;
    for (int l = 1; l <= net.L; ++l) if (net.dims[l] % 64 || net.dims[l] > 512) return;
    PinnedArgs q;
    if (pinned_lds(net, env, q) > 160 * 1024 || (env.kind == ENV_PENDULUM && !q.w1_lds) || !pinned_share(net, q.xo, p)) p.NB = 0;
}

template <int ENV>
static hipError_t launch_pinned_env(anakin* h, const PinnedArgs& q, size_t lds)
{
    auto kern = h->net.bf16 ? (q.p.NB == 4 ? rollout_pinned_kernel<ENV, 4, true> : rollout_pinned_kernel<ENV, 6, true>)
                            : (q.p.NB == 4 ? rollout_pinned_kernel<ENV, 4, false> : rollout_pinned_kernel<ENV, 6, false>);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, "rollout");
    hipLaunchKernelGGL(kern, dim3(h->B / PTM), dim3(PTHR), lds, h->stream, q);
    return hipGetLastError();
}

hipError_t launch_pinned(anakin* h, const RolloutArgs& args)
{
    PinnedArgs q;
    q.r = args; q.p = h->pinned;
    const size_t lds = pinned_lds(h->net, h->env, q);
    switch (h->env.kind) {
        case ENV_CATCH:    return launch_pinned_env<ENV_CATCH>(h, q, lds);
        case ENV_PENDULUM: return launch_pinned_env<ENV_PENDULUM>(h, q, lds);
        default:           return launch_pinned_env<ENV_MAZE>(h, q, lds);
    }
}

}  // namespace ank
