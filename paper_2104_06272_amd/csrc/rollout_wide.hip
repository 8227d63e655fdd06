// Acting of nets with wide layers at batches that leave compute units idle in tiles of 16 environments: 4 or 8 environments
// per workgroup, a workgroup per compute unit.
//
// What bounds it: an input costs the 16 x 16 x 4 matrix instruction eight cycles for 16 environments however few of them
// exist, and the weights of a step have to reach the compute unit -- a stream from L2 runs at 26 bytes per cycle and unit
// (36 with 16-byte loads through LDS, which then cost as much in LDS passes), 8 us for a 256 x 512 matrix every step.  So
//  - the products are v_mfma_f32_4x4x1: 4 environments x 64 outputs of one input in eight cycles, chained along the inputs as
//    the canonical order demands (a chain alone 12.6 cycles an input, two on a SIMD 16.7);
//  - weights stay on chip as far as they fit: ten chunks (16 inputs of 64 outputs) in each wavefront's registers, what LDS has
//    left behind that, and only the rest is streamed, two chunks ahead, across layers and steps;
//  - a layer with fewer than eight blocks of 64 outputs is cut along its inputs as well, a stage with a barrier each: the
//    chain is serial anyway, and every wavefront's registers hold a part;
//  - wavefront g also owns four environments, a row of 16 lanes each (heads by DPP row broadcast, sample, step); the others
//    meanwhile write the records, which reach them through LDS, and make the next draws; everybody takes part in the first
//    layer.
// An unroll of T = 16 (Catch 10 x 5; before: streaming kernel, for 256-256 the resident one), environments 64 / 1024 / 2048:
// 256-256 105 -> 75, 107 -> 80, 108 -> 99 us; 512-256 199 -> 128, 205 -> 136, 207 -> 176; 256-512 217 -> 122, 222 -> 132,
// 228 -> 165; 512-512 360 -> 249, 363 -> 264, 365 -> 314; 64-512 111 -> 71, 115 -> 76, 117 -> 86; 256-256-256 209 -> 133,
// 213 -> 140, 215 -> 175.  bf16 nets off the bf16 matrix path, 48 / 1040 / 2032: 256-256 160 -> 75, 163 -> 97, 166 -> 98;
// 512-512 500 -> 273, 506 -> 306, 507 -> 328.
#include <string.h>
#include "acting.h"

namespace ank {

constexpr int WW = 8;                                              // wavefronts of a workgroup
constexpr int WTHR = 64 * WW;
// A wavefront's share of a layer: 64 outputs, the inputs (or a cut of them) in chunks of 16 -- streamed ones first, then
// those in LDS, then those in registers.
struct WideJob {
    int stage;                   // barriers to pass before it
    int first, relu;             // starts from the bias (else from what the stage before left); ends the outputs
    uint32_t off, n4;            // bytes: its first weight, distance of two inputs
    int x, gs;                   // LDS: its first input, distance of two groups
    int y, ygs, bias;            // LDS: its outputs, distance of two groups, bias
    int n_stream, n_lds, n_reg;  // chunks; streamed: an even number
};
struct WidePlan {
    static constexpr int MAX_JOBS = 3;
    WideJob job[WW][MAX_JOBS];
    int slots;                   // most jobs of a wavefront: the register chunks are shared out among them evenly
    int jobs[WW], streamed[WW];
    int barriers;                // of a step
    int lds;                     // chunks in LDS per wavefront
    uint32_t lds_bytes;
};
struct WideArgs {
    RolloutArgs r;
    WidePlan p;
    int w1_lds;                  // first-layer rows (maze: agent plane and goal row) in LDS
    int xo[MAX_LAYERS];          // LDS offset of layer l's outputs, in floats: [R][dims][4 environments]
    int o_wh, o_b1, o_bias, o_rng, o_seen, o_obs, o_pre, o_w, o_w1;
};
static_assert(sizeof(WideArgs) <= 4096, "kernel arguments");
typedef const __attribute__((address_space(4))) WideArgs* kernarg_w;
constexpr int wide_slot(int slots) { return slots == 1 ? 10 : slots == 2 ? 5 : 3; }   // register chunks of a job

// 16 inputs of 64 outputs: x[g] holds x[environment lane % 4][input lane / 4] of group g; the broadcast control hands the
// four lanes of input KK to all 16 blocks of the instruction.  next(kk): asks for what comes behind, once w[kk] is used.
template <int R, int KK, class Next>
__device__ __forceinline__ void quad_mfma(const float (&x)[R], float (&w)[16], f4v (&acc)[R], const Next& next)
{
    if constexpr (KK < 16) {
#pragma unroll
        for (int g = 0; g < R; ++g) acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[g], w[KK], acc[g], 4, KK, 0);
        next(KK);
        __builtin_amdgcn_sched_barrier(0);
        quad_mfma<R, KK + 1>(x, w, acc, next);
    }
}

template <int ENV, int R, int SLOTS, bool BF>
__global__ __launch_bounds__(WTHR, 2) void rollout_wide_kernel(const WideArgs q)
{
    constexpr int NH = ENV == ENV_CATCH ? 4 : ENV == ENV_PENDULUM ? 3 : 5, NHP = NH <= 4 ? 4 : 8;
    constexpr int TM = 4 * R, SC = wide_slot(SLOTS), PC = SC * SLOTS;
    const RolloutArgs& a = q.r;
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int L = a.net.L, H1 = a.net.dims[1], HL = a.net.dims[L], D = a.net.dims[0], B = a.B, T = a.T;
    const int n_cells = a.env.rows * a.env.cols;
    float* whs = smem + q.o_wh;                                    // [NH][HL + 4] head weights, transposed
    float* b1s = smem + q.o_b1;                                    // [H1] biases of the first layer
    float* bias = smem + q.o_bias;                                 // biases of the hidden layers, one behind the other
    uint32_t* rng = reinterpret_cast<uint32_t*>(smem + q.o_rng);   // [2][TM][4] draws
    uint32_t* obs = reinterpret_cast<uint32_t*>(smem + q.o_obs);   // maze: [TM][OBS_WORDS], walls
    float* pre = smem + q.o_pre;                                   // maze: [TM][H1] wall sums
    float* w1s = smem + q.o_w1;                                    // first-layer rows
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];
    const int tid = threadIdx.x, lane0 = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.x * TM, ldw = HL + 4;

    // ---- what goes to LDS ----
    for (int i = tid; i < HL * NH; i += WTHR) whs[(i % NH) * ldw + i / NH] = round1<BF>(a.theta[a.net.wh_off + i]);
    for (int i = tid; i < H1; i += WTHR) b1s[i] = a.theta[a.net.b_off[0] + i];
    {
        float* dst = bias;
        for (int l = 1; l < L; ++l) {
            for (int i = tid; i < a.net.dims[l + 1]; i += WTHR) dst[i] = a.theta[a.net.b_off[l] + i];
            dst += a.net.dims[l + 1];
        }
    }
    if (q.w1_lds) {
        const f4v* src = reinterpret_cast<const f4v*>(w1g + (ENV == ENV_MAZE ? (size_t)n_cells * H1 : 0));
        f4v* dst = reinterpret_cast<f4v*>(w1s);
        const int n4 = (ENV == ENV_MAZE ? n_cells : D) * H1 / 4;
        for (int i0 = 0; i0 < n4; i0 += 4 * WTHR) {
            f4v v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int i = i0 + u * WTHR + tid; v[u] = src[i < n4 ? i : 0]; }
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int i = i0 + u * WTHR + tid; if (i < n4) { round4<BF>(v[u]); dst[i] = v[u]; } }
        }
        if (ENV == ENV_MAZE)
            for (int i = tid; i < H1; i += WTHR) w1s[(size_t)n_cells * H1 + i] = round1<BF>(w1g[(size_t)(3 * n_cells - 1) * H1 + i]);
    }
    if (ENV == ENV_MAZE) {
        for (int i = tid; i < TM * 8; i += WTHR) obs[(i >> 3) * OBS_WORDS + (i & 7)] = tp.walls[(size_t)(i & 7) * B + b0 + (i >> 3)];
        __syncthreads();
        maze_prefix<BF, WTHR>(a, TM, obs, w1g, b1s, pre, tid);
    }
    // the draws of step t for all environments of the workgroup: the action's two words (pendulum: noise), the reset's
    auto draw = [&](int t, int lane) __attribute__((always_inline)) {
        if (lane >= 2 * TM) return;
        const int m = lane & (TM - 1);
        const bool reset = lane >= TM;
        const u32x4 v = philox(a.seed, (uint32_t)(b0 + m), a.gstep + (uint64_t)t, reset ? DOM_RESET : DOM_ACTION);
        const uint32_t v0 = (ENV == ENV_PENDULUM && !reset) ? bits_from_f(gaussian_noise(v.x, v.y)) : v.x;
        *reinterpret_cast<uint2*>(rng + ((t & 1) * TM + m) * 4 + (reset ? 2 : 0)) = make_uint2(v0, v.y);
    };
    if (wave == WW - 1) draw(0, lane0);

    // ---- weights: this wavefront's chunks in registers and in LDS ----
    const __amdgpu_buffer_rsrc_t theta = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.theta), 0, (uint32_t)a.net.P * 4u, 0x00020000);
    const int jobs = q.p.jobs[wave];
    float wreg[PC][16];
    {
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) {
            const WideJob& d = q.p.job[wave][j];                   // (zero where there is none)
            const uint32_t off = d.off + (uint32_t)(16 * (d.n_stream + d.n_lds)) * d.n4;
#pragma unroll
            for (int i = 0; i < SC; ++i) {
#pragma unroll
                for (int kk = 0; kk < 16; ++kk) wreg[SC * j + i][kk] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(theta, 4 * lane0, off + (uint32_t)(16 * i + kk) * d.n4, 0));
#pragma unroll
                for (int kk = 0; kk < 16; kk += 2) round2<BF>(wreg[SC * j + i][kk], wreg[SC * j + i][kk + 1]);
            }
        }
        f4v* dst = reinterpret_cast<f4v*>(smem + q.o_w) + wave * q.p.lds * 256 + lane0;   // chunk: [4][64 lanes][4 inputs]
        for (int job = 0; job < jobs; ++job) {
            const WideJob& d = q.p.job[wave][job];
            for (int c = 0; c < d.n_lds; ++c, dst += 256) {
                const uint32_t o = d.off + (uint32_t)(16 * (d.n_stream + c)) * d.n4;
                f4v v[4];
#pragma unroll
                for (int kk = 0; kk < 16; ++kk) v[kk / 4][kk % 4] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(theta, 4 * lane0, o + (uint32_t)kk * d.n4, 0));
#pragma unroll
                for (int u = 0; u < 4; ++u) { round4<BF>(v[u]); dst[64 * u] = v[u]; }
            }
        }
    }
    __syncthreads();
    // ---- the streamed ones: a cursor over them, the same sequence every step, two chunks on their way or waiting ----
    int cjob = 0, cleft = 0;                                       // job of the next chunk to ask for, how many are left of it
    uint32_t coff = 0, cn4 = 0;
    auto advance = [&]() __attribute__((always_inline)) {
        --cleft; coff += 16u * cn4;
        if (cleft == 0) {
            do { cjob = cjob + 1 < jobs ? cjob + 1 : 0; } while (q.p.job[wave][cjob].n_stream == 0);
            cleft = q.p.job[wave][cjob].n_stream; coff = q.p.job[wave][cjob].off; cn4 = q.p.job[wave][cjob].n4;
        }
    };
    float ring[2][16];
    auto ask = [&](float& w, int kk) __attribute__((always_inline)) {
        w = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(theta, 4 * lane0, coff + (uint32_t)kk * cn4, 0));
    };
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) ring[c][kk] = 0.0f;
    if (q.p.streamed[wave]) {
        while (q.p.job[wave][cjob].n_stream == 0) ++cjob;
        cleft = q.p.job[wave][cjob].n_stream; coff = q.p.job[wave][cjob].off; cn4 = q.p.job[wave][cjob].n4;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) ask(ring[c][kk], kk);
            advance();
        }
    }

    const bool owner = wave < R;
    // ==== environments: row r of 16 lanes is environment r of the wavefront's four ==================
    const int grp = owner ? wave : 0, row0 = 4 * grp;              // (the others stand in the state of the first four)
    EnvState st{0u, 0.0f, 0.0f};
    st.s0 = tp.s0[b0 + row0 + (lane0 >> 4)];
    if (ENV == ENV_PENDULUM) { st.f0 = tp.f0[b0 + row0 + (lane0 >> 4)]; st.f1 = tp.f1[b0 + row0 + (lane0 >> 4)]; }
    const float hbias = a.theta[a.net.bh_off + ((lane0 & 15) < NH ? lane0 & 15 : 0)];
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0): inside the loop a wait for a load would be one for every older store

    const int lg1 = 31 - __builtin_clz((uint32_t)H1);
    float sine = 0.0f, hv = 0.0f, rew = 0.0f, actf = 0.0f, eps = 0.0f;
    int act = 0, done = 0;
    // what the first layer reads of an environment, left in LDS by its owner: Catch its two cells, pendulum its features, maze its cell
    float* seen = smem + q.o_seen;                                 // [TM][4]
    float* rec = seen + 4 * TM;                                    // [2][TM][16]: what its owner leaves for the records
    auto observe = [&](int t, int lane) __attribute__((always_inline)) {
        uint32_t* o = reinterpret_cast<uint32_t*>(seen) + 4 * (row0 + (lane >> 4));
        uint32_t v0 = st.s0 & 0xffffu, v1 = 0, v2 = 0;
        if (ENV == ENV_CATCH) {
            int bc, pc;
            catch_obs_cells(a.env, st.s0, bc, pc);
            v0 = (uint32_t)bc; v1 = (uint32_t)pc;
        } else if (ENV == ENV_PENDULUM) {
            float cs;
            det_sincos(st.f0, sine, cs);
            v0 = bits_from_f(round1<BF>(cs)); v1 = bits_from_f(round1<BF>(sine)); v2 = bits_from_f(round1<BF>(st.f1));
        }
        if ((lane & 15) == 0) *reinterpret_cast<uint4*>(o) = make_uint4(v0, v1, v2, 0u);
        // the state as observed, and what the step before did: one word per lane of the row
        uint32_t w = bits_from_f(hv);                              // lanes 0..NH-1: the heads
        const int i = lane & 15;
        if (i == 8) w = st.s0;
        if (i == 9) w = ENV == ENV_PENDULUM ? bits_from_f(eps) : (uint32_t)act;
        if (i == 10) w = bits_from_f(rew);
        if (i == 11) w = (uint32_t)done;
        if (ENV == ENV_PENDULUM) {
            if (i == 12) w = bits_from_f(st.f0);
            if (i == 13) w = bits_from_f(st.f1);
            if (i == 14) w = bits_from_f(actf);
        }
        reinterpret_cast<uint32_t*>(rec)[16 * ((t & 1) * TM + row0 + (lane >> 4)) + i] = w;
    };
    // first layer: everybody takes four columns of an environment at a time
    auto first = [&](int lane) __attribute__((always_inline)) {
        float* x1 = smem + q.xo[0];
#pragma unroll 1
        for (int i0 = 64 * wave + lane; i0 < (R << lg1); i0 += 2 * 64 * WW) {
            // two at a time (the second one again the first where there is no other): all loads, then all stores
            f4v v[2], p[2], u[2], y[2];
            float* out[2];
            uint4 o[2];
            auto row_of = [&](int i) __attribute__((always_inline)) { return 4 * (i >> lg1) + (i & 3); };   // environment
            auto col_of = [&](int i) __attribute__((always_inline)) { return (i & (H1 - 1)) & ~3; };        // its columns c .. c + 3
            const int i1 = i0 + 64 * WW < (R << lg1) ? i0 + 64 * WW : i0;
            const int row[2] = {row_of(i0), row_of(i1)}, c[2] = {col_of(i0), col_of(i1)};
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                o[z] = *reinterpret_cast<const uint4*>(seen + 4 * row[z]);
                out[z] = x1 + (row[z] >> 2) * 4 * H1 + 4 * c[z] + (row[z] & 3);
            }
            // (two separate sets of loads: a pointer that may be either would make flat loads)
            if (ENV == ENV_PENDULUM) {
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    v[z] = *reinterpret_cast<const f4v*>(b1s + c[z]);
                    p[z] = *reinterpret_cast<const f4v*>(w1s + c[z]); u[z] = *reinterpret_cast<const f4v*>(w1s + H1 + c[z]); y[z] = *reinterpret_cast<const f4v*>(w1s + 2 * H1 + c[z]);
                }
#pragma unroll
                for (int z = 0; z < 2; ++z)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[z][e] = fmaf(f_from_bits(o[z].z), y[z][e], fmaf(f_from_bits(o[z].y), u[z][e], fmaf(f_from_bits(o[z].x), p[z][e], v[z][e])));
            } else {
#pragma unroll
                for (int z = 0; z < 2; ++z) v[z] = *reinterpret_cast<const f4v*>((ENV == ENV_MAZE ? pre + (row[z] << lg1) : b1s) + c[z]);
                if (q.w1_lds) {
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        p[z] = *reinterpret_cast<const f4v*>(w1s + (o[z].x << lg1) + c[z]);
                        u[z] = *reinterpret_cast<const f4v*>(w1s + ((ENV == ENV_MAZE ? (uint32_t)n_cells : o[z].y) << lg1) + c[z]);
                    }
                } else {
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        p[z] = *reinterpret_cast<const f4v*>(w1g + ((size_t)(ENV == ENV_MAZE ? n_cells + o[z].x : o[z].x) << lg1) + c[z]);
                        u[z] = *reinterpret_cast<const f4v*>(w1g + ((size_t)(ENV == ENV_MAZE ? (uint32_t)(3 * n_cells - 1) : o[z].y) << lg1) + c[z]);
                    }
#pragma unroll
                    for (int z = 0; z < 2; ++z) { round4<BF>(p[z]); round4<BF>(u[z]); }
                }
#pragma unroll
                for (int z = 0; z < 2; ++z) { v[z] += p[z]; v[z] += u[z]; }
            }
#pragma unroll
            for (int z = 0; z < 2; ++z) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[z][e] = v[z][e] > 0.0f ? v[z][e] : 0.0f;
                round4<BF>(v[z]);
#pragma unroll
                for (int e = 0; e < 4; ++e) out[z][4 * e] = v[z][e];
            }
        }
    };
    if (owner) observe(0, lane0);
    __syncthreads();
    first(lane0);

    // What the owners left before step t: its state, and what was done in step t - 1.  (They leave the next one in the other half.)
    auto records = [&](int t, int lane) __attribute__((always_inline)) {
        kernarg_w k = (kernarg_w)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(k));
        const uint32_t* r = reinterpret_cast<const uint32_t*>(rec);
        if (lane < TM) {
            const size_t tb = (size_t)t * B + b0 + lane;
            r += 16 * ((t & 1) * TM + lane);
            k->r.tp.tr_s0[tb] = r[8];
            if (ENV == ENV_PENDULUM) { k->r.tp.tr_f0[tb] = f_from_bits(r[12]); k->r.tp.tr_f1[tb] = f_from_bits(r[13]); }
            if (t > 0) {
                const size_t tq = tb - B;
                if (ENV == ENV_PENDULUM) { k->r.tp.tr_eps[tq] = f_from_bits(r[9]); k->r.tp.tr_actf[tq] = f_from_bits(r[14]); }
                else k->r.tp.tr_act[tq] = (uint8_t)r[9];
                k->r.tp.tr_rew[tq] = f_from_bits(r[10]);
                k->r.tp.tr_done[tq] = (uint8_t)r[11];
                k->r.tp.tr_val[tq] = f_from_bits(r[NH - 1]);
#pragma unroll
                for (int j = 0; j < NHP; ++j) k->r.tp.tr_head[tq * NHP + j] = j < NH ? f_from_bits(r[j]) : 0.0f;
            }
        }
    };
    // Barriers of a step: one when the first layer's outputs are there, one behind every stage, one when its owners have
    // stepped the environments.
    for (int t = 0; t <= T; ++t) {
        // everything derived from the lane is worked out again from a value the compiler cannot see through: loop-invariant
        // addresses would otherwise be kept in registers, on top of the weights, and spilled
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        kernarg_w k = (kernarg_w)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(k));
        __syncthreads();
        int passed = 1;
        // ---- the hidden layers ----
        {
            int li = q.o_w + wave * q.p.lds * 1024;                // next chunk in LDS
#pragma unroll
            for (int j = 0; j < SLOTS; ++j) {
                if (j >= jobs) break;
                const auto& d = k->p.job[wave][j];
                const int stage = d.stage, n_stream = d.n_stream, n_lds = d.n_lds, n_reg = d.n_reg, gs = d.gs, ygs = d.ygs;
                int xi = d.x + lane;
                int yi = d.y + 4 * lane, bi = d.bias + lane;
                asm volatile("" : "+v"(xi), "+v"(yi), "+v"(bi));   // worked out here, not behind the barrier
                __builtin_amdgcn_sched_barrier(0);
                while (passed < stage) { __syncthreads(); ++passed; }
                f4v acc[R];
                float x[2][R];                                     // inputs of this chunk and the next one
                auto read_x = [&](float (&n)[R]) __attribute__((always_inline)) {   // (past the last one: what follows in LDS, not used)
                    xi += 64;
#pragma unroll
                    for (int g = 0; g < R; ++g) n[g] = smem[xi + g * gs];
                    __builtin_amdgcn_sched_barrier(0);
                };
#pragma unroll
                for (int g = 0; g < R; ++g) x[0][g] = smem[xi + g * gs];
                if (d.first) {
                    const float b = smem[bi];
#pragma unroll
                    for (int g = 0; g < R; ++g) acc[g] = f4v{b, b, b, b};
                } else {
#pragma unroll
                    for (int g = 0; g < R; ++g) acc[g] = *reinterpret_cast<const f4v*>(smem + yi + g * ygs);
                }
#pragma unroll 1
                for (int c0 = 0; c0 < n_stream; c0 += 2) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        read_x(x[c ^ 1]);
                        if (BF) {
#pragma unroll
                            for (int kk = 0; kk < 16; kk += 2) round2<BF>(ring[c][kk], ring[c][kk + 1]);
                        }
                        quad_mfma<R, 0>(x[c], ring[c], acc, [&](int kk) __attribute__((always_inline)) { ask(ring[c][kk], kk); });
                        advance();
                    }
                }
                if (n_lds) {
                    float w[16];
                    auto fetch = [&](int u) __attribute__((always_inline)) {
                        const f4v v = *reinterpret_cast<const f4v*>(smem + li + 256 * u + 4 * lane);
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[4 * u + e] = v[e];
                    };
#pragma unroll
                    for (int u = 0; u < 4; ++u) fetch(u);
#pragma unroll 1
                    for (int c = 0; c < n_lds; ++c) {
                        read_x(x[1]);
                        li += 1024;                                // (behind the last chunk: what follows in LDS, not used)
                        quad_mfma<R, 0>(x[0], w, acc, [&](int kk) __attribute__((always_inline)) { if (kk % 4 == 3) fetch(kk / 4); });
#pragma unroll
                        for (int g = 0; g < R; ++g) x[0][g] = x[1][g];
                    }
                }
#pragma unroll
                for (int i = 0; i < SC; ++i) {
                    if (i < n_reg) {
                        read_x(x[(i & 1) ^ 1]);
                        quad_mfma<R, 0>(x[i & 1], wreg[SC * j + i], acc, [](int) __attribute__((always_inline)) {});
                    }
                }
#pragma unroll
                for (int g = 0; g < R; ++g) {
                    if (d.relu) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[g][e] = acc[g][e] > 0.0f ? acc[g][e] : 0.0f;
                        round4<BF>(acc[g]);
                    }
                    *reinterpret_cast<f4v*>(smem + yi + g * ygs) = acc[g];
                }
            }
            asm volatile("" : "+v"(lane));
        }
        int xi = q.xo[L - 1] + 4 * grp * HL + 4 * (lane & 15) + (lane >> 4), di = ((t & 1) * TM + row0 + (lane >> 4)) * 4;
        asm volatile("" : "+v"(xi), "+v"(di));                     // worked out here, not behind the barriers
        __builtin_amdgcn_sched_barrier(0);
        while (passed < q.p.barriers) { __syncthreads(); ++passed; }
        if (owner) {
            // ---- heads: row r of lanes, lane j of it head j ----
            hv = hbias;
            const uint4 dr = *reinterpret_cast<const uint4*>(rng + di);
            const f4v* wr = reinterpret_cast<const f4v*>(whs + ((lane & 15) < NH ? lane & 15 : 0) * ldw);
            f4v wa[4], wb[4];
            float xa = smem[xi], xb;
#pragma unroll
            for (int u = 0; u < 4; ++u) wa[u] = wr[u];
#pragma unroll 1
            for (int k0 = 0; k0 < HL; k0 += 32) {
                xb = smem[xi + 4 * (k0 + 16)];
#pragma unroll
                for (int u = 0; u < 4; ++u) wb[u] = wr[k0 / 4 + 4 + u];
                __builtin_amdgcn_sched_barrier(0);
                chain16(xa, wa[0], wa[1], wa[2], wa[3], hv);
                const int kn = k0 + 32 < HL ? k0 + 32 : 0;
                xa = smem[xi + 4 * kn];
#pragma unroll
                for (int u = 0; u < 4; ++u) wa[u] = wr[kn / 4 + u];
                __builtin_amdgcn_sched_barrier(0);
                chain16(xb, wb[0], wb[1], wb[2], wb[3], hv);
            }
            if (t == T) break;
            row_step<ENV>(a.env, st, sine, hv, dr, obs + (row0 + (lane >> 4)) * OBS_WORDS, eps, actf, act, rew, done);
            asm volatile("" : "+v"(lane));
            observe(t + 1, lane);
        } else {
            // ---- meanwhile: the next draws, the activations' records ----
            if (t == T) break;
            if (wave == WW - 1) { draw(t + 1, lane); records(t, lane); }
            if (a.keep_acts)
                for (int l = 0; l < L; ++l) {
                    const int N = k->r.net.dims[l + 1], lg = 31 - __builtin_clz((uint32_t)N);
                    float* dst = k->r.tp.act[l] + ((size_t)t * B + b0) * N;
                    const float* src = smem + k->xo[l];
#pragma unroll 2
                    for (int i = 64 * (wave - R) + lane; i < (R << lg); i += 64 * (WW - R)) {
                        const int e = i & 3, c = (i & (N - 1)) >> 2, g = i >> lg;   // environment of its group, four columns, group
                        const float* s = src + 4 * g * N + 16 * c + e;
                        const f4v v = {s[0], s[4], s[8], s[12]};
                        *reinterpret_cast<f4v*>(dst + (size_t)(4 * g + e) * N + 4 * c) = v;
                    }
                }
        }
        __syncthreads();
        asm volatile("" : "+v"(lane));
        first(lane);
    }
    if (wave == WW - 1) records(T, lane0);
    if (!owner) return;
    const int i16 = lane0 & 15, b = b0 + row0 + (lane0 >> 4);
    const size_t tb = (size_t)T * B + b;
    if (i16 < NHP) tp.tr_head[tb * NHP + i16] = i16 < NH ? hv : 0.0f;
    if (i16 == NH - 1) tp.tr_val[tb] = hv;
    if (i16 == 0) {
        tp.s0[b] = st.s0;
        if (ENV == ENV_PENDULUM) { tp.f0[b] = st.f0; tp.f1[b] = st.f1; }
    }
}

// LDS of a workgroup (offsets in floats), and the plan: what is left of it takes weights first, then the first layer's rows
static bool wide_plan(const NetShape& net, const EnvDims& env, int R, WideArgs& q)
{
    const int H1 = net.dims[1], HL = net.dims[net.L], cells = env.rows * env.cols, TM = 4 * R, room = 160 * 256;
    int off = 0;
    for (int l = 0; l < net.L; ++l) { q.xo[l] = off; off += TM * net.dims[l + 1]; }
    q.o_wh = off; off += net.NH * (HL + 4);
    q.o_b1 = off; off += H1;
    q.o_bias = off;
    for (int l = 1; l < net.L; ++l) off += net.dims[l + 1];
    q.o_rng = off; off += 2 * TM * 4;
    q.o_seen = off; off += TM * 36;
    q.o_obs = off; off += env.kind == ENV_MAZE ? TM * OBS_WORDS : 0;
    q.o_pre = off; off += env.kind == ENV_MAZE ? TM * H1 : 0;
    const int w1 = (env.kind == ENV_MAZE ? cells + 1 : net.dims[0]) * H1, must = env.kind == ENV_PENDULUM ? w1 : 0;
    off += 64;                                                     // operand reads run a little past the end of an array
    if (off + must > room) return false;
    // jobs: a layer's outputs 64 at a time; where there are fewer than eight of those, the inputs are cut as well, a stage each
    WidePlan& p = q.p;
    memset(&p, 0, sizeof p);
    int stage = 1, bias = q.o_bias, total[WW] = {0};
    for (int l = 1; l < net.L; ++l) {
        const int K = net.dims[l], N = net.dims[l + 1], nb = N / 64;
        int cuts = 1;
        while (nb * cuts * 2 <= WW && K / (cuts * 2) >= 32) cuts *= 2;
        for (int w = 0; w < WW; ++w)
            for (int blk = w; blk < nb * cuts; blk += WW) {
                if (p.jobs[w] == WidePlan::MAX_JOBS) return false;
                WideJob& d = p.job[w][p.jobs[w]++];
                const int cut = blk / nb, c0 = 64 * (blk % nb), k0 = K / cuts * cut;
                d.stage = stage + cut; d.first = cut == 0; d.relu = cut == cuts - 1;
                d.off = 4u * (uint32_t)(net.w_off[l] + k0 * N + c0); d.n4 = 4u * (uint32_t)N;
                d.x = q.xo[l - 1] + 4 * k0; d.gs = 4 * K;
                d.y = q.xo[l] + 4 * c0; d.ygs = 4 * N; d.bias = bias + c0;
                d.n_stream = K / cuts / 16;                        // (chunks of the job, for now)
                total[w] += d.n_stream;
            }
        stage += cuts;
        bias += N;
    }
    p.barriers = stage;
    off += 1024;                                                   // and so does a prefetch behind the last chunk
    if (off + must > room) return false;
    p.lds = (room - off - must) / (1024 * WW);
    p.slots = 1;
    for (int w = 0; w < WW; ++w) if (p.jobs[w] > p.slots) p.slots = p.jobs[w];
    const int slot = wide_slot(p.slots);
    for (int w = 0; w < WW; ++w) {
        int lds = p.lds, want = 0;                                 // what the registers do not hold
        for (int j = 0; j < p.jobs[w]; ++j) { const int n = p.job[w][j].n_stream; want += n > slot ? n - slot : 0; }
        for (int j = 0; j < p.jobs[w]; ++j) {
            WideJob& d = p.job[w][j];
            const int n = d.n_stream, rest = n > slot ? n - slot : 0;
            int r = n - rest, m = want <= lds ? rest : lds * rest / want;
            if ((rest - m) & 1) { if (m > 0) --m; else --r; }      // pairs are streamed
            d.n_reg = r; d.n_lds = m; d.n_stream = n - r - m;
            p.streamed[w] += d.n_stream;
            want -= rest; lds -= m;
        }
    }
    int most = 0;                                                  // chunks in LDS that are really used
    for (int w = 0; w < WW; ++w) { int m = 0; for (int j = 0; j < p.jobs[w]; ++j) m += p.job[w][j].n_lds; if (m > most) most = m; }
    p.lds = most;
    q.o_w = off - 1024; off += most * 1024 * WW;
    q.o_w1 = off;
    q.w1_lds = off + w1 <= room ? 1 : 0;
    if (q.w1_lds) off += w1;
    else if (must) return false;
    p.lds_bytes = (uint32_t)off * 4u;
    return true;
}

// Where both this kernel and the pinned one can have a net, groups of four are faster under a top layer of 256 units, which all
// wavefronts share here and four of them there (T = 16, Catch / pendulum / 8 x 8 and 16 x 16 maze, pinned and here: 128-256, 1008
// environments 76.5 and 64.2 us / 82.7 and 66.2 / 81.8 and 68.9 / 87.1 and 73.0; 64-128-256 90.1 and 77.1 / 97.3 and 81.1; 128-128-256
// 99.2 and 92.4 / 106.4 and 96.2; 64-256 59.7 and 56.8 / 67.0 and 59.4), not under two of 64 (64-64-256 70.1 and 71.2 on Catch); pairs of
// groups only where the net has no other layer of 128 (2032 environments, 128-256 77.6 and 74.3 / 83.2 and 77.8, but 64-128-256
// 90.3 and 90.2, 128-128-256 99.7 and 110.9, 64-256 60.7 and 65.0).
bool wide_before_pinned(const NetShape& net, int B)
{
    if (net.L > 3 || net.dims[net.L] != 256) return false;
    const int below = net.dims[net.L - 1];
    if (net.L == 2) return B <= 1024 || below == 128;
    return B <= 1024 && below == 128;
}

// Which nets: two or more layers that rollout_pinned.hip does not take (or only behind this kernel, above), in whole blocks of 64, not two equal ones of 64 or 128
// (1024 environments, resident and here: 128-128 Catch 49 and 66 us, pendulum 51 and 68, maze of 12 x 14 65 and 73; 64-64 29 and
// 45, 36 and 49, 38 and 51).  Up to 1024 environments in groups of four, up to 2048 in pairs of groups; the pairs not where a
// layer's outputs leave most SIMDs idle (2032 environments on Catch, the pendulum and the maze, streamed and here: 512-128
// 134 and 135 us, 139 and 140, 152 and 150; 64-512-64 158 and 167, 164 and 193, 169 and 175; 512-64-512 190 and 194, 197 and
// 199, 212 and 213; but 256-128-256 140 and 131, 147 and 141, 157 and 146, 512-256 207 and 172, 211 and 168, 226 and 185) --
// unless the streaming kernel's buffers do not fit LDS and the vector-ALU kernel would run (maze of 12 x 14, 1024-128: 3190
// and 298).
int rollout_wide_groups(const NetShape& net, const EnvDims& env, int B)
{
    if (net.L < 2 || B > 2048) return 0;
    const int R = B <= 1024 ? 1 : 2, res = rollout_resident_tile(net, env.kind, B);
    if (res && net.dims[1] != 256) return 0;
    for (int l = 1; l <= net.L; ++l) if (net.dims[l] % 64) return 0;
    if (R == 2 && rollout_pick_tile_mfma(net, env, B) > 0)
        for (int l = 1; l < net.L; ++l) if (net.dims[l + 1] == 64 || (net.dims[l + 1] == 128 && net.dims[l] > 256)) return 0;
    WideArgs q;
    return wide_plan(net, env, R, q) ? R : 0;
}

template <int ENV, int R, int SLOTS>
static hipError_t launch_wide_slots(anakin* h, const WideArgs& q)
{
    auto kern = h->net.bf16 ? rollout_wide_kernel<ENV, R, SLOTS, true> : rollout_wide_kernel<ENV, R, SLOTS, false>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)q.p.lds_bytes);
    if (e != hipSuccess) return e;
    ProfScope prof(h, "rollout");
    hipLaunchKernelGGL(kern, dim3(h->B / (4 * R)), dim3(WTHR), q.p.lds_bytes, h->stream, q);
    return hipGetLastError();
}

template <int ENV>
static hipError_t launch_wide_env(anakin* h, const WideArgs& q)
{
    if (h->wide == 1) return q.p.slots == 1 ? launch_wide_slots<ENV, 1, 1>(h, q) : q.p.slots == 2 ? launch_wide_slots<ENV, 1, 2>(h, q) : launch_wide_slots<ENV, 1, 3>(h, q);
    return q.p.slots == 1 ? launch_wide_slots<ENV, 2, 1>(h, q) : q.p.slots == 2 ? launch_wide_slots<ENV, 2, 2>(h, q) : launch_wide_slots<ENV, 2, 3>(h, q);
}

hipError_t launch_wide(anakin* h, const RolloutArgs& args)
{
    WideArgs q;
    q.r = args;
    if (!wide_plan(h->net, h->env, h->wide, q)) return hipErrorInvalidValue;
    switch (h->env.kind) {
        case ENV_CATCH:    return launch_wide_env<ENV_CATCH>(h, q);
        case ENV_PENDULUM: return launch_wide_env<ENV_PENDULUM>(h, q);
        default:           return launch_wide_env<ENV_MAZE>(h, q);
    }
}

}  // namespace ank
