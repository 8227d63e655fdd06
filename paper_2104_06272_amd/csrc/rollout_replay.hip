// The learner's forward pass over a stored unroll (decoupled steps, sequential updates) for nets of two equal layers of 128
// or 256 units on boards of Catch and the pendulum: the hidden matrix stays in the register file, as in the resident acting
// kernel, but nothing ties the samples to an order, so a workgroup takes 32 to 64 of them at a time and the phases that
// cannot overlap the matrix layer (first layer, head chains, barriers: 5 k cycles) are paid once for that many instead of
// once for 16.  Bound by the fp32 matrix instruction: 8.2 k cycles for each 16 samples of 256-256.
// Accumulation is in the canonical order; records are what the acting kernels leave.  Beside the actor of a decoupled step,
// against the streaming kernel: 256-256, 270336 samples 408 -> 338 us (the step 1045 -> 978), 86016 samples 149 -> 121 (but the
// step 412 -> 403 at most: the loss launch behind the replay then waits for the actor's workgroups, 60 -> 121); 128-128 (two
// workgroups per compute unit), 253952 samples 152 -> 109 (418 -> 372), 34816 samples 36 -> 23 (106 -> 95).
#include "acting.h"

namespace ank {

constexpr int RPT = 512;                                           // threads: eight wavefronts, as many column blocks

template <int ENV, int RW, int G>
__global__ __launch_bounds__(RPT) void replay_resident_kernel(const RolloutArgs a, const int samples, const int tiles, const int w1_lds)
{
    constexpr int NH = ENV == ENV_CATCH ? 4 : 3, NHP = 4, TM = 16 * G, KS = RW / 4, NT = RW / 128, LDX = RW + 4, IT = TM * RW / 4 / RPT;
    extern __shared__ float4 smem4[];
    float* X = reinterpret_cast<float*>(smem4);                    // [TM][LDX] first layer's outputs, then the second's
    float* whs = X + TM * LDX;                                     // [4][LDX] head weights, transposed
    float* b1s = whs + 4 * LDX;                                    // [RW]
    float* seen = b1s + RW;                                        // [TM][4]: Catch: two cells; pendulum: features
    float* w1s = seen + TM * 4;                                    // [D][RW] first-layer rows
    const TrajPtrs& tp = a.tp;
    const float* w1g = a.theta + a.net.w_off[0];
    const int tid = threadIdx.x, lane0 = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kept = a.T * a.B;                                    // samples whose activations the update needs

    float wreg[KS][NT], bv[NT];
    {
        const int col0 = wave * 16 * NT + NT * (lane0 & 15), kq = lane0 >> 4;
#pragma unroll
        for (int n = 0; n < NT; ++n) bv[n] = a.theta[a.net.b_off[1] + col0 + n];
        const __amdgpu_buffer_rsrc_t theta = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.theta), 0, (uint32_t)a.net.P * 4u, 0x00020000);
        const uint32_t off = 4u * (uint32_t)(kq * RW + col0);
        typedef uint32_t u2v __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const uint32_t row = 4u * (uint32_t)(a.net.w_off[1] + 4 * s * RW);
            if (NT == 2) {
                const u2v v = __builtin_amdgcn_raw_buffer_load_b64(theta, off, row, 0);
                wreg[s][0] = f_from_bits(v[0]); wreg[s][NT - 1] = f_from_bits(v[1]);
            } else wreg[s][0] = f_from_bits(__builtin_amdgcn_raw_buffer_load_b32(theta, off, row, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
        for (int i = tid; i < RW * NH; i += RPT) whs[(i % NH) * LDX + i / NH] = a.theta[a.net.wh_off + i];
        for (int i = tid; i < RW; i += RPT) b1s[i] = a.theta[a.net.b_off[0] + i];
        if (w1_lds) {
            const f4v* src = reinterpret_cast<const f4v*>(w1g);
            f4v* dst = reinterpret_cast<f4v*>(w1s);
            const int n4 = a.net.dims[0] * RW / 4;
            for (int i0 = 0; i0 < n4; i0 += 4 * RPT) {
                f4v v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { const int i = i0 + u * RPT + tid; v[u] = src[i < n4 ? i : 0]; }
#pragma unroll
                for (int u = 0; u < 4; ++u) { const int i = i0 + u * RPT + tid; if (i < n4) dst[i] = v[u]; }
            }
        }
    }
    const float hbias = a.theta[a.net.bh_off + ((lane0 >> 4) < NH ? lane0 >> 4 : 0)];
    // the states of a tile, asked for a tile ahead
    uint32_t s0 = 0;
    float f0 = 0.0f, f1 = 0.0f;
    auto ask = [&](int tile) {
        if (tid >= TM || tile >= tiles) return;
        int m = tile * TM + tid;
        m = m < samples ? m : samples - 1;
        s0 = tp.tr_s0[m];
        if (ENV == ENV_PENDULUM) { f0 = tp.tr_f0[m]; f1 = tp.tr_f1[m]; }
    };
    ask(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        // (from a value the compiler cannot see through: addresses kept across the loop would not fit beside the weights)
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        const int m0 = tile * TM;
        if (tid < TM) {
            float* o = seen + 4 * tid;
            if (ENV == ENV_CATCH) {
                int bc, pc;
                catch_obs_cells(a.env, s0, bc, pc);
                reinterpret_cast<uint32_t*>(o)[0] = (uint32_t)bc; reinterpret_cast<uint32_t*>(o)[1] = (uint32_t)pc;
            } else {
                float sn, cs;
                det_sincos(f0, sn, cs);
                o[0] = cs; o[1] = sn; o[2] = f1;
            }
        }
        __syncthreads();
        ask(tile + gridDim.x);                                     // (in front of the stores: a wait for it is none for them)
        // ---- first layer ----
        {
            const int c = (4 * lane) & (RW - 1), r0 = (64 * wave + lane) / (RW / 4);
            constexpr int STEP = RPT / (RW / 4);                   // rows between a thread's items
            const f4v b = *reinterpret_cast<const f4v*>(b1s + c);
            f4v w[3];
            if (ENV == ENV_PENDULUM) {
#pragma unroll
                for (int k = 0; k < 3; ++k) w[k] = *reinterpret_cast<const f4v*>(w1s + k * RW + c);
            }
            // all loads, then all stores (which might be the same memory, for all the compiler knows)
            f4v v[IT];
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const float* o = seen + 4 * (r0 + it * STEP);
                if (ENV == ENV_PENDULUM) {
                    v[it] = b;
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[it][q] = fmaf(o[k], w[k][q], v[it][q]);
                } else {
                    const int i0 = (int)reinterpret_cast<const uint32_t*>(o)[0], i1 = (int)reinterpret_cast<const uint32_t*>(o)[1];
                    f4v x0, x1;
                    if (w1_lds) { x0 = *reinterpret_cast<const f4v*>(w1s + i0 * RW + c); x1 = *reinterpret_cast<const f4v*>(w1s + i1 * RW + c); }
                    else { x0 = *reinterpret_cast<const f4v*>(w1g + i0 * RW + c); x1 = *reinterpret_cast<const f4v*>(w1g + i1 * RW + c); }
                    v[it] = (b + x0) + x1;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) v[it][q] = v[it][q] > 0.0f ? v[it][q] : 0.0f;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int row = r0 + it * STEP;
                *reinterpret_cast<f4v*>(X + row * LDX + c) = v[it];
                if (m0 + row < kept) *reinterpret_cast<f4v*>(tp.act[0] + (size_t)(m0 + row) * RW + c) = v[it];
            }
        }
        __syncthreads();
        asm volatile("" : "+v"(lane));
        // ---- the matrix layer ----
        const int col0 = wave * 16 * NT + NT * (lane & 15), kq = lane >> 4;
        f4v acc[G][NT];
        {
            const float* xp = X + (lane & 15) * LDX + kq;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[g][n] = f4v{bv[n], bv[n], bv[n], bv[n]};
            constexpr int PF = 4;                                  // LDS reads run this many steps ahead of their MFMAs
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
            }
        }
        __syncthreads();                                           // the first layer's outputs have been read
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * g + 4 * kq + r;
                float* y = X + row * LDX + col0;
                float* rec = tp.act[1] + (size_t)(m0 + row) * RW + col0;
                const bool keep = m0 + row < kept;
                float o[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) o[n] = acc[g][n][r] > 0.0f ? acc[g][n][r] : 0.0f;
                if (NT == 2) {
                    const float2 v = make_float2(o[0], o[NT - 1]);
                    *reinterpret_cast<float2*>(y) = v;
                    if (keep) *reinterpret_cast<float2*>(rec) = v;
                } else {
                    y[0] = o[0];
                    if (keep) rec[0] = o[0];
                }
            }
        __syncthreads();
        asm volatile("" : "+v"(lane));
        // ---- heads: lane e + 16 j sums head j of sample e of the wavefront's group ----
        if (wave < G) {
            const int e = lane & 15, j = lane >> 4, m = m0 + 16 * wave + e;
            const f4v* x = reinterpret_cast<const f4v*>(X + (16 * wave + e) * LDX);
            const f4v* w = reinterpret_cast<const f4v*>(whs + (j < NH ? j : 0) * LDX);
            // 16 inputs at a time, the next 16 on their way
            float hv = hbias;
            f4v xa[4], wa[4], xb[4], wb[4];
            auto get = [&](f4v (&xv)[4], f4v (&wv)[4], int k) {
#pragma unroll
                for (int u = 0; u < 4; ++u) { xv[u] = x[k / 4 + u]; wv[u] = w[k / 4 + u]; }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto sum = [&](const f4v (&xv)[4], const f4v (&wv)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) hv = fmaf(xv[u][q], wv[u][q], hv);
                __builtin_amdgcn_sched_barrier(0);
            };
            get(xa, wa, 0);
#pragma unroll 1
            for (int k0 = 0; k0 < RW; k0 += 32) {
                get(xb, wb, k0 + 16);
                sum(xa, wa);
                get(xa, wa, k0 + 32 < RW ? k0 + 32 : 0);
                sum(xb, wb);
            }
            if (m < samples) {
                tp.tr_head[(size_t)m * NHP + j] = j < NH ? hv : 0.0f;
                if (j == NH - 1) tp.tr_val[m] = hv;
            }
        }
    }
}

static size_t replay_lds(const NetShape& net, int G, bool w1)
{
    const size_t w = net.dims[1], tm = 16 * (size_t)G;
    return (tm * (w + 4) + 4 * (w + 4) + w + tm * 4 + (w1 ? (size_t)net.dims[0] * w : 0)) * 4;
}

template <int ENV, int RW, int G>
static hipError_t launch_replay_g(anakin* h, const RolloutArgs& a, int samples)
{
    const bool w1 = replay_lds(h->net, G, true) <= 160 * 1024;
    const size_t lds = replay_lds(h->net, G, w1);
    const int tiles = (samples + 16 * G - 1) / (16 * G);
    auto kern = replay_resident_kernel<ENV, RW, G>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(h, "replay_forward");
    hipLaunchKernelGGL(kern, dim3(tiles < 65536 / RW ? tiles : 65536 / RW), dim3(RPT), lds, h->stream, a, samples, tiles, w1 ? 1 : 0);
    return hipGetLastError();
}

// From 4096 samples: a tile for every other compute unit (below, the streaming kernel cut along time is as fast: 4096 samples
// 15 -> 12 us for 128-128, 22 and 23 for 256-256).
bool replay_resident_ok(const anakin* h, int samples)
{
    const int w = rollout_resident_width(h->net);
    return (w == 128 || w == 256) && h->env.kind != ENV_MAZE && samples >= 4096 && !(h->mode & (ANAKIN_MODE_CANONICAL_ACTING | ANAKIN_MODE_STREAM_WEIGHTS));
}

hipError_t launch_replay_resident(anakin* h, const RolloutArgs& a, int samples)
{
    // Groups of 16 per tile: the number with the smallest cost for a compute unit.  A tile of G groups has G times a group's
    // matrix time (in 100 cycles: 82 for 256-256, 41 for 128-128), which the workgroups of a unit (one; two of 128-128) share,
    // and 50 or 40 that they do not wait for one another in: first layer, head chains, barriers.  Within 2 % of the best G for
    // 23 sample counts of 4608 to 524288, Catch and pendulum, both widths; counted as if two workgroups did not share the
    // matrix unit, 128-128 took G = 2 with 9216 samples (16.3 us; 3 now, 14.6), 2 with 12288 (17.3; 15.6) and 4 with 86016
    // (47.5; 3 now, 42.1).  256-256, G = 2, 3, 4: 12288 samples 31.9, 26.5, 30.5 us; 32768 53.4, 56.7, 51.4; 86016 128, 121, 132.
    const int w = rollout_resident_width(h->net);
    int best = 2;
    long cost = 0;
    for (int G = 2; G <= 4; ++G) {
        const long tiles = (samples + 16 * G - 1) / (16 * G), wgs = 65536 / w, per_unit = (tiles + 255) / 256, per_wg = (tiles + wgs - 1) / wgs;
        const long c = w == 256 ? per_unit * 82 * G + per_wg * 50 : per_unit * 41 * G + per_wg * 40;
        if (!cost || c <= cost) { best = G; cost = c; }
    }
    if (h->env.kind == ENV_CATCH) {
        if (w == 256) return best == 2 ? launch_replay_g<ENV_CATCH, 256, 2>(h, a, samples) : best == 3 ? launch_replay_g<ENV_CATCH, 256, 3>(h, a, samples) : launch_replay_g<ENV_CATCH, 256, 4>(h, a, samples);
        return best == 2 ? launch_replay_g<ENV_CATCH, 128, 2>(h, a, samples) : best == 3 ? launch_replay_g<ENV_CATCH, 128, 3>(h, a, samples) : launch_replay_g<ENV_CATCH, 128, 4>(h, a, samples);
    }
    if (w == 256) return best == 2 ? launch_replay_g<ENV_PENDULUM, 256, 2>(h, a, samples) : best == 3 ? launch_replay_g<ENV_PENDULUM, 256, 3>(h, a, samples) : launch_replay_g<ENV_PENDULUM, 256, 4>(h, a, samples);
    return best == 2 ? launch_replay_g<ENV_PENDULUM, 128, 2>(h, a, samples) : best == 3 ? launch_replay_g<ENV_PENDULUM, 128, 3>(h, a, samples) : launch_replay_g<ENV_PENDULUM, 128, 4>(h, a, samples);
}

}  // namespace ank
