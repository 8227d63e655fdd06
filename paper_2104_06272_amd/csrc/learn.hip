// The update on a stored unroll (paper section 3.1: the parameter update that
// follows the T interactions and reuses the policy's forward pass):
//   returns_scan          reverse scan over t of the lambda-return recursion
//   head_grad             actor-critic loss terms and the gradient w.r.t. head outputs
//   scan_loss             the two above in one launch; for an unroll acted by older parameters (decoupled steps)
//                         with off-policy targets in place of the returns
//   vtrace_ratio / _scan  those targets where the unroll does not fit scan_loss
//   head_backward(_mfma)  gradient of the head matrix, and of the last hidden layer
//   first_layer_grad*     gradient of the pendulum's first layer from the compact state (boards: first_layer.hip)
//   learn_catch_fused     returns, loss and backward pass of a small one-hidden-layer Catch net
//   adam_reduce(_narrow, _flat)  fixed-order sum of split-K partials fused with Adam
// Hidden-layer GEMMs live in gemm.hip (vector ALU), gemm_mfma.hip (tiled) and
// gemm_split.hip (layers in whole 64-wide tiles, which also take over the head
// pass of such a top layer); the bf16 update in learn_bf16.hip; the reverse
// sweep of the pathwise policy gradient in pathwise.hip.
// No floating-point atomics anywhere: every reduction has a fixed order, so runs
// are reproducible bit for bit.
#include <type_traits>
#include "internal.h"
#include "loss.h"
#include "split_terms.h"

namespace ank {

// ---------------------------------------------------------------------------
// G_T = V(s_T);  G_t = r + disc ((1-lambda) V_{t+1} + lambda G_{t+1});  A_t = G_t - V_t
// with disc = 0 after an episode end, gamma otherwise.  One lane per env walks
// its column backwards; consecutive lanes touch consecutive addresses of the
// time-major arrays, so every load and store is fully coalesced.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void returns_scan(int B, int T, const float* __restrict__ rew,
                                                   const uint8_t* __restrict__ done, const float* __restrict__ val,
                                                   float gamma, float lambda, float* __restrict__ adv,
                                                   float* __restrict__ ret)
{
    const int b = blockIdx.x * WG + threadIdx.x;
    if (b >= B) return;
    const float oml = 1.0f - lambda;
    float G = val[(size_t)T * B + b];
    float vnext = G;
#pragma unroll 4
    for (int t = T - 1; t >= 0; --t) {
        const size_t i = (size_t)t * B + b;
        const float r = rew[i], v = val[i];
        const float disc = done[i] ? 0.0f : gamma;
        const float mix = fmaf(lambda, G, oml * vnext);
        G = fmaf(disc, mix, r);
        ret[i] = G;
        adv[i] = G - v;
        vnext = v;
    }
}

// ---------------------------------------------------------------------------
// Off-policy targets for a stored unroll whose actions came from older parameters (decoupled acting
// and learning, paper section 3.2; the correction is IMPALA's V-trace, which the paper runs on that
// architecture).  head_old: head outputs stored at acting time (the behaviour policy mu); head_new:
// the learner's forward pass over the same states (policy pi and values V).  Per env, backwards in t:
//   w = pi(a|s) / mu(a|s),  rho = min(1, w),  c = lambda min(1, w),  disc = gamma (1 - done)
//   adv_t = rho (r + disc v_{t+1} - V_t)
//   v_t - V_t = rho (r + disc V_{t+1} - V_t) + disc c (v_{t+1} - V_{t+1}),   v_T = V_T
// ret = v, adv = the policy-gradient advantage: the loss kernel then treats them as it treats the
// on-policy return and advantage.  Gaussian policy: the densities are compared at the stored
// pre-squash sample z = mu_old + sigma_old eps_old, and eps_new = (z - mu_new) / sigma_new is
// written for the loss kernel's score function.  The ratios need no order and take a pass of
// their own, one lane per sample; the recursion then walks each env's column as returns_scan does.
// ---------------------------------------------------------------------------
struct VtraceArgs {
    int B, T, A, NH, NHP, policy;
    const float* head_old; const float* head_new; const float* val_new; const uint8_t* act; const float* eps_old;
    const float* rew; const uint8_t* done;
    float gamma, lambda;
    float* adv; float* ret; float* eps_new;
};

__device__ __forceinline__ void load_head(const float* p, int NHP, float (&hv)[8])
{
    const float4 h0 = *reinterpret_cast<const float4*>(p);
    hv[0] = h0.x; hv[1] = h0.y; hv[2] = h0.z; hv[3] = h0.w;
    if (NHP == 8) {
        const float4 h1 = *reinterpret_cast<const float4*>(p + 4);
        hv[4] = h1.x; hv[5] = h1.y; hv[6] = h1.z; hv[7] = h1.w;
    } else { hv[4] = hv[5] = hv[6] = hv[7] = 0.0f; }
}

__device__ __forceinline__ float log_softmax_at(const float (&hv)[8], int A, int act)
{
    float mx = hv[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) if (j < A) mx = fmaxf(mx, hv[j]);
    float Z = 0.0f, ha = hv[0];
#pragma unroll
    for (int j = 0; j < 8; ++j) { if (j < A) Z += det_exp(hv[j] - mx); if (j == act) ha = hv[j]; }
    return ha - mx - det_log(Z);
}

// the noise that reproduces the stored pre-squash sample under newer head outputs: eps_new = (z - mu_new) / sigma_new
__device__ __forceinline__ float noise_now(const float* ho, float eo, float mu, float sigma)
{
    const float2 o = *reinterpret_cast<const float2*>(ho);
    const float z = fmaf(det_exp(fminf(fmaxf(o.y, -5.0f), 2.0f)), eo, o.x);       // the sampler's own expression
    return (z - mu) / sigma;
}

// the truncated ratio rho of sample i, and the noise (Gaussian) that reproduces its action under the new head outputs
__device__ __forceinline__ float vtrace_rho(const VtraceArgs& a, size_t i)
{
    float hn[8], ho[8];
    load_head(a.head_new + i * a.NHP, a.NHP, hn);
    load_head(a.head_old + i * a.NHP, a.NHP, ho);
    float lw;
    if (a.policy == POLICY_CATEGORICAL) {
        const int act = a.act[i];
        lw = log_softmax_at(hn, a.A, act) - log_softmax_at(ho, a.A, act);
    } else {
        const float lso = fminf(fmaxf(ho[1], -5.0f), 2.0f), lsn = fminf(fmaxf(hn[1], -5.0f), 2.0f);
        const float eo = a.eps_old[i];
        const float en = noise_now(a.head_old + i * a.NHP, eo, hn[0], det_exp(lsn));
        a.eps_new[i] = en;
        lw = (-0.5f * en * en - lsn) - (-0.5f * eo * eo - lso);
    }
    return fminf(1.0f, det_exp(lw));
}

// first pass, one lane per sample, no order: the truncated ratio (parked in ret, where the scan picks it up before it
// overwrites the slot with v) and eps_new
__global__ __launch_bounds__(WG) void vtrace_ratio(const VtraceArgs a)
{
    const size_t i = (size_t)blockIdx.x * WG + threadIdx.x;
    if (i < (size_t)a.B * a.T) a.ret[i] = vtrace_rho(a, i);
}

// second pass, one lane per env, backwards in t
__global__ __launch_bounds__(WG) void vtrace_scan(const VtraceArgs a)
{
    const int b = blockIdx.x * WG + threadIdx.x;
    if (b >= a.B) return;
    const int B = a.B, T = a.T;
    float Vnext = a.val_new[(size_t)T * B + b];
    float tail = 0.0f;                                       // v_{t+1} - V_{t+1}
#pragma unroll 4
    for (int t = T - 1; t >= 0; --t) {
        const size_t i = (size_t)t * B + b;
        const float rho = a.ret[i], V = a.val_new[i], r = a.rew[i];
        const float c = a.lambda * rho;
        const float disc = a.done[i] ? 0.0f : a.gamma;
        a.adv[i] = rho * (fmaf(disc, Vnext + tail, r) - V);
        tail = fmaf(disc * c, tail, rho * (fmaf(disc, Vnext, r) - V));
        a.ret[i] = V + tail;
        Vnext = V;
    }
}

// ---------------------------------------------------------------------------
// Per sample: l = -A log pi(a|s) + c_v (G - V)^2 - beta H, and d l / d head / M.
// Categorical: d/dlogit_i = -A (1[i=a] - p_i) + beta p_i (log p_i + H).
// Gaussian (score function at the stored noise, log_sigma clamped to [-5,2]):
// d/dmu = -A eps / sigma, d/dlog_sigma = -A (eps^2 - 1) - beta (0 when clamped).
// Also block sums of the loss terms, rewards and episode ends for the metrics.
// ---------------------------------------------------------------------------
struct HeadGradArgs {
    int M, A, NH, NHP, policy;
    const float* head; const uint8_t* act; const float* eps; const float* adv; const float* ret;
    const float* rew; const uint8_t* done;
    float* dhead; float* loss_part;        // [blocks][8]
    float beta, cv, inv_m;
    const float* head_old;                 // Gaussian, forward pass repeated with newer parameters: head outputs at acting time, else null
    const float* path;                     // pathwise policy gradient: dL/d(mu, log_sigma) per sample replaces the
                                           // score-function term, and the reported policy loss is minus the mean reward
};

// what the loss of a sample reads, besides its advantage and return
struct HeadIn { float4 h0, h1; float eps, rew; int act, done; };
__device__ __forceinline__ HeadIn head_in(const HeadGradArgs& a, const int i)
{
    HeadIn x;
    const float* h = a.head + (size_t)i * a.NHP;
    x.h0 = *reinterpret_cast<const float4*>(h);
    x.h1 = a.NHP == 8 ? *reinterpret_cast<const float4*>(h + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    x.act = a.policy == POLICY_CATEGORICAL ? (int)a.act[i] : 0;
    x.eps = a.policy == POLICY_CATEGORICAL ? 0.0f : a.eps[i];
    x.rew = a.rew[i]; x.done = a.done[i];
    return x;
}

// one sample: its loss terms, and its head gradient to a.dhead.  A_, G_: advantage and return of the sample
__device__ __forceinline__ void head_grad_sample(const HeadGradArgs& a, const int i, const HeadIn& x, float A_, const float G_,
                                                 float& lp_term, float& v_term, float& e_term, float& rsum, float& dcount)
{
    {
        const float hv[8] = {x.h0.x, x.h0.y, x.h0.z, x.h0.w, x.h1.x, x.h1.y, x.h1.z, x.h1.w};
        if (a.path) A_ = 0.0f;
        float V = hv[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) if (j == a.NH - 1) V = hv[j];
        float d[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const float dv = G_ - V;
        v_term = a.cv * dv * dv;
        const float gV = -2.0f * a.cv * dv * a.inv_m;
        if (a.policy == POLICY_CATEGORICAL) {
            const int act = x.act;
            float mx = hv[0];
#pragma unroll
            for (int j = 1; j < 8; ++j) if (j < a.A) mx = fmaxf(mx, hv[j]);
            float e[8], Z = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) { e[j] = (j < a.A) ? det_exp(hv[j] - mx) : 0.0f; Z += e[j]; }
            const float logZ = det_log(Z), invZ = 1.0f / Z;
            float H = 0.0f, lpa = 0.0f, p[8], lp[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                lp[j] = hv[j] - mx - logZ;
                p[j] = e[j] * invZ;
                if (j < a.A) H -= p[j] * lp[j];
                if (j == act) lpa = lp[j];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < a.A) d[j] = (-A_ * ((j == act ? 1.0f : 0.0f) - p[j]) + a.beta * p[j] * (lp[j] + H)) * a.inv_m;
            lp_term = -A_ * lpa;
            e_term = -a.beta * H;
        } else {
            const float ls = hv[1];
            const bool clamped = ls < -5.0f || ls > 2.0f;
            const float lsc = fminf(fmaxf(ls, -5.0f), 2.0f);
            const float sigma = det_exp(lsc);
            float ep = x.eps;
            if (a.head_old) ep = noise_now(a.head_old + (size_t)i * a.NHP, ep, hv[0], sigma);
            d[0] = (-A_ * ep / sigma) * a.inv_m;
            d[1] = clamped ? 0.0f : (-A_ * (ep * ep - 1.0f) - a.beta) * a.inv_m;
            lp_term = -A_ * (-0.5f * ep * ep - lsc - 0x1.d67f1cp-1f);
            e_term = -a.beta * (lsc + 0x1.6b3f8ep+0f);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) if (j == a.NH - 1) d[j] = gV;
        if (a.path) {
            const float2 pg = *reinterpret_cast<const float2*>(a.path + (size_t)i * 2);
            d[0] += pg.x; d[1] += pg.y;
            lp_term = -x.rew;
        }
        float* o = a.dhead + (size_t)i * a.NHP;
        *reinterpret_cast<float4*>(o) = make_float4(d[0], d[1], d[2], d[3]);
        if (a.NHP == 8) *reinterpret_cast<float4*>(o + 4) = make_float4(d[4], d[5], d[6], d[7]);
        rsum = x.rew;
        dcount = x.done ? 1.0f : 0.0f;
    }
}

// fixed-order block reduction of the five loss / metric sums: butterfly inside a wave, then waves in order
__device__ __forceinline__ void loss_block_sums(float lp_term, float v_term, float e_term, float rsum, float dcount,
                                                float (&red)[WG / 64][8], float* __restrict__ loss_part)
{
    float vals[5] = {lp_term, v_term, e_term, rsum, dcount};
#pragma unroll
    for (int k = 0; k < 5; ++k)
        for (int off = 32; off > 0; off >>= 1) vals[k] += __shfl_xor(vals[k], off, 64);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 5; ++k) red[wave][k] = vals[k];
    __syncthreads();
    if (threadIdx.x < 8) {
        float s = 0.0f;
        if (threadIdx.x < 5)
            for (int w = 0; w < WG / 64; ++w) s += red[w][threadIdx.x];
        loss_part[(size_t)blockIdx.x * 8 + threadIdx.x] = s;
    }
}

__global__ __launch_bounds__(WG) void head_grad(const HeadGradArgs a, const SplitWeightsArgs sw, const int blocks)
{
    if ((int)blockIdx.x >= blocks) { split_weights(sw, (int)blockIdx.x - blocks); return; }
    __shared__ float red[WG / 64][8];
    const int i = blockIdx.x * WG + threadIdx.x;
    float lp_term = 0.0f, v_term = 0.0f, e_term = 0.0f, rsum = 0.0f, dcount = 0.0f;
    if (i < a.M) head_grad_sample(a, i, head_in(a, i), a.adv[i], a.ret[i], lp_term, v_term, e_term, rsum, dcount);
    loss_block_sums(lp_term, v_term, e_term, rsum, dcount, red, a.loss_part);
}

// ---------------------------------------------------------------------------
// Returns and loss in one launch (the plain on-policy update): a workgroup owns E envs for all T steps (8 or 16:
// 256 samples or fewer where that is possible, so that every thread takes one).  Its
// rewards, values and episode ends come into LDS with every thread loading, the first E lanes then run
// returns_scan's recursion out of LDS (returns and advantages to memory, for the caller to see, and to LDS), and
// every thread takes the samples s, s + 256, ... of the workgroup's T x E through head_grad's arithmetic.
// One launch and no trip of the advantages through memory between the two.
// VTRACE: the off-policy targets of a decoupled step in the same manner; the ratios take the place of the rewards' pass.
// ---------------------------------------------------------------------------
constexpr int SL_MAXN = 1024;            // samples of a workgroup at most (T x envs)
struct ScanLossArgs {
    HeadGradArgs g;
    int B, T, E;                           // E: envs per workgroup (8 or 16)
    const float* val;                      // [T + 1][B]
    float gamma, lambda;
    float* adv_out; float* ret_out;
    int blocks;                            // workgroups with environments; further ones split weights
    VtraceArgs v;                          // VTRACE: heads and noise of both policies
};

template <bool VTRACE>
__global__ __launch_bounds__(WG) void scan_loss(const ScanLossArgs a, const SplitWeightsArgs sw)
{
    if ((int)blockIdx.x >= a.blocks) { split_weights(sw, (int)blockIdx.x - a.blocks); return; }
    __shared__ float red[WG / 64][8];
    __shared__ float rews[SL_MAXN], vals[SL_MAXN + 16], discs[SL_MAXN];
    __shared__ float advs[SL_MAXN], rets[SL_MAXN], rhos[VTRACE ? SL_MAXN : 1];
    const int B = a.B, T = a.T, SL_E = a.E, lg = SL_E == 16 ? 4 : 3, tid = threadIdx.x;
    const int b0 = blockIdx.x * SL_E;
    const int n = T * SL_E;
    auto sample = [&](int s) { return (s >> lg) * B + b0 + (s & (SL_E - 1)); };
    // Latency is what this launch is made of: all loads of a thread's first samples go out before anything waits (loads of
    // one sample after another, and of the loss behind the scan, were a round trip to memory each, and so was a step of the
    // recursion to LDS: pendulum, 1024 environments, T = 32 7.5 -> 5.3 us; 8192, T = 32 10.5 -> 8.0; Catch, 4096, T = 20 7.1 -> 6.9)
    // (V-trace: few at a time, so that its workgroups find room beside the actor's, whose registers leave 80 per lane; with 93
    // they waited for the actor to end, and a decoupled step of two layers of 256 took 408 us instead of 392)
    constexpr int LB = VTRACE ? 1 : 4, PF = VTRACE ? 1 : 2, SB = VTRACE ? 4 : 8;
    HeadIn in[PF];
    for (int s0 = tid; s0 < n + SL_E; s0 += LB * WG) {
        float v[LB], r[LB];
        int d[LB];
#pragma unroll
        for (int q = 0; q < LB; ++q) {                           // past the end: the last one again, unused
            const int s = s0 + q * WG, i1 = sample(s < n + SL_E ? s : n + SL_E - 1), i = sample(s < n ? s : n - 1);
            v[q] = a.val[i1]; r[q] = a.g.rew[i]; d[q] = a.g.done[i];
        }
        if (!VTRACE && s0 == tid) {
#pragma unroll
            for (int q = 0; q < PF; ++q) in[q] = head_in(a.g, sample(tid + q * WG < n ? tid + q * WG : n - 1));
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int s = s0 + q * WG;
            if (s < n + SL_E) vals[s] = v[q];
            if (s < n) {
                rews[s] = r[q]; discs[s] = d[q] ? 0.0f : a.gamma;
                if (VTRACE) rhos[VTRACE ? s : 0] = vtrace_rho(a.v, sample(s));
            }
        }
    }
    __syncthreads();
    // the operands of several steps are read before the first of them is used: one LDS round trip for all of them
    if (tid < SL_E) {
        const float oml = 1.0f - a.lambda;
        float Vnext = vals[n + tid], tail = 0.0f;                // V-trace: v_{t+1} - V_{t+1}
        float G = Vnext;
        auto steps = [&](auto count, int t1) {
            constexpr int N = decltype(count)::value;
            float V[N], r[N], disc[N], rho[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int s = (t1 - 1 - u) * SL_E + tid;
                V[u] = vals[s]; r[u] = rews[s]; disc[u] = discs[s]; rho[u] = VTRACE ? rhos[VTRACE ? s : 0] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int s = (t1 - 1 - u) * SL_E + tid;
                if (VTRACE) {
                    const float c = a.lambda * rho[u];
                    advs[s] = rho[u] * (fmaf(disc[u], Vnext + tail, r[u]) - V[u]);
                    tail = fmaf(disc[u] * c, tail, rho[u] * (fmaf(disc[u], Vnext, r[u]) - V[u]));
                    rets[s] = V[u] + tail;
                } else {
                    const float mix = fmaf(a.lambda, G, oml * Vnext);
                    G = fmaf(disc[u], mix, r[u]);
                    rets[s] = G;
                    advs[s] = G - V[u];
                }
                Vnext = V[u];
            }
        };
        int t1 = T;
        for (; t1 >= SB; t1 -= SB) steps(std::integral_constant<int, SB>(), t1);
        for (; t1 > 0; --t1) steps(std::integral_constant<int, 1>(), t1);
    }
    __syncthreads();
    float lp_term = 0.0f, v_term = 0.0f, e_term = 0.0f, rsum = 0.0f, dcount = 0.0f;
    for (int s0 = tid; s0 < n; s0 += PF * WG) {
        if (VTRACE || s0 != tid) {
#pragma unroll
            for (int q = 0; q < PF; ++q) in[q] = head_in(a.g, sample(s0 + q * WG < n ? s0 + q * WG : n - 1));
        }
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const int s = s0 + q * WG;
            if (s >= n) break;
            const int i = sample(s);
            const float A_ = advs[s], G_ = rets[s];
            a.adv_out[i] = A_;
            a.ret_out[i] = G_;
            float l0, l1, l2, l3, l4;
            head_grad_sample(a.g, i, in[q], A_, G_, l0, l1, l2, l3, l4);
            lp_term += l0; v_term += l1; e_term += l2; rsum += l3; dcount += l4;
        }
    }
    loss_block_sums(lp_term, v_term, e_term, rsum, dcount, red, a.g.loss_part);
}

// ---------------------------------------------------------------------------
// Heads: dWh[j][a] = sum_m h[m][j] dhead[m][a], dbh[a] = sum_m dhead[m][a] (per
// row chunk, as split-K partials) and dZ[m][j] = (h[m][j] > 0) sum_a Wh[j][a]
// dhead[m][a].  K = NH <= 5 is no matrix-core shape: plain vector FMAs, one
// pass over h (read) and dZ (write), both coalesced.
// A workgroup handles `rows` consecutive samples; when the hidden width is
// below 256 several rows are processed side by side and their partial sums are
// combined through LDS in a fixed order.
// ---------------------------------------------------------------------------
struct HeadBwdArgs {
    int M, H, NH, NHP, rows;
    const float* h; const float* dhead; const float* wh;   // wh: theta + wh_off, [H][NH]
    float* dz; float* partial;                             // partial: [splits][H*NH + NH]
    int bf16;
};

// Each lane owns four consecutive hidden units (16-byte loads and stores), H/4 lanes
// cover a row, and 256/(H/4) rows are processed side by side by one workgroup.
__global__ __launch_bounds__(WG) void head_backward(const HeadBwdArgs a)
{
    extern __shared__ float lds[];                          // [groups][H*NH + NH] for the final combine
    const int H = a.H, NH = a.NH, NHP = a.NHP;
    const int hw = H >> 2;                                  // lanes across the hidden dimension (<= 256)
    const int groups = WG / hw;                             // rows processed side by side
    const int g = threadIdx.x / hw, j = (threadIdx.x % hw) << 2;
    const int split = blockIdx.x;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    float w[4][8], dw[4][8], db[8];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float x = (k < NH) ? a.wh[(size_t)(j + c) * NH + k] : 0.0f;
            if (a.bf16) x = bf16_to_f(bf16_bits(x));
            w[c][k] = x; dw[c][k] = 0.0f;
        }
#pragma unroll
    for (int k = 0; k < 8; ++k) db[k] = 0.0f;
    const float* __restrict__ hin = a.h;
    const float* __restrict__ dhin = a.dhead;
    float* __restrict__ dzo = a.dz;
    constexpr int RB = 4;                                   // rows in flight per lane
    for (int mb = m_begin + g; mb < m_end; mb += RB * groups) {
        float4 hv4[RB], d0[RB], d1[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int m = mb + u * groups;
            const bool ok = m < m_end;
            hv4[u] = ok ? *reinterpret_cast<const float4*>(hin + (size_t)m * H + j) : make_float4(0, 0, 0, 0);
            d0[u] = ok ? *reinterpret_cast<const float4*>(dhin + (size_t)m * NHP) : make_float4(0, 0, 0, 0);
            d1[u] = (ok && NHP == 8) ? *reinterpret_cast<const float4*>(dhin + (size_t)m * NHP + 4) : make_float4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int m = mb + u * groups;
            if (m >= m_end) break;
            const float d[8] = {d0[u].x, d0[u].y, d0[u].z, d0[u].w, d1[u].x, d1[u].y, d1[u].z, d1[u].w};
            const float hv[4] = {hv4[u].x, hv4[u].y, hv4[u].z, hv4[u].w};
            float o[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float sacc = 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (k < NH) {
                        sacc = fmaf(w[c][k], d[k], sacc);
                        dw[c][k] = fmaf(hv[c], d[k], dw[c][k]);
                    }
                }
                o[c] = hv[c] > 0.0f ? sacc : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) if (k < NH) db[k] += d[k];
            *reinterpret_cast<float4*>(dzo + (size_t)m * H + j) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
    // combine the row groups in ascending group order
    const int stride = H * NH + NH;
    float* out = a.partial + (size_t)split * stride;
    float* mine = lds + (size_t)g * stride;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        for (int k = 0; k < NH; ++k) mine[(j + c) * NH + k] = dw[c][k];
    if (j == 0) for (int k = 0; k < NH; ++k) mine[H * NH + k] = db[k];
    __syncthreads();
    for (int i = threadIdx.x; i < stride; i += WG) {
        float s = 0.0f;
        for (int gg = 0; gg < groups; ++gg) s += lds[(size_t)gg * stride + i];
        out[i] = s;
    }
}

// The same pass on the matrix cores (v_mfma_f32_32x32x2_f32, whose sum over the reduction index is
// the same ascending fma chain the vector kernel uses, so dZ_L is unchanged bit for bit):
//   dZ_L tile [32 samples][32 units] = dhead[32][8] Wh^T[8][32]        4 MFMAs, then the ReLU mask
//   dWh  tile [32 units][heads]     += h^T[32][2 samples] dhead[2][..]  16 MFMAs per 32 samples
// The reduction over samples may take them in any order as long as both operands agree; step (g, q)
// uses sample 8g + 4kg + q for lane half kg, which is the row of the dZ_L accumulator that lane holds,
// so one load of h serves as operand and as mask.  A workgroup walks its rows 32 at a time;
// wavefront w owns units 64w..64w+63 of the 256 the workgroup covers.
typedef float f16v_h __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(WG) void head_backward_mfma(const HeadBwdArgs a)
{
    __shared__ float Dl[2][32 * 8];                          // head gradients of the current 32 samples, double buffered
    __shared__ float red[WG];
    const int H = a.H, NH = a.NH, NHP = a.NHP;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, kg = lane >> 5;
    const int jw = blockIdx.y * 256 + wave * 64;             // first unit of this wavefront
    const bool active = jw < H;                              // H is a multiple of 64
    const int split = blockIdx.x;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    // Wh of this lane's unit in both tiles, as B operand of the dZ product: step i takes heads 2i + kg
    float wB[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 2 * i + kg;
            float x = (active && k < NH) ? a.wh[(size_t)(jw + 32 * t + l32) * NH + k] : 0.0f;
            if (a.bf16) x = bf16_to_f(bf16_bits(x));
            wB[t][i] = x;
        }
    f16v_h accw[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) accw[t][r] = 0.0f;
    // staging: thread (sample tid / 8, head tid % 8) moves one head gradient per step and keeps its sum
    const int ss = tid >> 3, sk = tid & 7;
    float dsum = 0.0f;
    auto stage = [&](int buf, int m0) {
        const float v = (sk < NH) ? a.dhead[(size_t)(m0 + ss) * NHP + sk] : 0.0f;
        Dl[buf][tid] = v;
        dsum += v;
    };
    const float* __restrict__ hin = a.h + jw + l32;
    float* __restrict__ dzo = a.dz + jw + l32;
    stage(0, m_begin);
    __syncthreads();
    int buf = 0;
    for (int m0 = m_begin; m0 < m_end; m0 += 32, buf ^= 1) {
        if (m0 + 32 < m_end) stage(buf ^ 1, m0 + 32);        // visible after the barrier at the end of this step
        if (active) {
            float hv[2][16];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    hv[t][r] = hin[(size_t)(m0 + 8 * (r >> 2) + 4 * kg + (r & 3)) * H + 32 * t];
            // dZ product: A = dhead[sample l32][head 2i + kg]
            float dA[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dA[i] = Dl[buf][l32 * 8 + 2 * i + kg];
            // dWh product: B = dhead[sample 8g + 4kg + q][head l32] for l32 < 8, zero columns beyond
            float dB[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) dB[r] = l32 < 8 ? Dl[buf][(8 * (r >> 2) + 4 * kg + (r & 3)) * 8 + l32] : 0.0f;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f16v_h accz;
#pragma unroll
                for (int r = 0; r < 16; ++r) accz[r] = 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) accz = __builtin_amdgcn_mfma_f32_32x32x2f32(dA[i], wB[t][i], accz, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r) accw[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(hv[t][r], dB[r], accw[t], 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    dzo[(size_t)(m0 + 8 * (r >> 2) + 4 * kg + (r & 3)) * H + 32 * t] = hv[t][r] > 0.0f ? accz[r] : 0.0f;
            }
        }
        __syncthreads();
    }
    // dWh: row = unit 8(r/4) + 4kg + r%4 of the tile, column = head l32
    float* out = a.partial + (size_t)split * ((size_t)H * NH + NH);
    if (active && l32 < NH) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                out[(size_t)(jw + 32 * t + 8 * (r >> 2) + 4 * kg + (r & 3)) * NH + l32] = accw[t][r];
    }
    if (blockIdx.y == 0) {
        red[tid] = dsum;
        __syncthreads();
        if (tid < NH) {
            float sum = 0.0f;
            for (int i = 0; i < 32; ++i) sum += red[i * 8 + tid];
            out[(size_t)H * NH + tid] = sum;
        }
    }
}

// ---------------------------------------------------------------------------
// Second stage of a two-level split-K sum: dst[s][i] = sum_{f < fan} src[s*fan + f][i],
// in ascending f.  Lets a bandwidth-bound producer use many small workgroups while the
// Adam kernel still sees few partials.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void partial_reduce(const float* __restrict__ src, float* __restrict__ dst, int count, int fan)
{
    const int i = blockIdx.x * WG + threadIdx.x, s = blockIdx.y;
    if (i >= count) return;
    const float* p = src + (size_t)s * fan * count + i;
    float acc = 0.0f;
#pragma unroll 4
    for (int f = 0; f < fan; ++f) acc += p[(size_t)f * count];
    dst[(size_t)s * count + i] = acc;
}

// ---------------------------------------------------------------------------
// First-layer gradient of the pendulum without a GEMM (boards: first_layer.hip): the three observation features are
// rebuilt from the stored angle and velocity and lane j keeps three register sums of its column, and the column sum
// (the bias gradient).  Widths under 256: the workgroup's row groups are added in ascending order.
// ---------------------------------------------------------------------------
struct FirstGradArgs {
    int M, K, N, rows, bf16;  // bf16: the features are rounded, as the forward pass read them
    const float* dy;          // [M][N] gradient w.r.t. the first layer's pre-activations
    float* partial;           // [splits][K*N + N]
    ObsLite obs;
};

__global__ __launch_bounds__(WG) void first_layer_grad(const FirstGradArgs a)
{
    __shared__ float sums[4][WG];
    const int N = a.N, K = a.K;
    const int cw = N < WG ? N : WG, groups = WG / cw;
    const int g = threadIdx.x / cw, jl = threadIdx.x % cw;
    const int j = blockIdx.y * WG + jl;
    const int split = blockIdx.x;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    float bsum = 0.0f, r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;
    const float* __restrict__ dyin = a.dy;
    constexpr int RB = 16;                                   // rows in flight per lane
    for (int mb = m_begin + g; mb < m_end; mb += RB * groups) {
        float d[RB], f0[RB], f1[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int m = mb + u * groups;
            const bool ok = m < m_end;
            d[u] = ok ? dyin[(size_t)m * N + j] : 0.0f;
            f0[u] = ok ? a.obs.f0[m] : 0.0f; f1[u] = ok ? a.obs.f1[m] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            if (mb + u * groups >= m_end) break;
            bsum += d[u];
            float sn, cs, td = f1[u];
            det_sincos(f0[u], sn, cs);
            if (a.bf16) { cs = bf16_to_f(bf16_bits(cs)); sn = bf16_to_f(bf16_bits(sn)); td = bf16_to_f(bf16_bits(td)); }
            r0 = fmaf(cs, d[u], r0); r1 = fmaf(sn, d[u], r1); r2 = fmaf(td, d[u], r2);
        }
    }
    float* out = a.partial + (size_t)split * ((size_t)K * N + N);
    sums[0][threadIdx.x] = r0; sums[1][threadIdx.x] = r1; sums[2][threadIdx.x] = r2; sums[3][threadIdx.x] = bsum;
    __syncthreads();
    // combine the row groups in ascending order; row 3 is the bias, behind the three weight rows
    for (int i = threadIdx.x; i < 4 * cw; i += WG) {
        const int k = i / cw, c = i % cw;
        float s = 0.0f;
        for (int gg = 0; gg < groups; ++gg) s += sums[k][gg * cw + c];
        out[(size_t)k * N + blockIdx.y * WG + c] = s;
    }
}

// Pendulum first layer for widths that are multiples of 256: the three observation features of a
// row (cos, sin, angular velocity) are computed once per row by one thread and shared through LDS,
// instead of once per row by every column; lane j then walks the rows in ascending order.
__global__ __launch_bounds__(WG) void first_layer_grad_pendulum(const FirstGradArgs a)
{
    __shared__ float feat[3][WG];
    const int N = a.N;
    const int j = blockIdx.y * WG + threadIdx.x;
    const int split = blockIdx.x;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    float bsum = 0.0f, r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;
    const float* __restrict__ dy = a.dy + j;
    for (int mb = m_begin; mb < m_end; mb += WG) {
        const int m = mb + threadIdx.x;
        float sn = 0.0f, cs = 0.0f, td = 0.0f;
        if (m < m_end) { det_sincos(a.obs.f0[m], sn, cs); td = a.obs.f1[m]; }
        if (a.bf16) { cs = bf16_to_f(bf16_bits(cs)); sn = bf16_to_f(bf16_bits(sn)); td = bf16_to_f(bf16_bits(td)); }
        __syncthreads();                                     // the previous batch has been consumed
        feat[0][threadIdx.x] = cs; feat[1][threadIdx.x] = sn; feat[2][threadIdx.x] = td;
        __syncthreads();
        const int n = m_end - mb < WG ? m_end - mb : WG;
        constexpr int RB = 16;
        for (int u0 = 0; u0 < n; u0 += RB) {
            float d[RB];
#pragma unroll
            for (int u = 0; u < RB; ++u) d[u] = u0 + u < n ? dy[(size_t)(mb + u0 + u) * N] : 0.0f;
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                if (u0 + u >= n) break;
                bsum += d[u];
                r0 = fmaf(feat[0][u0 + u], d[u], r0); r1 = fmaf(feat[1][u0 + u], d[u], r1); r2 = fmaf(feat[2][u0 + u], d[u], r2);
            }
        }
    }
    float* out = a.partial + (size_t)split * ((size_t)a.K * N + N);
    out[j] = r0; out[(size_t)N + j] = r1; out[(size_t)2 * N + j] = r2;
    out[(size_t)a.K * N + j] = bsum;
}

typedef float f4v_l __attribute__((ext_vector_type(4)));

hipError_t launch_first_layer_grad(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    FirstGradArgs a;
    a.M = h->B * h->T; a.K = n.dims[0]; a.N = n.dims[1]; a.bf16 = n.bf16;
    a.rows = chunk_rows(a.M, h->splits[0], h->quanta[0]);
    a.dy = at<const float>(h, L.dz[0]); a.partial = at<float>(h, L.part[0]);
    a.obs.env = h->env; a.obs.s0 = at<const uint32_t>(h, L.tr_s0);
    a.obs.f0 = at<const float>(h, L.tr_f0); a.obs.f1 = at<const float>(h, L.tr_f1);
    ProfScope prof(h, "first_layer_grad");
    if (a.N % WG == 0) hipLaunchKernelGGL(first_layer_grad_pendulum, dim3(h->splits[0], a.N / WG), dim3(WG), 0, h->stream, a);
    else hipLaunchKernelGGL(first_layer_grad, dim3(h->splits[0], (a.N + WG - 1) / WG), dim3(WG), 0, h->stream, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Catch with one hidden layer of 32 units (the throughput workload): the WHOLE update up to the
// partial sums in one launch -- returns and advantages, loss and head gradients, and the backward
// pass above -- so that advantages, returns and head gradients never make a round trip through
// HBM (the returns are still written once, for the caller to see) and three launches become one.
// A workgroup of four wavefronts owns a range of envs for all T steps; each wavefront takes 64 of
// them at a time:
//   A1  lane = env: the reverse scan of its column (returns_scan's recursion), adv / ret to HBM
//   A2  lane = env, four time steps at a time: the loss terms and head gradients of its samples
//       (head_grad's arithmetic) into LDS, with the two board cells of the sample as LDS offsets
//   B   lane = (hidden unit, half): each half-wavefront walks every other sample of the chunk:
//       h = relu(b1 + W1[ball] + W1[paddle]) in the acting order, dZ1, the head-matrix sums, and
//       the scatter of dZ1 into the two rows of its own LDS copy of dW1
// A2 and B exchange through the wavefront's own LDS, so no barrier stands between them.  Catch 10 x 5, 262144 environments,
// T = 16: 150 us (155 with a bias sum of its own, the bias added per sample and word offsets); 47 of them are A1 and A2, the
// rest the walk's LDS reads and writes: half the vector instructions, with the head products on the matrix instruction, took
// 148, two samples per LDS round trip 148, 16 lanes of two units per row 172, the paddle's row by matrix instruction 161.
// ---------------------------------------------------------------------------
struct CatchFusedArgs {
    int B, T, D, envs_per_wg;
    EnvDims env;
    const float* theta; int w1_off, b1_off, wh_off;
    const uint32_t* s0; const uint8_t* act; const float* rew; const uint8_t* done; const float* val; const float* head;
    float* adv; float* ret;
    float* partial0;          // [workgroups][D*32 + 32]
    float* partial1;          // [workgroups][32*4 + 4]
    float* loss_part;         // [workgroups][8]
    float gamma, lambda, beta, cv, inv_m;
};

constexpr int CF_WG = 256;              // four wavefronts
constexpr int CF_H = 32;                // hidden units
constexpr int CF_TC = 4;                // time steps per chunk of phases A2 / B

__global__ __launch_bounds__(CF_WG) void learn_catch_fused(const CatchFusedArgs a)
{
    extern __shared__ float lds[];
    const int D = a.D, B = a.B, T = a.T;
    constexpr int H = CF_H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* w1s = lds;                                            // [D][H]
    float* accw = w1s + D * H + (size_t)wave * (2 * D * H + CF_TC * 64 * 4 + CF_TC * 64);
    float* acc = accw;                                           // [2 halves][D][H] this wavefront's dW1 sums
    float4* dh = reinterpret_cast<float4*>(accw + 2 * D * H);    // [CF_TC][64] head gradients of the chunk
    uint32_t* cells = reinterpret_cast<uint32_t*>(dh + CF_TC * 64);   // [CF_TC][64] LDS offsets of the two board cells
    // W1 into LDS in batches of four 16-byte loads per thread (one load, one wait, one store at a time would be a
    // memory round trip per 4 KB); H is a multiple of 4, and so is the offset of W1 in the parameter vector
    {
        const int n4 = D * H / 4;
        const f4v_l* src = reinterpret_cast<const f4v_l*>(a.theta + a.w1_off);
        f4v_l* dst = reinterpret_cast<f4v_l*>(w1s);
        for (int i0 = 0; i0 < n4; i0 += 4 * CF_WG) {
            f4v_l pw[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) { const int i = i0 + q * CF_WG + tid; pw[q] = src[i < n4 ? i : 0]; }
#pragma unroll
            for (int q = 0; q < 4; ++q) { const int i = i0 + q * CF_WG + tid; if (i < n4) dst[i] = pw[q]; }
        }
    }
    for (int i = lane; i < 2 * D * H; i += 64) acc[i] = 0.0f;
    // phase B identity: hidden unit u, half hf (the two halves of a wavefront take alternate samples)
    const int u = lane & 31, hf = lane >> 5;
    float wh[4], dwh[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) wh[k] = a.theta[a.wh_off + u * 4 + k];
    const uint32_t w_at = (uint32_t)u * 4;                       // LDS byte offsets of this lane's column of W1 and of its sums
    const uint32_t m_at = (uint32_t)(acc - lds + hf * D * H + u) * 4;
    auto word = [&](uint32_t at) -> float& { return *reinterpret_cast<float*>(reinterpret_cast<char*>(lds) + at); };
    // phase A identity: env e of the wavefront's block; sums of the loss terms and of the head gradients
    float dbh[4] = {0, 0, 0, 0}, sums[5] = {0, 0, 0, 0, 0};
    __syncthreads();
    // the bias joins the rows of the cells a ball can be in (the paddle's row is the last, and the ball is never in it):
    // b1 + W1[ball] is the first sum of the acting order
    for (int i = tid; i < (D - a.env.cols) * H; i += CF_WG) w1s[i] = a.theta[a.b1_off + (i & (H - 1))] + w1s[i];
    __syncthreads();
    const float oml = 1.0f - a.lambda;
    const int wg_b0 = blockIdx.x * a.envs_per_wg;
    for (int blk = 0; blk < a.envs_per_wg; blk += CF_WG) {
        const int b = wg_b0 + blk + wave * 64 + lane;
        // ---- A1: returns and advantages of this env, newest step first ----
        {
            float G = a.val[(size_t)T * B + b], vnext = G;
            // eight steps' records are asked for before the first of them is used: the stores of one step and the
            // loads of the next may be the same memory as far as the compiler knows, so step by step every load
            // would wait for its own round trip
            for (int t1 = T; t1 > 0; t1 -= 8) {
                float r8[8], v8[8], d8[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int t = t1 - 1 - u;
                    const size_t i = (size_t)(t >= 0 ? t : 0) * B + b;
                    r8[u] = a.rew[i]; v8[u] = a.val[i]; d8[u] = a.done[i] ? 0.0f : a.gamma;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int t = t1 - 1 - u;
                    if (t >= 0) {
                        const size_t i = (size_t)t * B + b;
                        const float mix = fmaf(a.lambda, G, oml * vnext);
                        G = fmaf(d8[u], mix, r8[u]);
                        a.ret[i] = G;
                        a.adv[i] = G - v8[u];
                        vnext = v8[u];
                    }
                }
            }
        }
        // the records of a chunk's samples: asked for one chunk ahead, so that they arrive while the chunk before is in
        // phase B (straight after the barrier every load would be a round trip to memory with nothing to hide it)
        f4v_l in_h[CF_TC]; float in_adv[CF_TC], in_ret[CF_TC], in_rew[CF_TC]; uint32_t in_s0[CF_TC]; int in_act[CF_TC], in_done[CF_TC];
        auto fetch_chunk = [&](int t0) {
#pragma unroll
            for (int tt = 0; tt < CF_TC; ++tt) {
                const int t = t0 + tt < T ? t0 + tt : T - 1;         // past the end: re-read the last step, unused
                const size_t i = (size_t)t * B + b;
                in_h[tt] = *reinterpret_cast<const f4v_l*>(a.head + i * 4);
                in_act[tt] = (int)a.act[i]; in_adv[tt] = a.adv[i]; in_ret[tt] = a.ret[i];
                in_rew[tt] = a.rew[i]; in_done[tt] = a.done[i]; in_s0[tt] = a.s0[i];
            }
        };
        fetch_chunk(0);
        for (int t0 = 0; t0 < T; t0 += CF_TC) {
            const int tn = T - t0 < CF_TC ? T - t0 : CF_TC;
            // ---- A2: loss terms and head gradients of (t0 .. t0 + tn - 1, b) ----
#pragma unroll
            for (int tt = 0; tt < CF_TC; ++tt) {
                if (tt < tn) {
                    const float4 hv4 = make_float4(in_h[tt][0], in_h[tt][1], in_h[tt][2], in_h[tt][3]);
                    float d[4], lp_term, v_term, e_term;
                    catch_head_grad(hv4, in_act[tt], in_adv[tt], in_ret[tt], a.beta, a.cv, a.inv_m, d, lp_term, v_term, e_term);
                    sums[0] += lp_term; sums[1] += v_term; sums[2] += e_term; sums[3] += in_rew[tt]; sums[4] += in_done[tt] ? 1.0f : 0.0f;
#pragma unroll
                    for (int k = 0; k < 4; ++k) dbh[k] += d[k];
                    dh[tt * 64 + lane] = make_float4(d[0], d[1], d[2], d[3]);
                    int bc, pc;
                    catch_obs_cells(a.env, in_s0[tt], bc, pc);
                    cells[tt * 64 + lane] = (uint32_t)(bc * H * 4) | ((uint32_t)(pc * H * 4) << 16);
                }
            }
            wave_fence();
            if (t0 + CF_TC < T) fetch_chunk(t0 + CF_TC);
            // ---- B: half hf takes samples hf, hf + 2, ... of the chunk's tn * 64 ----
            const int ns = tn * 64;
            constexpr int RB = 8;
            for (int s0 = 0; s0 < ns; s0 += 2 * RB) {
                float4 dd[RB];
                uint32_t cc[RB];
#pragma unroll
                for (int q = 0; q < RB; ++q) { dd[q] = dh[s0 + 2 * q + hf]; cc[q] = cells[s0 + 2 * q + hf]; }
                float w0[RB], w1[RB];
#pragma unroll
                for (int q = 0; q < RB; ++q) { w0[q] = word(w_at + (cc[q] & 0xffffu)); w1[q] = word(w_at + (cc[q] >> 16)); }
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    const float d[4] = {dd[q].x, dd[q].y, dd[q].z, dd[q].w};
                    float hv = w0[q] + w1[q];
                    hv = hv > 0.0f ? hv : 0.0f;
                    float s = 0.0f;
#pragma unroll
                    for (int k = 0; k < 4; ++k) { s = fmaf(wh[k], d[k], s); dwh[k] = fmaf(hv, d[k], dwh[k]); }
                    const float dz = hv > 0.0f ? s : 0.0f;
                    // the ball is never in the paddle's row, so the two sums are different words: both reads go out
                    // before either store, one LDS round trip per sample instead of two (two samples per round
                    // trip, with the second taking the first's result where they share a word, measured slower)
                    float &pa = word(m_at + (cc[q] & 0xffffu)), &pb = word(m_at + (cc[q] >> 16));
                    const float xa = pa, xb = pb;
                    pa = xa + dz;
                    pb = xb + dz;
                }
            }
            wave_fence();
        }
    }
    __syncthreads();
    // ---- sums of the workgroup, in a fixed order: wavefronts ascending, half 0 before half 1 ----
    // every wavefront's dW1 copies are complete (barrier above); the per-lane sums go through the wavefront's
    // head-gradient area, free now: 16 floats per lane
    const size_t ws = (size_t)2 * D * H + CF_TC * 64 * 4 + CF_TC * 64;        // floats per wavefront
    auto red_of = [&](int w, int l) { return w1s + D * H + (size_t)w * ws + 2 * D * H + (size_t)l * 16; };
    {
        float* r = red_of(wave, lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) { r[k] = dwh[k]; r[4 + k] = dbh[k]; }
#pragma unroll
        for (int k = 0; k < 5; ++k) r[8 + k] = sums[k];
    }
    __syncthreads();
    float* out0 = a.partial0 + (size_t)blockIdx.x * ((size_t)D * H + H);
    float* out1 = a.partial1 + (size_t)blockIdx.x * ((size_t)H * 4 + 4);
    float* acc_all = w1s + D * H;                                // wavefront w at stride ws
    for (int i = tid; i < D * H; i += CF_WG) {
        float sum = 0.0f;
        for (int w = 0; w < 4; ++w) { sum += acc_all[w * ws + i]; sum += acc_all[w * ws + D * H + i]; }
        out0[i] = sum;
        if (i >= (D - a.env.cols) * H) acc_all[i] = sum;         // this thread's word alone
    }
    __syncthreads();
    if (tid < H) {
        // every sample has its paddle in one cell of the last row, so the bias gradient is the sum of that row's cells
        float sb = 0.0f, sw[4] = {0, 0, 0, 0};
        for (int c = D - a.env.cols; c < D; ++c) sb += acc_all[c * H + tid];
        for (int w = 0; w < 4; ++w)
            for (int hh = 0; hh < 2; ++hh) {
                const float* r = red_of(w, hh * 32 + tid);
#pragma unroll
                for (int k = 0; k < 4; ++k) sw[k] += r[k];
            }
        out0[(size_t)D * H + tid] = sb;
#pragma unroll
        for (int k = 0; k < 4; ++k) out1[(size_t)tid * 4 + k] = sw[k];
    }
    if (tid < 9) {
        // dbh[0..3] and the five metric sums: over all 256 lanes (envs), ascending
        const int off = tid < 4 ? 4 + tid : 8 + (tid - 4);
        float sum = 0.0f;
        for (int l = 0; l < CF_WG; ++l) sum += red_of(l >> 6, l & 63)[off];
        if (tid < 4) out1[(size_t)H * 4 + tid] = sum;
        else a.loss_part[(size_t)blockIdx.x * 8 + (tid - 4)] = sum;
    }
    if (tid >= 9 && tid < 12) a.loss_part[(size_t)blockIdx.x * 8 + tid - 4] = 0.0f;
}

// whether the fused launch above serves this handle's update (else: scan, loss and one-layer kernels)
bool catch_fused_ok(const anakin* h)
{
    const NetShape& n = h->net;
    return one_layer_fused(h) && catch_fused_groups(n, h->env, h->B, h->T) > 0 && h->env.rows >= 2 && n.NH == 4 && h->n_updates == 1 &&
           !h->traj_decoupled && !h->pathwise &&
           n.dims[0] * CF_H * 4 < 65536 && n.w_off[0] % 4 == 0;           // board-cell offsets are packed into 16 bits; W1 is read 16 bytes at a time
}

hipError_t launch_learn_catch_fused(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    CatchFusedArgs a;
    a.B = h->B; a.T = h->T; a.D = n.dims[0]; a.envs_per_wg = h->B / h->splits[0];
    a.env = h->env;
    a.theta = at<const float>(h, L.w_src); a.w1_off = n.w_off[0]; a.b1_off = n.b_off[0]; a.wh_off = n.wh_off;
    a.s0 = at<const uint32_t>(h, L.tr_s0); a.act = at<const uint8_t>(h, L.tr_act); a.rew = at<const float>(h, L.tr_rew);
    a.done = at<const uint8_t>(h, L.tr_done); a.val = at<const float>(h, L.tr_val); a.head = at<const float>(h, L.tr_head);
    a.adv = at<float>(h, L.adv); a.ret = at<float>(h, L.ret);
    a.partial0 = at<float>(h, L.part[0]); a.partial1 = at<float>(h, L.part[1]); a.loss_part = at<float>(h, L.loss_part);
    a.gamma = h->net_cfg.gamma; a.lambda = h->net_cfg.lambda_; a.beta = h->net_cfg.entropy_coef; a.cv = h->net_cfg.value_coef;
    a.inv_m = (float)(1.0 / ((double)h->B * h->T));
    const size_t lds = ((size_t)a.D * CF_H + 4 * ((size_t)2 * a.D * CF_H + CF_TC * 64 * 4 + CF_TC * 64)) * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(learn_catch_fused), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    h->metric_blocks = h->splits[0];
    ProfScope prof(h, "learn_catch_fused");
    hipLaunchKernelGGL(learn_catch_fused, dim3(h->splits[0]), dim3(CF_WG), lds, h->stream, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adam with the gradient reduction fused in: g = sum over split-K partials in
// ascending split order, then m, v, theta.  Streams theta, m, v once in and
// once out (28 bytes per parameter besides the partials).  For bf16 networks
// the rounded copies the matrix-core kernels read are refreshed here too.
// ---------------------------------------------------------------------------
constexpr int ADAM_WAVES = 16;
typedef float f4v_a __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int adam_region_of(const AdamArgs& a, int i)
{
    int r = 0;
#pragma unroll
    for (int k = 1; k < MAX_ADAM_REGIONS; ++k) if (k < a.n_regions && i >= a.reg[k].start) r = k;
    return r;
}
__global__ __launch_bounds__(ADAM_WAVES * 64) void adam_reduce(const AdamArgs a)
{
    // 256 consecutive parameters per workgroup, four per lane; each of the 16 wavefronts adds its share of the
    // split-K partials (splits w, w+16, w+32, ...) with 16-byte loads -- one KiB per wavefront and partial row --
    // then the 16 sums are combined in wave order.  A group of four that straddles two regions, or lies in a
    // region whose rows are not 16-byte aligned, is summed parameter by parameter.
    __shared__ f4v_a red[ADAM_WAVES][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = (blockIdx.x * 64 + lane) * 4;
    f4v_a g = {0.0f, 0.0f, 0.0f, 0.0f};
    if (i < a.P) {
        const int r = adam_region_of(a, i);
        const Region rg = a.reg[r];
        const int off = i - rg.start;
        if (i + 3 < a.P && off + 3 < rg.count && ((rg.count | off) & 3) == 0) {
            const float* p = rg.partial + off;
#pragma unroll 4
            for (int s = wave; s < rg.splits; s += ADAM_WAVES) g += *reinterpret_cast<const f4v_a*>(p + (size_t)s * rg.count);
        } else {
            // the four parameters side by side, so that their loads overlap as the 16-byte ones do
            const float* pe[4]; size_t cnt[4]; int sp[4], smax = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ie = i + e < a.P ? i + e : i;
                const Region re = a.reg[adam_region_of(a, ie)];
                pe[e] = re.partial + (ie - re.start); cnt[e] = (size_t)re.count;
                sp[e] = i + e < a.P ? re.splits : 0;
                smax = sp[e] > smax ? sp[e] : smax;
            }
#pragma unroll 4
            for (int s = wave; s < smax; s += ADAM_WAVES) {
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] += s < sp[e] ? pe[e][(size_t)s * cnt[e]] : 0.0f;
            }
        }
    }
    red[wave][lane] = g;
    __syncthreads();
    if (wave != 0 || i >= a.P) return;
    g = red[0][lane];
#pragma unroll
    for (int w = 1; w < ADAM_WAVES; ++w) g += red[w][lane];
    if (i + 3 < a.P) {
        const f4v_a mo = *reinterpret_cast<const f4v_a*>(a.m + i), vo = *reinterpret_cast<const f4v_a*>(a.v + i);
        const f4v_a to = *reinterpret_cast<const f4v_a*>(a.theta + i);
        f4v_a m, v, th;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            m[e] = a.beta1 * mo[e] + (1.0f - a.beta1) * g[e];
            v[e] = a.beta2 * vo[e] + (1.0f - a.beta2) * g[e] * g[e];
            const float mh = m[e] / a.bc1, vh = v[e] / a.bc2;
            th[e] = to[e] - a.lr * mh / (sqrtf(vh) + a.eps);
        }
        *reinterpret_cast<f4v_a*>(a.grad + i) = g;
        *reinterpret_cast<f4v_a*>(a.m + i) = m;
        *reinterpret_cast<f4v_a*>(a.v + i) = v;
        *reinterpret_cast<f4v_a*>(a.theta + i) = th;
        if (a.w_bf16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint16_t hb = bf16_bits(th[e]);
                a.w_bf16[i + e] = hb;
                a.wt_bf16[transposed_index(a.net, i + e)] = hb;
            }
        }
        return;
    }
    for (int e = 0; e < 4 && i + e < a.P; ++e) {
        const float m = a.beta1 * a.m[i + e] + (1.0f - a.beta1) * g[e];
        const float v = a.beta2 * a.v[i + e] + (1.0f - a.beta2) * g[e] * g[e];
        const float mh = m / a.bc1, vh = v / a.bc2;
        const float th = a.theta[i + e] - a.lr * mh / (sqrtf(vh) + a.eps);
        a.grad[i + e] = g[e];
        a.m[i + e] = m;
        a.v[i + e] = v;
        a.theta[i + e] = th;
        if (a.w_bf16) {
            const uint16_t hb = bf16_bits(th);
            a.w_bf16[i + e] = hb;
            a.wt_bf16[transposed_index(a.net, i + e)] = hb;
        }
    }
}

// One parameter per lane, 64 per workgroup: four times the workgroups of adam_reduce, which is what small parameter
// vectors (under about 2^18) need to keep every compute unit loading.  Also where the partials are few: the 16 shares
// are one partial each, side by side, and their order is then ascending order, so the bits are adam_reduce_flat's
// (Catch 128-128, 256 samples, 16 partials: 24.0 us there, 6.7 here; 64-64-128: 24.0 and 6.5; 512-128 in bf16: 21 and
// 10.5).  What bounds it is the round trips to memory of a workgroup and how many rounds of workgroups there are: with 16
// wavefronts per workgroup, four loads in flight each and the moments asked for behind the sum, 79876 parameters with 128
// partials took 13.6 us, now 11.4; 158468 with 126 16.3 and 11.5; 67587 10.3 and 8.8; 17411 unchanged at 4.9 and
// (bf16) 6.3.  Vectors of less than a workgroup per unit keep a share to a wavefront: 1764 parameters with 512 partials 5.3 us,
// 6.4 with four shares.  (The moments beside the partials in adam_reduce as well: 58.5 -> 63.5 us on the maze's 921605 parameters.)
template <int SH>
__global__ __launch_bounds__(ADAM_WAVES * 64 / SH) void adam_reduce_narrow(const AdamArgs a)
{
    // 64 consecutive parameters per workgroup, 16 shares of the split-K partials (splits w, w + 16, w + 32, ...), SH to a
    // wavefront; then the 16 sums are combined in ascending order.  With four a wavefront has 32 loads in flight and a unit
    // room for four workgroups, so that the largest vectors that come here take little more than one round of them, or two.
    __shared__ float red[ADAM_WAVES][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    const bool ok = i < a.P;
    float g[SH], mo = 0.0f, vo = 0.0f, to = 0.0f;
#pragma unroll
    for (int h = 0; h < SH; ++h) g[h] = 0.0f;
    if (ok) {
        // the wavefront that takes the step has its parameters and moments under way beside the partials (asked for behind
        // the sum, they were a second memory round trip of every workgroup)
        if (wave == 0) { mo = a.m[i]; vo = a.v[i]; to = a.theta[i]; }
        int r = 0;
#pragma unroll
        for (int k = 1; k < MAX_ADAM_REGIONS; ++k) if (k < a.n_regions && i >= a.reg[k].start) r = k;
        const Region rg = a.reg[r];
        const float* p = rg.partial + (i - rg.start);
        constexpr int UF = 8;                                    // of each share
        for (int s0 = wave; s0 < rg.splits; s0 += UF * ADAM_WAVES) {
            float v[SH][UF];
#pragma unroll
            for (int u = 0; u < UF; ++u)
#pragma unroll
                for (int h = 0; h < SH; ++h) { const int s = s0 + h * (ADAM_WAVES / SH) + u * ADAM_WAVES; v[h][u] = p[(size_t)(s < rg.splits ? s : s0) * rg.count]; }
#pragma unroll
            for (int u = 0; u < UF; ++u)
#pragma unroll
                for (int h = 0; h < SH; ++h) g[h] = s0 + h * (ADAM_WAVES / SH) + u * ADAM_WAVES < rg.splits ? g[h] + v[h][u] : g[h];
        }
    }
#pragma unroll
    for (int h = 0; h < SH; ++h) red[wave + h * (ADAM_WAVES / SH)][lane] = g[h];
    __syncthreads();
    if (wave != 0 || !ok) return;
    float gs = red[0][lane];
#pragma unroll
    for (int w = 1; w < ADAM_WAVES; ++w) gs += red[w][lane];
    const float m = a.beta1 * mo + (1.0f - a.beta1) * gs;
    const float v = a.beta2 * vo + (1.0f - a.beta2) * gs * gs;
    const float mh = m / a.bc1, vh = v / a.bc2;
    const float th = to - a.lr * mh / (sqrtf(vh) + a.eps);
    a.grad[i] = gs;
    a.m[i] = m;
    a.v[i] = v;
    a.theta[i] = th;
    if (a.w_bf16) {
        const uint16_t hb = bf16_bits(th);
        a.w_bf16[i] = hb;
        a.wt_bf16[transposed_index(a.net, i)] = hb;
    }
}

// The same update for parameter regions with few partials (at most 16): one lane per parameter adds its
// partials in ascending order itself, so a wavefront streams 64 consecutive parameters of every array --
// the shape that reaches the HBM roofline when P is large (2^18 and up; below that it is a handful of workgroups).  The
// loads of four partials of all four parameters are in flight together (290820 parameters, 16 partials: 24.8 us one after
// another, 9.9 now; adam_reduce 10.5; 658949 parameters, 8 and 16 partials: 11.9, adam_reduce 18.5).
__global__ __launch_bounds__(WG) void adam_reduce_flat(const AdamArgs a)
{
    constexpr int UF = 4;                                        // parameters per lane, WG apart: loads of all four in flight
    const int i0 = blockIdx.x * (WG * UF) + threadIdx.x;
    float g[UF], mo[UF], vo[UF], to[UF];
    const float* p[UF];
    size_t cnt[UF];
    int sp[UF], smax = 0;
#pragma unroll
    for (int u = 0; u < UF; ++u) {
        const int i = i0 + u * WG;
        g[u] = 0.0f; mo[u] = 0.0f; vo[u] = 0.0f; to[u] = 0.0f; sp[u] = 0; p[u] = nullptr; cnt[u] = 0;
        if (i < a.P) {
            const Region rg = a.reg[adam_region_of(a, i)];
            p[u] = rg.partial + (i - rg.start); cnt[u] = (size_t)rg.count; sp[u] = rg.splits;
            smax = sp[u] > smax ? sp[u] : smax;
            mo[u] = a.m[i]; vo[u] = a.v[i]; to[u] = a.theta[i];
        }
    }
#pragma unroll 4
    for (int s = 0; s < smax; ++s) {
#pragma unroll
        for (int u = 0; u < UF; ++u) g[u] += s < sp[u] ? p[u][(size_t)s * cnt[u]] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < UF; ++u) {
        const int i = i0 + u * WG;
        if (i >= a.P) continue;
        const float m = a.beta1 * mo[u] + (1.0f - a.beta1) * g[u];
        const float v = a.beta2 * vo[u] + (1.0f - a.beta2) * g[u] * g[u];
        const float mh = m / a.bc1, vh = v / a.bc2;
        const float th = to[u] - a.lr * mh / (sqrtf(vh) + a.eps);
        a.grad[i] = g[u];
        a.m[i] = m;
        a.v[i] = v;
        a.theta[i] = th;
        if (a.w_bf16) {
            const uint16_t hb = bf16_bits(th);
            a.w_bf16[i] = hb;
            a.wt_bf16[transposed_index(a.net, i)] = hb;
        }
    }
}

static void launch_adam_kernel(const AdamArgs& a, hipStream_t s)
{
    int max_splits = 0;
    for (int r = 0; r < a.n_regions; ++r) max_splits = a.reg[r].splits > max_splits ? a.reg[r].splits : max_splits;
    if (max_splits <= 16 && a.P >= (1 << 18)) hipLaunchKernelGGL(adam_reduce_flat, dim3((a.P + 4 * WG - 1) / (4 * WG)), dim3(WG), 0, s, a);
    else if (a.P >= (1 << 18)) hipLaunchKernelGGL(adam_reduce, dim3((a.P + 255) / 256), dim3(ADAM_WAVES * 64), 0, s, a);
    else if (a.P < 64 * 256) hipLaunchKernelGGL(adam_reduce_narrow<1>, dim3((a.P + 63) / 64), dim3(ADAM_WAVES * 64), 0, s, a);   // less than a workgroup per unit
    else hipLaunchKernelGGL(adam_reduce_narrow<4>, dim3((a.P + 63) / 64), dim3(ADAM_WAVES * 64 / 4), 0, s, a);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_returns(anakin* h)
{
    const Layout& L = h->lay;
    ProfScope prof(h, "returns_scan");
    hipLaunchKernelGGL(returns_scan, dim3((h->B + WG - 1) / WG), dim3(WG), 0, h->stream, h->B, h->T,
                       at<const float>(h, L.tr_rew), at<const uint8_t>(h, L.tr_done), at<const float>(h, L.tr_val),
                       h->net_cfg.gamma, h->net_cfg.lambda_, at<float>(h, L.adv), at<float>(h, L.ret));
    return hipGetLastError();
}

hipError_t launch_head_grad(anakin* h)
{
    const Layout& L = h->lay;
    HeadGradArgs a;
    a.M = h->B * h->T; a.A = h->net.A; a.NH = h->net.NH; a.NHP = h->net.NHP; a.policy = h->net.policy;
    a.head = at<const float>(h, L.tr_head); a.act = at<const uint8_t>(h, L.tr_act); a.eps = at<const float>(h, L.tr_eps);
    a.adv = at<const float>(h, L.adv); a.ret = at<const float>(h, L.ret);
    a.rew = at<const float>(h, L.tr_rew); a.done = at<const uint8_t>(h, L.tr_done);
    a.dhead = at<float>(h, L.dhead); a.loss_part = at<float>(h, L.loss_part);
    a.beta = h->net_cfg.entropy_coef; a.cv = h->net_cfg.value_coef; a.inv_m = (float)(1.0 / (double)a.M);
    a.path = h->pathwise ? at<const float>(h, L.path) : nullptr;
    a.head_old = L.head_old && h->net.policy != POLICY_CATEGORICAL ? at<const float>(h, L.head_old) : nullptr;
    h->metric_blocks = h->loss_blocks;
    const SplitWeightsArgs sw = split_weights_args(h);
    ProfScope prof(h, "head_grad");
    hipLaunchKernelGGL(head_grad, dim3(h->loss_blocks + split_weights_blocks(sw)), dim3(WG), 0, h->stream, a, sw, h->loss_blocks);
    return hipGetLastError();
}

// whether returns and loss go out as one launch: the plain update of a whole unroll, and room for one block of loss
// sums per workgroup
// 16 envs per workgroup unless that leaves the second pass over the samples mostly empty (256 < 16 T < 512)
static int scan_loss_envs(const anakin* h) { return (h->T * 16 <= WG || h->T * 16 >= 2 * WG) ? 16 : 8; }
static bool scan_loss_shape(const anakin* h)
{
    const int E = scan_loss_envs(h);
    return h->B % E == 0 && h->T * E <= SL_MAXN &&
           h->B / E <= h->loss_blocks;
}

bool scan_loss_ok(const anakin* h) { return h->n_updates == 1 && !h->pathwise && !h->traj_decoupled && scan_loss_shape(h); }

static void fill_vtrace_args(anakin* h, VtraceArgs& a)
{
    const Layout& L = h->lay;
    a.B = h->B; a.T = h->T; a.A = h->net.A; a.NH = h->net.NH; a.NHP = h->net.NHP; a.policy = h->net.policy;
    a.head_old = at<const float>(h, L.tr_head); a.head_new = at<const float>(h, L.head_new); a.val_new = at<const float>(h, L.val_new);
    a.act = at<const uint8_t>(h, L.tr_act); a.eps_old = at<const float>(h, L.tr_eps);
    a.rew = at<const float>(h, L.tr_rew); a.done = at<const uint8_t>(h, L.tr_done);
    a.gamma = h->net_cfg.gamma; a.lambda = h->net_cfg.lambda_;
    a.adv = at<float>(h, L.adv); a.ret = at<float>(h, L.ret); a.eps_new = at<float>(h, L.eps_new);
}

// V-trace targets and the loss of a decoupled step: one launch where a workgroup holds its environments' whole unroll
hipError_t launch_vtrace_loss(anakin* h)
{
    if (scan_loss_shape(h)) return launch_scan_loss(h, true);
    VtraceArgs a;
    fill_vtrace_args(h, a);
    {
        ProfScope prof(h, "vtrace_ratio");
        hipLaunchKernelGGL(vtrace_ratio, dim3((unsigned)(((size_t)h->B * h->T + WG - 1) / WG)), dim3(WG), 0, h->stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    {
        ProfScope prof(h, "vtrace_scan");
        hipLaunchKernelGGL(vtrace_scan, dim3((h->B + WG - 1) / WG), dim3(WG), 0, h->stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const Layout keep = h->lay;
    h->lay.tr_head = keep.head_new; h->lay.tr_eps = keep.eps_new;        // the loss is taken at the learner's heads
    hipError_t e = launch_head_grad(h);
    h->lay = keep;
    return e;
}

hipError_t launch_scan_loss(anakin* h, bool vtrace)
{
    const Layout& L = h->lay;
    ScanLossArgs s;
    fill_vtrace_args(h, s.v);
    HeadGradArgs& a = s.g;
    a.M = h->B * h->T; a.A = h->net.A; a.NH = h->net.NH; a.NHP = h->net.NHP; a.policy = h->net.policy;
    a.head = at<const float>(h, L.tr_head); a.act = at<const uint8_t>(h, L.tr_act); a.eps = at<const float>(h, L.tr_eps);
    a.adv = nullptr; a.ret = nullptr;
    a.rew = at<const float>(h, L.tr_rew); a.done = at<const uint8_t>(h, L.tr_done);
    a.dhead = at<float>(h, L.dhead); a.loss_part = at<float>(h, L.loss_part);
    a.beta = h->net_cfg.entropy_coef; a.cv = h->net_cfg.value_coef; a.inv_m = (float)(1.0 / (double)a.M);
    a.path = nullptr; a.head_old = nullptr;
    s.B = h->B; s.T = h->T; s.E = scan_loss_envs(h); s.val = at<const float>(h, L.tr_val);
    s.gamma = h->net_cfg.gamma; s.lambda = h->net_cfg.lambda_;
    s.adv_out = at<float>(h, L.adv); s.ret_out = at<float>(h, L.ret);
    if (vtrace) { a.head = at<const float>(h, L.head_new); a.eps = at<const float>(h, L.eps_new); s.val = at<const float>(h, L.val_new); }
    s.blocks = h->B / s.E;
    h->metric_blocks = s.blocks;
    const SplitWeightsArgs sw = split_weights_args(h);
    // LDS that it does not use keeps a V-trace workgroup off the actor's units where that pays
    constexpr unsigned arrays = (6 * SL_MAXN + 16) * sizeof(float), more = 64 * 1024;
    const unsigned pad = vtrace && vtrace_off_the_actor(h, arrays + more) ? more : 0;
    if (pad) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(scan_loss<true>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)pad);
        if (e != hipSuccess) return e;
    }
    ProfScope prof(h, vtrace ? "vtrace_loss" : "scan_loss");
    hipLaunchKernelGGL(vtrace ? scan_loss<true> : scan_loss<false>, dim3(s.blocks + split_weights_blocks(sw)), dim3(WG), pad, h->stream, s, sw);
    return hipGetLastError();
}

hipError_t launch_partial_reduce(const float* src, float* dst, int count, int fan, int splits, hipStream_t s)
{
    hipLaunchKernelGGL(partial_reduce, dim3((count + WG - 1) / WG, splits), dim3(WG), 0, s, src, dst, count, fan);
    return hipGetLastError();
}

hipError_t launch_head_backward(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    HeadBwdArgs a;
    a.M = h->B * h->T; a.H = n.dims[n.L]; a.NH = n.NH; a.NHP = n.NHP;
    const int splits = h->splits[n.L], fan = h->head_fan;
    const int stage1 = splits * fan;                        // workgroups of the streaming pass
    a.rows = chunk_rows(a.M, stage1, h->quanta[n.L]);
    a.h = at<const float>(h, L.act[n.L - 1]); a.dhead = at<const float>(h, L.dhead);
    a.wh = at<const float>(h, L.w_src) + n.wh_off;
    a.dz = at<float>(h, L.dz[n.L - 1]);
    a.partial = fan > 1 ? at<float>(h, L.head_stage) : at<float>(h, L.part[n.L]);
    a.bf16 = n.bf16;
    const int groups = WG / (a.H >> 2);
    const int stride = a.H * a.NH + a.NH;
    const size_t lds = (size_t)groups * stride * sizeof(float);
    {
        ProfScope prof(h, "head_backward");
        if (a.H % 64 == 0 && a.rows % 32 == 0 && a.M % 32 == 0 && !(h->mode & ANAKIN_MODE_VALU_GEMM))
            hipLaunchKernelGGL(head_backward_mfma, dim3(stage1, (a.H + 255) / 256), dim3(WG), 0, h->stream, a);
        else
            hipLaunchKernelGGL(head_backward, dim3(stage1), dim3(WG), lds, h->stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || fan == 1) return e;
    ProfScope prof(h, "partial_reduce");
    hipLaunchKernelGGL(partial_reduce, dim3((stride + WG - 1) / WG, splits), dim3(WG), 0, h->stream,
                       at<const float>(h, L.head_stage), at<float>(h, L.part[n.L]), stride, fan);
    return hipGetLastError();
}

hipError_t launch_adam(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    AdamArgs a;
    a.P = n.P;
    int r = 0;
    for (int l = 0; l < n.L; ++l) {
        if (l == 0 && h->env.kind == ENV_MAZE && (first_layer_split(h) || first_onehot(h))) {
            // wall rows, agent rows, goal rows (zero but the last, which equals the bias gradient), bias
            const int H1 = n.dims[1], plane = h->env.rows * h->env.cols * H1;
            const int sw = first_layer_split(h) ? h->splits_w : h->splits[0];
            const float* pw = at<const float>(h, L.part[0]);
            const float* pa = pw + (size_t)plane * sw;
            const float* pg = pa + (size_t)plane * h->splits[0];
            a.reg[r++] = Region{n.w_off[0], plane, sw, pw};
            a.reg[r++] = Region{n.w_off[0] + plane, plane, h->splits[0], pa};
            a.reg[r++] = Region{n.w_off[0] + 2 * plane, plane - H1, 0, nullptr};
            a.reg[r++] = Region{n.w_off[0] + 3 * plane - H1, H1, sw, pg};
            a.reg[r++] = Region{n.b_off[0], H1, sw, pg};
            continue;
        }
        a.reg[r++] = Region{n.w_off[l], n.dims[l] * n.dims[l + 1] + n.dims[l + 1], h->splits[l], at<const float>(h, L.part[l])};
    }
    a.reg[r++] = Region{n.wh_off, n.dims[n.L] * n.NH + n.NH, h->splits[n.L], at<const float>(h, L.part[n.L])};
    a.n_regions = r;
    for (; r < MAX_ADAM_REGIONS; ++r) a.reg[r] = Region{0x7fffffff, 0, 0, nullptr};
    a.theta = at<float>(h, L.theta); a.grad = at<float>(h, L.grad); a.m = at<float>(h, L.m); a.v = at<float>(h, L.v);
    a.w_bf16 = n.bf16 ? at<uint16_t>(h, L.w_bf16) : nullptr;
    a.wt_bf16 = n.bf16 ? at<uint16_t>(h, L.wt_bf16) : nullptr;
    a.net = n;
    h->adam_t += 1;
    a.lr = h->net_cfg.lr; a.beta1 = h->net_cfg.beta1; a.beta2 = h->net_cfg.beta2; a.eps = h->net_cfg.eps;
    a.bc1 = (float)(1.0 - pow((double)h->net_cfg.beta1, (double)h->adam_t));
    a.bc2 = (float)(1.0 - pow((double)h->net_cfg.beta2, (double)h->adam_t));
    ProfScope prof(h, "adam_reduce");
    launch_adam_kernel(a, h->stream);
    return hipGetLastError();
}

// Adam on a synthetic parameter vector (measurement only): one region, one partial, P parameters laid out
// as theta | grad | m | v | partial in `base`.  Shows the kernel against the HBM roofline at a size that
// does not fit any cache; inside the real workloads P is small and the launch is latency bound.
hipError_t launch_adam_probe(float* base, int P, hipStream_t s)
{
    AdamArgs a;
    a.P = P; a.n_regions = 1;
    a.reg[0] = Region{0, P, 1, base + (size_t)4 * P};
    for (int r = 1; r < MAX_ADAM_REGIONS; ++r) a.reg[r] = Region{0x7fffffff, 0, 0, nullptr};
    a.theta = base; a.grad = base + (size_t)P; a.m = base + (size_t)2 * P; a.v = base + (size_t)3 * P;
    a.w_bf16 = nullptr; a.wt_bf16 = nullptr;
    a.net = NetShape{};
    a.lr = 3e-4f; a.beta1 = 0.9f; a.beta2 = 0.999f; a.eps = 1e-8f; a.bc1 = 0.1f; a.bc2 = 0.001f;
    launch_adam_kernel(a, s);
    return hipGetLastError();
}

}  // namespace ank
