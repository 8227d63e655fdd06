// Pathwise policy gradient through the environment (paper section 3.1: with the environment inside
// the program, the unit of T interactions can be differentiated all the way through).  For the
// pendulum with the tanh-Gaussian policy, L_path = -(1/(B T)) sum r over the stored unroll, seen as
// a function of the parameters with the noise fixed.  This kernel walks every env's unroll
// backwards with the adjoint lambda_t = dL_path/ds_t and writes dL_path/d(mu, log_sigma) per
// sample; the ordinary backward pass then turns head gradients into parameter gradients.
//
// A workgroup owns 16 or 32 envs for the whole sweep, a wavefront 32 rows of W2.  Per step: (A) every lane turns
// lambda_{t+1} of its env into the gradient of the action and of (mu, log_sigma); (B) dZ2 = relu'(h2) (Wh g), split into
// matrix operands on the way to LDS; (C) dZ1 = relu'(h1) (dZ2 W2^T) on the matrix cores, W2 on chip for the whole sweep;
// (D) g_obs = dZ1 W1^T, three dot products per env, summed over the wavefronts through LDS; (E) lambda_t from the step's
// and the reward's own derivatives plus g_obs through o = (cos, sin, thd).  Two barriers a step: the sums of (D) are
// added by every wavefront for itself, so (E), (A) and (B) need none in between.
// An episode end cuts the adjoint (the next state is a reset state).  The velocity clip is decided
// with the env step's own binary32 expression, so it agrees with what the env did.
//
// The products run on the bf16 matrix instructions with both operands as three bfloat16 terms (gemm_split.hip: six of the
// nine products, the rest below one binary32 rounding).  The sweep is serial in time and its matrix layer is most of a
// step: 32 envs, 256 x 256 take 6.1 k matrix-core cycles per compute unit that way, 16.4 k on the fp32 instruction.
// 256-256, 8192 envs, T = 32: 412 us with the fp32 instruction, 175 to 190 now: 10.1 k cycles a step, of which the products
// 6.4 k, (E) to (B) 2.7 k, (D) 0.7 k, and a clock that the bf16 instructions lower to about 1.9 GHz.  Against binary64 the
// gradient of the path term is off by 0.7 to 4.4e-7 with either (six shapes, two seeds each).
// Range (split_terms.h): W2 is taken whole at every finite value, so a weight at the type's lowest, the mask of a unit that
// never fires, gives the zero it gives in binary32.  dZ2 is whole from 2^-102 to 3.39e38: smaller entries lose their last terms,
// up to 2^-126 each (with head weights of 2^-60, as scaled layers below them may have, entries are still around 2^-90); at
// infinity or above 3.39e38 they turn the env's adjoint, and all earlier ones of its episode, into NaN, where binary32
// would carry infinities of both signs to the same end a layer further on.
#include <type_traits>
#include "split_terms.h"
#include "detmath.h"

namespace ank {

struct PathArgs {
    const float* theta; int w1_off, w2_off, wh_off;
    const float* tr_f0; const float* tr_f1; const uint8_t* tr_done; const float* tr_actf; const float* tr_eps;
    const float* tr_head; int NH, NHP;
    const float* act0; const float* act1;     // hidden activations of the unroll, [T*B][RW] each
    float* path;                              // [T*B][2]: dL_path / d(mu, log_sigma)
    int B, T;
    float w;                                  // dL_path / dr = -1 / (B T)
};

// TM envs per workgroup: 32 on v_mfma_f32_32x32x16_bf16, 16 on v_mfma_f32_16x16x32_bf16.  W2 is the A operand (rows i of a
// wavefront, reduction over j), dZ2 the B operand (columns: envs), so a lane ends up with 16 resp. 8 entries of dZ1 of one
// env and sums its share of g_obs without a shuffle.
// Operand layout: lane l feeds A[row l % TM][k 8 (l / TM) .. +7] and B[k ..][col l % TM]; accumulator register r of a tile is
// D[row 8 (r / 4) + 4 (l / 32) + r % 4][col l % 32] resp. D[row 4 (l / 16) + r][col l % 16].
template <int RW, int TM> struct PathLds {
    static constexpr int WAVES = RW / 32, KS = RW / 16;              // wavefronts; operand pieces of a wavefront's 32 rows of W2
    // a wavefront's pieces of W2 whose third term is in registers: all 3 x 16 pieces of four registers each do not fit
    static constexpr int LREG = RW == 256 ? 5 : KS;
    static constexpr int BLOCK = RW == 256 && TM == 32 ? 8 : 16;     // steps whose factors are worked out at a time
    static constexpr int DZ = 3 * (TM * RW / 8), WL = WAVES * (KS - LREG) * 64, RED = WAVES * 64, TAB = BLOCK * TM;
    static constexpr size_t bytes = (size_t)(DZ + WL + RED + 2 * TAB) * 16 + (size_t)TAB * 4 + (size_t)5 * RW * 4;
};

// the sum of x over the lanes of an env (TM lanes apart), in all of them
template <int TM>
__device__ __forceinline__ float env_sum(float x)
{
    typedef uint32_t u2_p __attribute__((ext_vector_type(2)));
    if (TM == 16) {
        const u2_p s = __builtin_bit_cast(u2_p, __builtin_amdgcn_permlane16_swap(bits_from_f(x), bits_from_f(x), false, false));
        x = f_from_bits(s[0]) + f_from_bits(s[1]);
    }
    const u2_p s = __builtin_bit_cast(u2_p, __builtin_amdgcn_permlane32_swap(bits_from_f(x), bits_from_f(x), false, false));
    return f_from_bits(s[0]) + f_from_bits(s[1]);
}

template <int RW, int TM>
__global__ __launch_bounds__(2 * RW) void pathwise_sweep(const PathArgs a)
{
    typedef PathLds<RW, TM> L;
    constexpr int BLOCK = L::BLOCK, NT = 2 * RW, KS = L::KS, WAVES = L::WAVES, LREG = L::LREG;
    constexpr int IT = 32 / TM, NK = KS / IT;                          // tiles of a wavefront's rows; k steps of 16 resp. 32
    constexpr int ROWS = TM == 32 ? 16 : 4;                            // accumulator registers of a tile
    constexpr int NP = TM / 16;                                        // pieces of dZ2 a lane forms
    constexpr int NH1 = IT * ROWS / 4, NLD = NH1 + 2 * NP;             // loads of h1 and of both layers per step
    extern __shared__ float4 smem_p[];
    u4v_s* dz = reinterpret_cast<u4v_s*>(smem_p);                      // [3 terms][RW / 8 groups of j][TM] operand pieces
    u4v_s* wl = dz + L::DZ;                                            // third terms of W2 beyond LREG, [wave][piece][lane]
    f4v_s* red = reinterpret_cast<f4v_s*>(wl + L::WL);                 // [wave][lane] shares of g_obs
    f4v_s* tab = red + L::RED;                                         // [BLOCK][TM][2]: factors of a step
    uint32_t* flags = reinterpret_cast<uint32_t*>(tab + 2 * L::TAB);   // [BLOCK][TM]: 1 episode end, 2 velocity clipped
    float* w1s = reinterpret_cast<float*>(flags + L::TAB);             // first-layer matrix, [3][RW]
    float* whs = w1s + 3 * RW;                                         // head matrix columns of mu and log_sigma, [2][RW]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane % TM, kq = lane / TM;
    const int b0 = blockIdx.x * TM, B = a.B, T = a.T;

    for (int i = tid; i < 3 * RW; i += NT) w1s[i] = a.theta[a.w1_off + i];
    for (int i = tid; i < 2 * RW; i += NT) { const int c = i / RW, k = i - c * RW; whs[i] = a.theta[a.wh_off + k * a.NH + c]; }
    // piece p of the wavefront's rows: tile p % IT, k step p / IT
    u4v_s w0[KS], w1[KS], w2[LREG];
    {
        const float* W2 = a.theta + a.w2_off;
#pragma unroll
        for (int p = 0; p < KS; ++p) {
            const float* src = W2 + (size_t)(wave * 32 + (p % IT) * TM + m) * RW + (p / IT) * (16 * IT) + 8 * kq;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = src[e];
            u4v_s t[3];
            split_terms<true>(x, t);
            w0[p] = t[0]; w1[p] = t[1];
            if (p < LREG) w2[p < LREG ? p : 0] = t[2];
            else wl[(wave * (KS - LREG) + (p < LREG ? 0 : p - LREG)) * 64 + lane] = t[2];
        }
    }
    // The lane's dZ2 pieces: env m, reduction indices j0 .. j0 + 7 (and j0 + 16 ..): what it stores is what some lane reads as
    // an operand, consecutive lanes side by side.  h2 of a step is asked for a step ahead, h1 ahead of the step's products.
    const int g0 = wave * 4 + kq;                                      // group of eight j; TM == 32: and g0 + 2
    // Both go between the products' MFMAs, a load at a time: 32 rows per load keep the address path busy for longer than a
    // phase of their own would hide.
    f4v_s h2v[NP][2], h1v[IT][ROWS / 4];
    auto fetch_h2 = [&](int t, int n) {
        h2v[n / 2][n % 2] = *reinterpret_cast<const f4v_s*>(a.act1 + ((size_t)t * B + b0 + m) * RW + 8 * g0 + 16 * (n / 2) + 4 * (n % 2));
    };
    auto fetch_h1 = [&](int t, int n) {
        h1v[n / (ROWS / 4)][n % (ROWS / 4)] = *reinterpret_cast<const f4v_s*>(a.act0 + ((size_t)t * B + b0 + m) * RW + wave * 32 + 4 * kq + 16 * (n / (ROWS / 4)) + 8 * (n % (ROWS / 4)));
    };
    // factors of steps t0 .. t0 + n - 1 that need no adjoint
    const float dt = 0x1.99999ap-5f;
    auto factors = [&](int t0, int n) {
        for (int u = tid; u < n * TM; u += NT) {
            const int mm = u % TM;
            const size_t i = (size_t)(t0 + u / TM) * B + b0 + mm;
            const float th = a.tr_f0[i], thd = a.tr_f1[i], act = a.tr_actf[i], eps = a.tr_eps[i];
            const float ls = a.tr_head[i * a.NHP + 1];
            const bool clamped = ls < -5.0f || ls > 2.0f;
            const float sigma = det_exp(fminf(fmaxf(ls, -5.0f), 2.0f));
            float f = 2.0f * act;
            f = f < -2.0f ? -2.0f : f;
            f = f > 2.0f ? 2.0f : f;
            float sn, cs;
            det_sincos(th, sn, cs);
            const float pre = fmaf(fmaf(15.0f, sn, 3.0f * f), dt, thd);          // the env step's expression
            const bool clipped = pre < -8.0f || pre > 8.0f;
            f4v_s v0 = {15.0f * cs, a.w * (-2.0f * th), a.w * (-2.0f * 0x1.99999ap-4f * thd), a.w * (-2.0f * 0x1.0624dep-10f * f)};
            f4v_s v1 = {1.0f - act * act, clamped ? 0.0f : sigma * eps, sn, cs};
            tab[2 * u] = v0; tab[2 * u + 1] = v1;
            flags[u] = (a.tr_done[i] ? 1u : 0u) | (clipped ? 2u : 0u) | (clamped ? 4u : 0u);
        }
    };
#pragma unroll
    for (int n = 0; n < 2 * NP; ++n) fetch_h2(T - 1, n);
    float lam_th = 0.0f, lam_thd = 0.0f;
    int t0 = T;                                                        // first step of the block in the table
    f4v_s f0, f1;
    uint32_t ff;
    constexpr bool AHEAD = L::BLOCK == 16;                             // a step's factors a step ahead, where registers allow
    auto read_factors = [&](int t) { const int u = (t - t0) * TM + m; f0 = tab[2 * u]; f1 = tab[2 * u + 1]; ff = flags[u]; };
    for (int t = T - 1; t >= 0; --t) {
        if (t < t0) {
            __syncthreads();                                           // (the table's readers are done)
            const int n = t + 1 < BLOCK ? t + 1 : BLOCK;
            t0 = t + 1 - n;
            factors(t0, n);
            __syncthreads();
            if (AHEAD) read_factors(t);
        }
        if (!AHEAD) read_factors(t);
        // ---- (A) ------------------------------------------------------------------
        const f4v_s v0 = f0, v1 = f1;
        const uint32_t fl = ff;
        if (fl & 1u) { lam_th = 0.0f; lam_thd = 0.0f; }
        const float g_nthd = fmaf(dt, lam_th, lam_thd);
        const float g_pre = (fl & 2u) ? 0.0f : g_nthd;
        const float g_th = lam_th + g_pre * dt * v0[0] + v0[1];
        const float g_thd = g_pre + v0[2];
        const float g_u = g_pre * dt * 3.0f + v0[3];
        const float g_z = 2.0f * g_u * v1[0];
        const float g_ls = (fl & 4u) ? 0.0f : g_z * v1[1];
        if (wave == 0 && kq == 0) *reinterpret_cast<float2*>(a.path + ((size_t)t * B + b0 + m) * 2) = make_float2(g_z, g_ls);
        // ---- (B) dZ2[m][j] = (h2 > 0) (Wh[j][mu] g_mu + Wh[j][ls] g_ls) ---------------
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int j = 8 * g0 + 16 * q;
            float d[8];
#pragma unroll
            for (int e4 = 0; e4 < 2; ++e4) {
                const f4v_s wa = *reinterpret_cast<const f4v_s*>(whs + j + 4 * e4), wb = *reinterpret_cast<const f4v_s*>(whs + RW + j + 4 * e4);
#pragma unroll
                for (int e = 0; e < 4; ++e) d[4 * e4 + e] = h2v[q][e4][e] > 0.0f ? fmaf(wb[e], g_ls, wa[e] * g_z) : 0.0f;
            }
            u4v_s tt[3];
            split_terms(d, tt);
#pragma unroll
            for (int k = 0; k < 3; ++k) dz[(k * (RW / 8) + g0 + 2 * q) * TM + m] = tt[k];
        }
        __syncthreads();
        // ---- (C) dZ1 = (h1 > 0) (dZ2 W2^T) -------------------------------------------
        typedef typename std::conditional<TM == 32, f16v_s, f4v_s>::type acc_t;
        acc_t acc[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) acc[i][r] = 0.0f;
        {
            const u4v_s* xp = dz + kq * TM + m;
            const u4v_s* wp = wl + wave * (KS - LREG) * 64 + lane;
            // the next step's operands are read as soon as this step's last MFMA on them is issued: one register set for
            // all but the first terms of dZ2, which the last MFMA of a step and the second of the next both need
            u4v_s b0[2], b1, b2, wv[IT];
            auto read_x = [&](int k, int ks) { return xp[(k * (RW / 8) + ks * 2 * IT) * TM]; };
            auto read_w = [&](int ks) {
#pragma unroll
                for (int i = 0; i < IT; ++i)
                    if (ks * IT + i >= LREG) wv[i] = wp[(ks * IT + i - LREG) * 64];
            };
            b2 = read_x(2, 0); b0[0] = read_x(0, 0); b1 = read_x(1, 0);
            read_w(0);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                const bool more = ks + 1 < NK;
#pragma unroll
                for (int n = NLD * ks / NK; n < NLD * (ks + 1) / NK; ++n) {
                    if (n < NH1) fetch_h1(t, n);
                    else fetch_h2(t > 0 ? t - 1 : 0, n - NH1);
                }
#pragma unroll
                for (int pr = 0; pr < 6; ++pr) {
                    constexpr int PW[6] = {0, 2, 1, 1, 0, 0}, PX[6] = {2, 0, 1, 0, 1, 0};   // terms of W2 and of dZ2, smallest products first
                    const u4v_s xt = PX[pr] == 0 ? b0[ks & 1] : PX[pr] == 1 ? b1 : b2;
#pragma unroll
                    for (int i = 0; i < IT; ++i) {
                        const int p = ks * IT + i;
                        const u4v_s wt = PW[pr] == 0 ? w0[p] : PW[pr] == 1 ? w1[p] : p < LREG ? w2[p < LREG ? p : 0] : wv[i];
                        if constexpr (TM == 32) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8_s, wt), __builtin_bit_cast(bf8_s, xt), acc[i], 0, 0, 0);
                        else acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_s, wt), __builtin_bit_cast(bf8_s, xt), acc[i], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (more && pr == 0) { b2 = read_x(2, ks + 1); b0[(ks + 1) & 1] = read_x(0, ks + 1); }
                    if (more && pr == 1) read_w(ks + 1);
                    if (more && pr == 4) b1 = read_x(1, ks + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // ---- (D) g_obs[m][c] = sum_i dZ1[m][i] W1[c][i] ----------------------------------
        float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int i = 0; i < IT; ++i)
#pragma unroll
            for (int g = 0; g < ROWS / 4; ++g) {
                const float* w = w1s + wave * 32 + i * 16 + 8 * g + 4 * kq;
                const f4v_s x0 = *reinterpret_cast<const f4v_s*>(w), x1 = *reinterpret_cast<const f4v_s*>(w + RW), x2 = *reinterpret_cast<const f4v_s*>(w + 2 * RW);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = h1v[i][g][e] > 0.0f ? acc[i][4 * g + e] : 0.0f;
                    s0 = fmaf(d, x0[e], s0); s1 = fmaf(d, x1[e], s1); s2 = fmaf(d, x2[e], s2);
                }
            }
        f4v_s sv = {s0, s1, s2, 0.0f};
        red[wave * 64 + lane] = sv;
        const float sn = v1[2], cs = v1[3];
        if (AHEAD && t > t0) read_factors(t - 1);
        __syncthreads();
        // ---- (E) lambda_t, through o = (cos th, sin th, thd) -----------------------------
        f4v_s o = red[lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) o += red[w * 64 + lane];
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = env_sum<TM>(o[c]);
        lam_th = g_th - sn * o[0] + cs * o[1];
        lam_thd = g_thd + o[2];
    }
}

bool pathwise_ok(const anakin* h)
{
    const NetShape& n = h->net;
    if (h->env.kind != ENV_PENDULUM || n.policy != POLICY_TANH_GAUSSIAN || n.bf16 || n.L != 2 || n.dims[1] != n.dims[2]) return false;
    if (n.dims[1] != 64 && n.dims[1] != 128 && n.dims[1] != 256) return false;
    return h->B % 16 == 0;
}

hipError_t launch_pathwise(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    PathArgs a;
    a.theta = at<const float>(h, L.w_src); a.w1_off = n.w_off[0]; a.w2_off = n.w_off[1]; a.wh_off = n.wh_off;
    a.tr_f0 = at<const float>(h, L.tr_f0); a.tr_f1 = at<const float>(h, L.tr_f1); a.tr_done = at<const uint8_t>(h, L.tr_done);
    a.tr_actf = at<const float>(h, L.tr_actf); a.tr_eps = at<const float>(h, L.tr_eps);
    a.tr_head = at<const float>(h, L.tr_head); a.NH = n.NH; a.NHP = n.NHP;
    a.act0 = at<const float>(h, L.act[0]); a.act1 = at<const float>(h, L.act[1]);
    a.path = at<float>(h, L.path);
    a.B = h->B; a.T = h->T; a.w = (float)(-1.0 / ((double)h->B * (double)h->T));
    ProfScope prof(h, "pathwise_sweep");
    // 32 envs per workgroup where 16 would not all be on the chip at once (one such workgroup per compute unit for 256 units
    // per layer, two for 128).  T = 16, 16 / 32 envs: 256-256 with 4096 envs 66.8 / 93.5 us, 8192 125 / 106, 65536 901 / 772;
    // 128-128 with 8192 envs 38.6 / 46.4, 16384 85.3 / 76.8, 65536 341 / 326; 64-64 with 16384 envs 35.5 / 38.5, 65536 161 / 159
    const int RW = n.dims[1];
    const bool m32 = RW >= 128 && h->B % 32 == 0 && h->B / 16 > 65536 / RW;
    auto go = [&](auto kern, int TM, size_t lds) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(h->B / TM), dim3(2 * RW), lds, h->stream, a);
        return hipGetLastError();
    };
    switch (RW) {
        case 64:  return go(pathwise_sweep<64, 16>, 16, PathLds<64, 16>::bytes);
        case 128: return m32 ? go(pathwise_sweep<128, 32>, 32, PathLds<128, 32>::bytes) : go(pathwise_sweep<128, 16>, 16, PathLds<128, 16>::bytes);
        default:  return m32 ? go(pathwise_sweep<256, 32>, 32, PathLds<256, 32>::bytes) : go(pathwise_sweep<256, 16>, 16, PathLds<256, 16>::bytes);
    }
}

}  // namespace ank
