// The whole update of a small Catch agent in ONE launch (paper section 3.1: the unit of T interactions and one
// parameter update is a single device program; for a net and an unroll this small the seven kernels of the
// general update do a few microseconds of work each and the step is bound by their launches).
//
// Shape: Catch, fp32, two hidden layers of 64 units, three actions + value; at most 16 workgroups, each owning
// E envs for all T steps (R = E T <= 112 samples).  Nothing depends on another workgroup's samples until the
// gradient is summed, so every workgroup runs the whole chain on its own rows:
//   scan       returns and advantages of its envs (returns_scan's recursion)
//   loss       loss terms and head gradients of its samples (head_grad's arithmetic)
//   dZ2, dWh   from the stored h2 and the head matrix
//   dZ1        = relu'(h1) (dZ2 W2^T), W2 in registers
//   dW2, db2   = h1^T dZ2
//   dW1, db1   = X^T dZ1 with the 0/1 board X
// and writes one partial gradient.  Then the workgroups wait for each other at an integer counter (ordinary vector
// atomics; device-scope fences around them), and each adds the partials of its slice of the parameters in ascending
// workgroup order -- so the bytes do not depend on who arrived when -- and applies Adam to it.
//
// What the time is (64 environments, T = 20: 16 workgroups of 80 samples, 18.2 us; cycles of one workgroup, 38.5 k in all):
// first loads and their way into LDS 4.0 k, scan 2.8 k, loss 1.4 k, dZ2 2.8 k, dZ1 4.5 k, dW2 4.2 k (matrix-core time 2.6 k
// each), sums over lanes 1.9 k, dW1 4.7 k, biases 0.7 k, publishing the partial 2.5 k, rendezvous 4.0 k, Adam 4.2 k, departure
// 0.8 k: a chain of short phases, a third of it round trips to memory, on 16 of 256 compute units.  26.6 us before: rows by
// 16-byte pieces and one multiplication for a sample's place (loads of a word each, a division for each, 11.6 k), tiles of
// 16 x 16 so that all four wavefronts have the same work (32-row tiles: the third of them cost as much as the first two),
// dZ2 and dWh on the matrix cores, an entry of the 0/1 board worked out once for all 64 columns (compares through the scalar
// unit in front of every product: 7.6 k).
#include <type_traits>
#include "internal.h"
#include "loss.h"

namespace ank {

constexpr int SF_WG = 256;
constexpr int SF_H = 64;
constexpr int SF_MAX_WG = 16;
constexpr int SF_MAX_R = 112;

struct SmallFusedArgs {
    int B, T, D, E, n_wg, P;
    uint32_t inv_E;            // 65536 / E, rounded up: (r inv_E) >> 16 is r / E for r < 128
    EnvDims env;
    NetShape net;
    const float* w;            // parameters the unroll was acted with
    const uint32_t* s0; const uint8_t* act; const float* rew; const uint8_t* done; const float* val; const float* head;
    const float* h1; const float* h2;       // [B*T][64] stored activations
    float* adv; float* ret;
    float* part;               // [n_wg][P]
    float* loss_part;          // [n_wg][8]
    unsigned* counter;         // [0] arrivals, [1] departures: both zero between launches
    int max_spin;              // bound on the polls of the rendezvous
    float* theta; float* grad; float* m; float* v;
    float gamma, lambda, beta, cv, inv_m;
    float lr, beta1, beta2, eps, bc1, bc2;
};

typedef float f4_s __attribute__((ext_vector_type(4)));

// sum over the 64 lanes of a wavefront, same value in every lane, fixed order
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__global__ __launch_bounds__(SF_WG) void learn_small_fused(const SmallFusedArgs a)
{
    extern __shared__ float lds[];
    constexpr int H = SF_H, LD = H + 1;                  // row stride 65: a column walk touches every bank once
    const int B = a.B, T = a.T, D = a.D, E = a.E, R = E * T, R16 = (R + 15) & ~15;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kq = lane >> 4;
    const int b0 = blockIdx.x * E;
    float* W2s = lds;                                    // [64][LD]
    float* dhk = W2s + H * LD;                           // [4][R16] head gradients, one array per head output, zero from R on
    float* advs = dhk + 4 * R16;                         // [R16]
    float* rets = advs + R16;                            // [R16]
    float* rews = rets + R16;                            // [R16] rewards, then (scan) discounts
    float* vals = rews + R16;                            // [R16 + E rounded up to 4] values of the T + 1 rows
    const int Ep4 = (E + 3) & ~3;
    float* cells = vals + R16 + Ep4;                     // [2][R16] the ball's and the paddle's cell, no cell from R on
    float* dz1s = cells + 2 * R16;                       // [R16][LD]
    float* red = dz1s + R16 * LD;                        // [4 waves][16] + [2][256] db1 and db2 partials
    float* un = red + 64 + 2 * SF_WG;                    // dz2s [R16][LD], h1s [R16][LD]
    float* dz2s = un;
    float* h1s = un + R16 * LD;
    const NetShape& n = a.net;
    auto sample = [&](int r) { const int t = (int)((uint32_t)r * a.inv_E >> 16); return (size_t)t * B + b0 + (r - t * E); };

    // ---- everything this workgroup reads from memory is requested here, before anything is computed: the phases
    //      below then depend on LDS and registers only, not on one round trip to memory after another ----
    const int piece = tid & 15, row0 = tid >> 4;          // 16 bytes of every 16th row
    f4_s w2v[H / 16];
#pragma unroll
    for (int u = 0; u < H / 16; ++u) w2v[u] = *reinterpret_cast<const f4_s*>(a.w + n.w_off[1] + (row0 + 16 * u) * H + 4 * piece);
    const int col = 16 * wave + l16;                     // this lane's unit in the products
    const float wh = a.w[n.wh_off + col * 4 + kq];
    // per-sample records: lane r < R (R <= 112 < 256)
    float4 hv4 = make_float4(0, 0, 0, 0);
    int my_act = 0; uint32_t my_s0 = 0u; float my_rew = 0.0f, my_val = 0.0f, boot = 0.0f; bool my_done = false;
    if (tid < R) {
        const size_t i = sample(tid);
        hv4 = *reinterpret_cast<const float4*>(a.head + i * 4);
        my_act = (int)a.act[i]; my_s0 = a.s0[i]; my_rew = a.rew[i]; my_done = a.done[i] != 0; my_val = a.val[i];
    }
    if (tid < E) boot = a.val[(size_t)T * B + b0 + tid];
    // stored activations of the workgroup's rows: h1 as it is, h2 parked where dZ2 will go; rows from R up to the next
    // multiple of 16 are zero (they are reduction steps of the dW products)
    constexpr int NB = SF_MAX_R / 16;
    f4_s h2v[NB], h1v[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int r = row0 + 16 * u;
        const size_t i = sample(r < R ? r : R - 1) * H + 4 * piece;
        h2v[u] = *reinterpret_cast<const f4_s*>(a.h2 + i);
        h1v[u] = *reinterpret_cast<const f4_s*>(a.h1 + i);
    }
    __builtin_amdgcn_sched_barrier(0);
    // ... and only now the first use of any of them
#pragma unroll
    for (int u = 0; u < H / 16; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) W2s[(row0 + 16 * u) * LD + 4 * piece + e] = w2v[u][e];
    if (tid < R) {
        rews[tid] = my_rew;
        vals[tid] = my_val;
        advs[tid] = my_done ? 0.0f : a.gamma;                // discount of the step, for the scan
    }
    if (tid < E) vals[R + tid] = boot;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int r = row0 + 16 * u;
        if (16 * u < R) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                h1s[r * LD + 4 * piece + e] = r < R ? h1v[u][e] : 0.0f;
                dz2s[r * LD + 4 * piece + e] = r < R ? h2v[u][e] : 0.0f;
            }
        }
    }
    __syncthreads();
    // ---- scan: one lane per env, all operands in LDS (advs holds the discounts until it is overwritten) ----
    if (tid < E) {
        const float oml = 1.0f - a.lambda;
        float G = vals[R + tid], vnext = G;
        // the operands of eight (at the end, four) steps are read before the first of them is used: one LDS round trip
        auto steps = [&](auto n8, int t1) {
            constexpr int N = decltype(n8)::value;
            float rr[N], vv[N], dd[N];
#pragma unroll
            for (int u = 0; u < N; ++u) { const int r = (t1 - 1 - u) * E + tid; rr[u] = rews[r]; vv[u] = vals[r]; dd[u] = advs[r]; }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int r = (t1 - 1 - u) * E + tid;
                const float mix = fmaf(a.lambda, G, oml * vnext);
                G = fmaf(dd[u], mix, rr[u]);
                rets[r] = G; advs[r] = G - vv[u];
                vnext = vv[u];
            }
        };
        int t1 = T;
        for (; t1 >= 8; t1 -= 8) steps(std::integral_constant<int, 8>(), t1);
        if (t1 >= 4) { steps(std::integral_constant<int, 4>(), t1); t1 -= 4; }
        for (; t1 > 0; --t1) steps(std::integral_constant<int, 1>(), t1);
    }
    __syncthreads();
    // ---- loss terms and head gradients: lane r < R ----
    float sums[5] = {0, 0, 0, 0, 0}, dbh[4] = {0, 0, 0, 0};
    if (tid < R) {
        const size_t i = sample(tid);
        a.ret[i] = rets[tid]; a.adv[i] = advs[tid];
        float d[4], lp_term, v_term, e_term;
        catch_head_grad(hv4, my_act, advs[tid], rets[tid], a.beta, a.cv, a.inv_m, d, lp_term, v_term, e_term);
        sums[0] = lp_term; sums[1] = v_term; sums[2] = e_term; sums[3] = my_rew; sums[4] = my_done ? 1.0f : 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) { dbh[k] = d[k]; dhk[k * R16 + tid] = d[k]; }
        int bc, pc;
        catch_obs_cells(a.env, my_s0, bc, pc);
        cells[tid] = (float)bc; cells[R16 + tid] = (float)pc;
    } else if (tid < R16) {
        cells[tid] = -8.0f; cells[R16 + tid] = -8.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dhk[k * R16 + tid] = 0.0f;
    }
    __syncthreads();
    // ---- dZ2 (in place of the parked h2) and the head-matrix sums, on the matrix cores (v_mfma_f32_16x16x4_f32: lane
    //      (l16, kq) feeds A[row l16][k kq] and B[k kq][col l16], accumulator register r is D[row 4 kq + r][col l16]; it
    //      chains at full rate).  Wavefront w has the units 16 w .. in this product and the next three, so that every
    //      wavefront has the same work.  dZ2 has a reduction of the four heads; for dWh the h2 that mask it are the B
    //      operand, register r the samples 4 kq + r, and the heads are rows 0 to 3 (the others repeat them, unused) ----
    f4_s dwh = {0.0f, 0.0f, 0.0f, 0.0f};
    float db2 = 0.0f;
#pragma unroll 1
    for (int rt = 0; rt < R16; rt += 16) {
        const float d = dhk[kq * R16 + rt + l16];
        const f4_s dt = *reinterpret_cast<const f4_s*>(dhk + (l16 & 3) * R16 + rt + 4 * kq);
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = dz2s[(rt + 4 * kq + r) * LD + col];
        const f4_s dz = __builtin_amdgcn_mfma_f32_16x16x4f32(d, wh, f4_s{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) dwh = __builtin_amdgcn_mfma_f32_16x16x4f32(dt[r], h[r], dwh, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float o = h[r] > 0.0f ? dz[r] : 0.0f;                                // (rows from R on have h2 = 0)
            dz2s[(rt + 4 * kq + r) * LD + col] = o;
            db2 += o;
        }
    }
    __syncthreads();
    float* out = a.part + (size_t)blockIdx.x * a.P;
    // ---- dZ1 = relu'(h1) (dZ2 W2^T), a wavefront's 16 x 64 block of W2 in registers; the operands of the next 16 rows are
    //      read between the products (in all three loops that follow) ----
    float db1 = 0.0f;
    {
        float w2k[H / 4], av[H / 4];
#pragma unroll
        for (int q = 0; q < H / 4; ++q) w2k[q] = W2s[col * LD + 4 * q + kq];          // B[k = 4q + kq][col] = W2[col][k]
#pragma unroll
        for (int q = 0; q < H / 4; ++q) av[q] = dz2s[l16 * LD + 4 * q + kq];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int rt = 16 * u;
            if (rt >= R16) break;
            float hm[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) hm[r] = h1s[(rt + 4 * kq + r) * LD + col];
            const float* next = dz2s + ((rt + 16 < R16 ? rt + 16 : 0) + l16) * LD + kq;
            f4_s acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int q = 0; q < H / 4; ++q) {
                const float x = av[q];
                av[q] = next[4 * q];
                __builtin_amdgcn_sched_barrier(0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w2k[q], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float dz = hm[r] > 0.0f ? acc[r] : 0.0f;                        // (rows from R on have h1 = 0)
                dz1s[(rt + 4 * kq + r) * LD + col] = dz;
                db1 += dz;
            }
        }
    }
    // ---- dW2 = h1^T dZ2: the reduction runs over the rows of the workgroup (from R on they are zero) ----
    {
        f4_s acc[4];
        float av[4][4], bv[4];
        auto operands = [&](int r0, int q) {
            const int at = (r0 + 4 * q + kq) * LD;
            bv[q] = dz2s[at + col];
#pragma unroll
            for (int it = 0; it < 4; ++it) av[q][it] = h1s[at + 16 * it + l16];
        };
#pragma unroll
        for (int it = 0; it < 4; ++it) acc[it] = f4_s{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < 4; ++q) operands(0, q);
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int r0 = 16 * u;
            if (r0 >= R16) break;
            const int next = r0 + 16 < R16 ? r0 + 16 : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float x[4];
                const float b = bv[q];
#pragma unroll
                for (int it = 0; it < 4; ++it) x[it] = av[q][it];
                operands(next, q);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int it = 0; it < 4; ++it) acc[it] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[it], b, acc[it], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[n.w_off[1] + (16 * it + 4 * kq + r) * H + col] = acc[it][r];
    }
    // sums over the lanes of every wavefront (butterfly, fixed order), one row of `red` per wavefront
    {
        float q9[9] = {dbh[0], dbh[1], dbh[2], dbh[3], sums[0], sums[1], sums[2], sums[3], sums[4]};
#pragma unroll
        for (int k = 0; k < 9; ++k) q9[k] = wave_sum(q9[k]);
        if (lane < 9) {
            float v = q9[0];
#pragma unroll
            for (int k = 1; k < 9; ++k) if (lane == k) v = q9[k];
            red[wave * 16 + lane] = v;
        }
        red[64 + tid] = db1;
    }
    red[64 + SF_WG + tid] = db2;
    if (kq == 0) *reinterpret_cast<f4_s*>(out + n.wh_off + col * 4) = dwh;
    __syncthreads();                                     // dz1s and red are complete
    // ---- dW1 = X^T dZ1 with X the 0/1 board (two ones per row), on the matrix cores: wavefront w owns the board cells
    //      16 w .. (at most 64 here), so that an entry of X is worked out once and used for all 64 columns; a product with a
    //      one is exact ----
    if (16 * wave < D) {
        f4_s acc[4];
        float c0[4], c1[4], bv[4][4];
        auto operands = [&](int r0, int q) {
            const int r = r0 + 4 * q + kq;
            c0[q] = cells[r]; c1[q] = cells[R16 + r];
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) bv[q][jt] = dz1s[r * LD + 16 * jt + l16];
        };
        const float me = (float)col;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) acc[jt] = f4_s{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < 4; ++q) operands(0, q);
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int r0 = 16 * u;
            if (r0 >= R16) break;
            const int next = r0 + 16 < R16 ? r0 + 16 : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // 1 where the row's ball or paddle is in this cell, else 0, without a trip through the scalar unit: 1 - the
                // distance to the nearer of the two, clamped
                const float near = fminf(fabsf(c0[q] - me), fabsf(c1[q] - me)), x = __builtin_amdgcn_fmed3f(1.0f - near, 0.0f, 1.0f);
                float b[4];
#pragma unroll
                for (int jt = 0; jt < 4; ++jt) b[jt] = bv[q][jt];
                operands(next, q);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int jt = 0; jt < 4; ++jt) acc[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[jt], acc[jt], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = 16 * wave + 4 * kq + r;
            if (c < D) {
#pragma unroll
                for (int jt = 0; jt < 4; ++jt) out[n.w_off[0] + c * H + 16 * jt + l16] = acc[jt][r];
            }
        }
    }
    if (tid >= 128 && tid < 128 + H) {
        const int c = tid - 128;
        float sb = 0.0f;
        for (int hh = 0; hh < 4; ++hh) sb += red[64 + SF_WG + (c >> 4) * 64 + hh * 16 + (c & 15)];
        out[n.b_off[1] + c] = sb;
    }
    if (tid < H) {
        // db1 of column tid: the four lanes of its wavefront that have it, ascending
        float sb = 0.0f;
        for (int hh = 0; hh < 4; ++hh) sb += red[64 + (tid >> 4) * 64 + hh * 16 + (tid & 15)];
        out[n.b_off[0] + tid] = sb;
    }
    if (tid >= 64 && tid < 73) {
        const int q = tid - 64;
        const float s = ((red[q] + red[16 + q]) + red[32 + q]) + red[48 + q];
        if (q < 4) out[n.bh_off + q] = s;
        else a.loss_part[(size_t)blockIdx.x * 8 + (q - 4)] = s;
    }
    if (tid >= 73 && tid < 76) a.loss_part[(size_t)blockIdx.x * 8 + tid - 68] = 0.0f;
    // ---- rendezvous.  Every workgroup publishes its partial device-wide, takes a ticket, and waits until all
    //      n_wg tickets are out (all workgroups are resident: there are at most 16, one per compute unit).  The wait
    //      is bounded; a workgroup that gives up marks the metrics not-finite and leaves the parameters alone. ----
    __shared__ int go;
    const int per = (((a.P + a.n_wg - 1) / a.n_wg) + 3) & ~3, p = blockIdx.x * per + tid * 4;
    const bool mine = tid * 4 < per && p < a.P;              // P % 4 == 0: whole groups of four
    f4_s mo = {}, vo = {}, to = {};
    if (mine) { mo = *reinterpret_cast<const f4_s*>(a.m + p); vo = *reinterpret_cast<const f4_s*>(a.v + p); to = *reinterpret_cast<const f4_s*>(a.theta + p); }
    __threadfence();
    __syncthreads();
    if (tid == 0) {
        atomicAdd(a.counter, 1u);
        int ok = 0;
        for (int spin = 0; spin < a.max_spin; ++spin) {
            if (__hip_atomic_load(a.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (unsigned)a.n_wg) { ok = 1; break; }
            __builtin_amdgcn_s_sleep(4);
        }
        go = ok;
    }
    __syncthreads();
    if (go) {
        __threadfence();                                 // the other workgroups' partials, published before their tickets
        // ---- Adam on this workgroup's slice of the parameters: partials added in ascending workgroup order ----
        if (mine) {
            f4_s pw[SF_MAX_WG];
#pragma unroll
            for (int w = 0; w < SF_MAX_WG; ++w)
                pw[w] = w < a.n_wg ? *reinterpret_cast<const f4_s*>(a.part + (size_t)w * a.P + p) : f4_s{0.0f, 0.0f, 0.0f, 0.0f};
            f4_s gs = {0.0f, 0.0f, 0.0f, 0.0f}, mn, vn, tn;
#pragma unroll
            for (int w = 0; w < SF_MAX_WG; ++w) gs += pw[w];         // absent workgroups add zero
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float m = a.beta1 * mo[c] + (1.0f - a.beta1) * gs[c];
                const float v = a.beta2 * vo[c] + (1.0f - a.beta2) * gs[c] * gs[c];
                const float mh = m / a.bc1, vh = v / a.bc2;
                mn[c] = m; vn[c] = v; tn[c] = to[c] - a.lr * mh / (sqrtf(vh) + a.eps);
            }
            *reinterpret_cast<f4_s*>(a.grad + p) = gs;
            *reinterpret_cast<f4_s*>(a.m + p) = mn;
            *reinterpret_cast<f4_s*>(a.v + p) = vn;
            *reinterpret_cast<f4_s*>(a.theta + p) = tn;
        }
    } else if (tid == 0) {
        a.loss_part[(size_t)blockIdx.x * 8] = __builtin_nanf("");
    }
    // ---- departure: the last workgroup to leave puts both counters back to zero for the next launch ----
    __syncthreads();
    if (tid == 0) {
        const unsigned d = atomicAdd(a.counter + 1, 1u);
        if (d == (unsigned)a.n_wg - 1u) { a.counter[1] = 0u; a.counter[0] = 0u; }
    }
}

// envs per workgroup for the single-launch update, 0 when the shape does not qualify
int small_fused_envs(const EnvDims& ed, const NetShape& ns, int B, int T)
{
    if (ed.kind != ENV_CATCH || ns.bf16 || ns.L != 2 || ns.dims[1] != SF_H || ns.dims[2] != SF_H || ns.NH != 4) return 0;
    if (ns.dims[0] > 64) return 0;                       // the board's cells are four 16-row tiles of the dW1 product, one to a wavefront
    for (int E = (B + SF_MAX_WG - 1) / SF_MAX_WG; E <= B && E * T <= SF_MAX_R; ++E)
        if (B % E == 0) return E;
    return 0;
}

size_t small_fused_part_bytes(const EnvDims& ed, const NetShape& ns, int B, int T)
{
    const int E = small_fused_envs(ed, ns, B, T);
    return E ? (size_t)(B / E) * ns.P * sizeof(float) : 0;
}

bool small_fused_ok(const anakin* h)
{
    return small_fused_envs(h->env, h->net, h->B, h->T) > 0 && h->mode == 0 && h->n_updates == 1 && !h->traj_decoupled &&
           !h->pathwise && !h->traj_packed && !h->traj_no_acts;
}

hipError_t launch_learn_small_fused(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    SmallFusedArgs a;
    a.B = h->B; a.T = h->T; a.D = n.dims[0]; a.E = small_fused_envs(h->env, n, h->B, h->T); a.n_wg = h->B / a.E; a.P = n.P; a.inv_E = 65536u / (uint32_t)a.E + 1u;
    a.env = h->env; a.net = n;
    a.w = at<const float>(h, L.w_src);
    a.s0 = at<const uint32_t>(h, L.tr_s0); a.act = at<const uint8_t>(h, L.tr_act); a.rew = at<const float>(h, L.tr_rew);
    a.done = at<const uint8_t>(h, L.tr_done); a.val = at<const float>(h, L.tr_val); a.head = at<const float>(h, L.tr_head);
    a.h1 = at<const float>(h, L.act[0]); a.h2 = at<const float>(h, L.act[1]);
    a.adv = at<float>(h, L.adv); a.ret = at<float>(h, L.ret);
    a.part = at<float>(h, L.small_part); a.loss_part = at<float>(h, L.loss_part);
    a.counter = at<unsigned>(h, L.counters);
    a.max_spin = 1 << 22;                                        // some seconds: only a device that never runs the others gets there
    a.theta = at<float>(h, L.theta); a.grad = at<float>(h, L.grad); a.m = at<float>(h, L.m); a.v = at<float>(h, L.v);
    a.gamma = h->net_cfg.gamma; a.lambda = h->net_cfg.lambda_; a.beta = h->net_cfg.entropy_coef; a.cv = h->net_cfg.value_coef;
    a.inv_m = (float)(1.0 / ((double)h->B * h->T));
    h->adam_t += 1;
    a.lr = h->net_cfg.lr; a.beta1 = h->net_cfg.beta1; a.beta2 = h->net_cfg.beta2; a.eps = h->net_cfg.eps;
    a.bc1 = (float)(1.0 - pow((double)h->net_cfg.beta1, (double)h->adam_t));
    a.bc2 = (float)(1.0 - pow((double)h->net_cfg.beta2, (double)h->adam_t));
    const int R = a.E * a.T, R16 = (R + 15) & ~15, LD = SF_H + 1, Ep4 = (a.E + 3) & ~3;
    const size_t un = (size_t)2 * R16 * LD;
    const size_t lds = ((size_t)SF_H * LD + (size_t)10 * R16 + Ep4 + (size_t)R16 * LD + 64 + 2 * SF_WG + un) * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(learn_small_fused), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    h->metric_blocks = a.n_wg;
    ProfScope prof(h, "learn_small_fused");
    hipLaunchKernelGGL(learn_small_fused, dim3(a.n_wg), dim3(SF_WG), lds, h->stream, a);
    return hipGetLastError();
}

}  // namespace ank
