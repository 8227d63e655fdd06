// The whole backward pass of a one-hidden-layer net in one launch (paper section 3.1: the update differentiates through the
// policy network).  Nothing of the forward pass is read back and nothing is written but a chunk's partial sums.
//
//   learn_one_catch      the first layer's gradient on the matrix cores
//   learn_one_pendulum   three features a sample, all on the vector units
//
// Catch: h = relu((b1 + W1[ball]) + W1[paddle]) is rebuilt from the 4-byte state with W1
// in LDS, in the acting order, so the bits equal the acting ones; then dZ1 = relu'(h) (Wh dhead), the head matrix's sums and
// dW1 = X^T dZ1 with the board X as the 0/1 operand and dZ1 as three bfloat16 terms (exact products, binary32 sums; see
// split_terms.h).  A sample costs 20 bytes of memory.  The 0/1 operand meets every sample of a unit, so an infinite dZ1, or one
// above the largest bfloat16, would make its whole column NaN: a sum that is not finite is taken again, in binary32, over the
// samples that have its cell set.  (Below 2^-102 a dZ1 may lose its last terms, up to 2^-126 each.)
//
// Bound by vector instructions: some 30 per sample and unit, 4 of them the board operand (shared by CB column tiles) and 6 the
// terms.  A wavefront owns 32 * CB columns and walks units of 16 samples, lane (l32, kg) its columns l32 + 32 c for samples
// 8 kg + 0..7, which is at once the layout of the matrix instruction's operands, so nothing crosses lanes, and no barrier
// stands in the walk.  States and head gradients come as loads that 32 lanes share, a unit ahead.
// Before, a lane per unit added dZ1 to two rows of dW1 in LDS, a chain of read, add and write per sample.  Catch 10 x 5, before
// and now: 128 units, 1024 samples 27.9 -> 8.4 us, 65536 56.8 -> 21.1, 524288 188 -> 72; 64 units 17.1 -> 8.1, 34.4 -> 14.7,
// 99 -> 41; 256 units (activations read, dZ1 written and read), 524288 samples 360 -> 152.
#include "onehot.h"

namespace ank {

struct LearnOneArgs {
    int M, D, H, units, per;  // units of 16 samples, and how many of them a chunk has
    int cols, paddle_row0;    // board columns, first cell of the bottom row
    const float* theta; int w1_off, b1_off, wh_off;
    const float* dhead;       // [M][4]
    const uint32_t* s0;       // [M] Catch
    const float* f0; const float* f1;   // [M] pendulum
    float* partial0;          // [splits][D*H + H]
    float* partial1;          // [splits][H*NH + NH]
};

// dW1 of one cell and column over the samples m .. end
__device__ __forceinline__ float cell_sum(const LearnOneArgs& a, int m, int end, int cell, int col)
{
    const float* w1 = a.theta + a.w1_off + col;
    const float b1 = a.theta[a.b1_off + col];
    const f4v_s wh = reinterpret_cast<const f4v_s*>(a.theta + a.wh_off)[col];
    float sum = 0.0f;
    for (; m < end && sum == sum; ++m) {                         // (not a number: it stays that)
        const uint32_t s = a.s0[m];
        const int ball = (int)((s >> 8) & 0xffu) * a.cols + (int)(s & 0xffu), pad = (int)((s >> 16) & 0xffu) + a.paddle_row0;
        if (ball != cell && pad != cell) continue;
        const f4v_s d = reinterpret_cast<const f4v_s*>(a.dhead)[m];
        float dz = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dz = fmaf(wh[k], d[k], dz);
        if ((b1 + w1[ball * a.H]) + w1[pad * a.H] > 0.0f) sum += dz;
    }
    return sum;
}

// RT: tiles of 32 cells; CG wavefronts share a workgroup's 32 * CB * CG columns, 4 / CG the samples
template <int RT, int CB, int CG>
__global__ __launch_bounds__(256, 2) void learn_one_catch(const LearnOneArgs a)
{
    constexpr int W = 32 * CB * CG, SG = 4 / CG;
    extern __shared__ float lds[];                               // W1 [D][W], later the sums [SG][D + 5][W]
    __shared__ f4v_s dbh_red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, kg = lane >> 5;
    const int sg = wave / CG, j = (wave % CG) * 32 * CB + l32;   // this lane's first column
    const int D = a.D, H = a.H, j0 = blockIdx.y * W;             // j0: the workgroup's first column
    const int u0 = blockIdx.x * a.per, u1 = u0 + a.per < a.units ? u0 + a.per : a.units;
    struct In { u4v_s s[2]; f4v_s d[8]; };
    auto load = [&](In& z, int u) {
        const u4v_s* p = reinterpret_cast<const u4v_s*>(a.s0 + 16 * u + 8 * kg);
        z.s[0] = p[0]; z.s[1] = p[1];
        const f4v_s* q = reinterpret_cast<const f4v_s*>(a.dhead) + 16 * (size_t)u + 8 * kg;
#pragma unroll
        for (int e = 0; e < 8; ++e) z.d[e] = q[e];
    };
    In in[2];
    load(in[0], u0 + sg < u1 ? u0 + sg : u1 - 1);                // past the end: the last unit again, not used
    const f4v_s* w1g = reinterpret_cast<const f4v_s*>(a.theta + a.w1_off + j0);
    f4v_s* w1l = reinterpret_cast<f4v_s*>(lds);
    const int pieces = D * (W / 4);
    for (int i = tid; i < pieces; i += 256 * 8) {                // eight loads in flight
        f4v_s w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int q = i + 256 * k < pieces ? i + 256 * k : i;
            w[k] = w1g[(q / (W / 4)) * (H / 4) + q % (W / 4)];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) if (i + 256 * k < pieces) w1l[i + 256 * k] = w[k];
    }
    float b1[CB], dwh[CB][4], db1[CB];
    f4v_s wh[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        b1[c] = a.theta[a.b1_off + j0 + j + 32 * c];
        wh[c] = reinterpret_cast<const f4v_s*>(a.theta + a.wh_off)[j0 + j + 32 * c];   // every offset here is a multiple of the width
        db1[c] = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dwh[c][k] = 0.0f;
    }
    f4v_s dbh = {0.0f, 0.0f, 0.0f, 0.0f};                        // the head biases: every thread a sample of 256
    for (int m = 16 * u0 + tid; m < 16 * u1; m += 256) dbh += reinterpret_cast<const f4v_s*>(a.dhead)[m];
    f16v_s acc[RT][CB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][c][r] = 0.0f;
    const uint32_t idx2 = (uint32_t)l32 * 0x10001u;
    uint32_t ones = 0x10001u;
    asm("" : "+v"(ones));
    __syncthreads();
    const float* w1 = lds + j;
    auto unit = [&](const In& z) {
        uint32_t ball[8], pad[8], balls[4], pads[4];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t s = z.s[e >> 2][e & 3];
            ball[e] = ((s >> 8) & 0xffu) * (uint32_t)a.cols + (s & 0xffu);
            pad[e] = ((s >> 16) & 0xffu) + (uint32_t)a.paddle_row0;
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            balls[p] = ball[2 * p] | (ball[2 * p + 1] << 16);
            pads[p] = pad[2 * p] | (pad[2 * p + 1] << 16);
        }
        u4v_s t[CB][3];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            float dz[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float hv = (b1[c] + w1[ball[e] * W + 32 * c]) + w1[pad[e] * W + 32 * c];
                hv = hv > 0.0f ? hv : 0.0f;
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) { s = fmaf(wh[c][k], z.d[e][k], s); dwh[c][k] = fmaf(hv, z.d[e][k], dwh[c][k]); }
                dz[e] = hv > 0.0f ? s : 0.0f;
                db1[c] += dz[e];
            }
            split_terms(dz, t[c]);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const uint32_t at = idx2 + (uint32_t)i * 0x200020u;
            u4v_s x;
#pragma unroll
            for (int p = 0; p < 4; ++p) x[p] = one_where_zero(min_pair(balls[p] ^ at, pads[p] ^ at), ones);
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int k = 2; k >= 0; --k) acc[i][c] = mfma_f(x, t[c][k], acc[i][c]);   // smallest terms first
        }
    };
    for (int u = u0 + sg; u < u1; u += 2 * SG) {
        load(in[1], u + SG < u1 ? u + SG : u1 - 1);
        unit(in[0]);
        load(in[0], u + 2 * SG < u1 ? u + 2 * SG : u1 - 1);
        if (u + SG < u1) unit(in[1]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int o = 32; o; o >>= 1) dbh[k] += __shfl_xor(dbh[k], o);
    if (lane == 0) dbh_red[wave] = dbh;
#pragma unroll
    for (int c = 0; c < CB; ++c) {                               // both halves' samples of a column
        db1[c] += __shfl_xor(db1[c], 32);
#pragma unroll
        for (int k = 0; k < 4; ++k) dwh[c][k] += __shfl_xor(dwh[c][k], 32);
    }
    __syncthreads();
    const int rows = D + 5;
    float* mine = lds + (size_t)sg * rows * W + j;
#pragma unroll
    for (int c = 0; c < CB; ++c) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int cell = 32 * i + 8 * (r >> 2) + (r & 3) + 4 * kg;
                if (cell < D) mine[cell * W + 32 * c] = acc[i][c][r];
            }
        if (kg == 0) {
            mine[D * W + 32 * c] = db1[c];
#pragma unroll
            for (int k = 0; k < 4; ++k) mine[(D + 1 + k) * W + 32 * c] = dwh[c][k];
        }
    }
    __syncthreads();
    float* out0 = a.partial0 + (size_t)blockIdx.x * ((size_t)D * H + H);
    float* out1 = a.partial1 + (size_t)blockIdx.x * ((size_t)H * 4 + 4);
    float zero = 0.0f;                                           // NaN if a sum is not finite
    for (int i = tid; i < rows * W; i += 256) {
        float s = lds[i];
#pragma unroll
        for (int g = 1; g < SG; ++g) s += lds[(size_t)g * rows * W + i];
        const int k = i / W, col = j0 + i % W;
        zero = fmaf(s, 0.0f, zero);
        if (k <= D) out0[k * H + col] = s;                       // the bias stands behind the weights
        else out1[col * 4 + (k - D - 1)] = s;
    }
    if (zero != 0.0f) {
        // the arguments are read again: kept alive over the walk for this, they changed its registers and order (32 units,
        // 524288 samples, the step 77.1 -> 78.0 us)
        const LearnOneArgs* again = (const LearnOneArgs*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(again));
        const LearnOneArgs b = *again;
        const int v0 = blockIdx.x * b.per, v1 = v0 + b.per < b.units ? v0 + b.per : b.units;
        for (int i = tid; i < D * W; i += 256) {                 // this thread's own stores
            float* o = out0 + (i / W) * H + j0 + i % W;
            if (!(fabsf(*o) <= 0x1.fffffep127f)) *o = cell_sum(b, 16 * v0, 16 * v1, i / W, j0 + i % W);
        }
    }
    if (tid < 4 && blockIdx.y == 0) out1[(size_t)H * 4 + tid] = (dbh_red[0][tid] + dbh_red[1][tid]) + (dbh_red[2][tid] + dbh_red[3][tid]);
}

// The pendulum.  Bound by vector instructions: 16 per sample and unit.  A lane owns CB units (H = 32: half a wavefront takes
// every other sample).  A block of 64 samples has its sines and cosines made one sample a lane and handed round through LDS
// with the head gradients; made by every lane for itself they took most of the time.  Before and now: 524288
// samples, 32 units 31 -> 11 us, 64 56 -> 18, 128 107 -> 28, 256 177 -> 61; 65536 samples, 128 units 16.8 -> 7.4; 1024 samples,
// 128 units 8.8 -> 4.7.  Wavefronts share nothing until their sums are added at the end.
template <int H>
__global__ __launch_bounds__(256) void learn_one_pendulum(const LearnOneArgs a)
{
    constexpr int CB = H < 64 ? 1 : H / 64, HALVES = H == 32 ? 2 : 1;
    __shared__ float sums[4 * HALVES][7][H];                     // dW1 (three rows), db1, dWh by head
    __shared__ f4v_s xs[4][64], dbh_red[4];
    __shared__ float2 ds[4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = HALVES == 2 ? lane >> 5 : 0, j = HALVES == 2 ? lane & 31 : lane;
    // the chunk's units of 16 samples, a run of them to every wavefront
    const int u0 = blockIdx.x * a.per, u1 = u0 + a.per < a.units ? u0 + a.per : a.units, each = (a.per + 3) / 4;
    const int m0 = 16 * (u0 + wave * each), end = u0 + (wave + 1) * each, m1 = 16 * (end < u1 ? end : u1);
    float w[CB][3], b1[CB], wh[CB][3], r[CB][7];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const int col = j + 64 * c;
#pragma unroll
        for (int k = 0; k < 3; ++k) { w[c][k] = a.theta[a.w1_off + k * H + col]; wh[c][k] = a.theta[a.wh_off + col * 3 + k]; }
        b1[c] = a.theta[a.b1_off + col];
#pragma unroll
        for (int k = 0; k < 7; ++k) r[c][k] = 0.0f;
    }
    f4v_s dbh = {0.0f, 0.0f, 0.0f, 0.0f};
    struct In { float th, dot; f4v_s d; };
    auto load = [&](In& z, int m) {                              // past the end: an earlier sample again, not used
        m = m + lane < a.M ? m + lane : a.M - 1;
        z.th = a.f0[m]; z.dot = a.f1[m]; z.d = reinterpret_cast<const f4v_s*>(a.dhead)[m];
    };
    In in;
    load(in, m0);
    for (int m = m0; m < m1; m += 64) {
        const int n = m1 - m < 64 ? m1 - m : 64;                 // a multiple of 16
        float sn, cs;
        det_sincos(in.th, sn, cs);
        xs[wave][lane] = f4v_s{cs, sn, in.dot, in.d[0]};
        ds[wave][lane] = make_float2(in.d[1], in.d[2]);
        if (lane < n) dbh += in.d;
        wave_fence();
        load(in, m + 64);
        for (int e0 = 0; e0 < n; e0 += 16) {
#pragma unroll
            for (int q = 0; q < 16; q += HALVES) {
                const f4v_s x = xs[wave][e0 + q + half];
                const float2 y = ds[wave][e0 + q + half];
                const float d[3] = {x[3], y.x, y.y};
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    float hv = fmaf(x[2], w[c][2], fmaf(x[1], w[c][1], fmaf(x[0], w[c][0], b1[c])));
                    hv = hv > 0.0f ? hv : 0.0f;
                    float s = 0.0f;
#pragma unroll
                    for (int k = 0; k < 3; ++k) { s = fmaf(wh[c][k], d[k], s); r[c][4 + k] = fmaf(hv, d[k], r[c][4 + k]); }
                    const float dz = hv > 0.0f ? s : 0.0f;
#pragma unroll
                    for (int k = 0; k < 3; ++k) r[c][k] = fmaf(x[k], dz, r[c][k]);
                    r[c][3] += dz;
                }
            }
        }
        wave_fence();
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int o = 32; o; o >>= 1) dbh[k] += __shfl_xor(dbh[k], o);
    if (lane == 0) dbh_red[wave] = dbh;
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int k = 0; k < 7; ++k) sums[wave * HALVES + half][k][j + 64 * c] = r[c][k];
    __syncthreads();
    float* out0 = a.partial0 + (size_t)blockIdx.x * (4 * H);
    float* out1 = a.partial1 + (size_t)blockIdx.x * (3 * H + 3);
    for (int i = tid; i < 7 * H; i += 256) {
        const int k = i / H, col = i % H;
        float s = sums[0][k][col];
#pragma unroll
        for (int g = 1; g < 4 * HALVES; ++g) s += sums[g][k][col];
        if (k < 4) out0[i] = s;
        else out1[col * 3 + k - 4] = s;
    }
    if (tid < 3) out1[3 * H + tid] = (dbh_red[0][tid] + dbh_red[1][tid]) + (dbh_red[2][tid] + dbh_red[3][tid]);
}

hipError_t launch_learn_one_layer(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    LearnOneArgs a;
    a.M = h->B * h->T; a.D = n.dims[0]; a.H = n.dims[1];
    a.units = a.M / 16; a.per = chunk_rows(a.M, h->splits[0], h->quanta[0]) / 16;
    a.cols = h->env.cols; a.paddle_row0 = (h->env.rows - 1) * h->env.cols;
    a.theta = at<const float>(h, L.w_src); a.w1_off = n.w_off[0]; a.b1_off = n.b_off[0]; a.wh_off = n.wh_off;
    a.dhead = at<const float>(h, L.dhead); a.s0 = at<const uint32_t>(h, L.tr_s0);
    a.f0 = at<const float>(h, L.tr_f0); a.f1 = at<const float>(h, L.tr_f1);
    a.partial0 = at<float>(h, L.part[0]); a.partial1 = at<float>(h, L.part[1]);
    if (h->env.kind == ENV_PENDULUM) {
        ProfScope prof(h, "learn_one_layer");
        const auto kern = a.H == 32 ? learn_one_pendulum<32> : a.H == 64 ? learn_one_pendulum<64> : a.H == 128 ? learn_one_pendulum<128> : learn_one_pendulum<256>;
        hipLaunchKernelGGL(kern, dim3(h->splits[0]), dim3(256), 0, h->stream, a);
        return hipGetLastError();
    }
    auto go = [&](auto kern, int sg, int width) {
        const size_t lds = (size_t)sg * (a.D + 5) * width * sizeof(float);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        ProfScope prof(h, "learn_one_layer");
        hipLaunchKernelGGL(kern, dim3(h->splits[0], a.H / width), dim3(256), lds, h->stream, a);
        return hipGetLastError();
    };
    // two column tiles a wavefront share the board operand (64 units, 524288 samples: one tile 47.8 us, two 40.9; 128 units 88.3
    // and 72), but not with three tiles of cells, whose sums then leave one workgroup to a compute unit (7 x 11 cells, 64 units,
    // 65536 samples 23.8 us, one tile 17.2; 524288 60.6 and 52.9)
    const int rt = (a.D + 31) / 32;
    if (a.H == 32) return rt <= 2 ? go(learn_one_catch<2, 1, 1>, 4, 32) : go(learn_one_catch<4, 1, 1>, 4, 32);
    if (a.H == 64) return rt <= 2 ? go(learn_one_catch<2, 2, 1>, 4, 64) : go(learn_one_catch<3, 1, 2>, 2, 64);
    return go(learn_one_catch<2, 2, 2>, 2, 128);
}

}  // namespace ank
