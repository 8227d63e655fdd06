// The update for bf16 networks on the matrix cores (paper section 3.1: the
// parameter update reuses the forward pass; section 3.2: backward is the
// expensive half).  fp32 master weights and fp32 accumulation; operands of the
// matrix cores are bfloat16.
//
// Data layout.  v_mfma_f32_32x32x16_bf16 wants eight consecutive values of the
// reduction index per lane.  For dX = dY W^T the reduction runs over features,
// so row-major [M][H] operands work.  For dW = X^T dY it runs over the M = B*T
// samples, so X and dY are also kept "sample-packed": P8[M/8][H][8], eight
// consecutive samples of one feature adjacent in memory.  The accumulator
// layout of the MFMA (four consecutive rows per register group) maps directly
// onto that packing, so producers write it with 8-byte stores and consumers
// read whole operands with 16-byte loads, coalesced across lanes.
//
// Layers in whole 256-wide tiles: backward_bf16.hip.  Here:
//   head_backward_bf16   dZ_L (row-major + packed), partial dWh / dbh
//   gemm_nt_bf16         dZ_{l-1} = (dZ_l W_l^T) masked by relu'(h_{l-1}), both layouts out
//   gemm_tn_nt_bf16      both products of a layer off the 256-wide tiles: that, and partial dW_l = h_{l-1}^T dZ_l
//                        (+ column sums), split over samples
//   gemm_tn_obs_bf16     dW_1 of a Catch board of more than 256 cells: x is rebuilt from the states
//                        (other first layers: first_layer.hip, and mazes in whole 256-wide tiles below)
#include "gemm_bf16.h"
#include "detmath.h"

namespace ank {

__device__ __forceinline__ float bfu(uint16_t h) { return bf16_to_f(h); }

// ---------------------------------------------------------------------------
// heads.  Both products run on the matrix cores with the fp32 head gradient
// split into two bfloat16 terms (d = hi + lo, 16 significant bits):
//   dZ_L[m][j] = relu'(h[m][j]) * sum_k d[m][k] Wh[j][k]   one MFMA per 32x32 tile with the
//                reduction index running over (hi_0..7, lo_0..7) against (Wh_0..7, Wh_0..7)
//   dWh[j][k]  = sum_m h[m][j] d[m][k]                      reduction over samples, hi parts in
//                output columns 0..7 and lo parts in 8..15, added at the end
// The reduction over samples may visit them in any order as long as both operands agree; the
// order used here (per lane half kg: samples 4kg..4kg+3 of two consecutive groups of eight) makes
// the 8-byte pieces of packed h that feed it the same ones that mask dZ_L.
// A workgroup walks 64 samples at a time for 256 columns; wavefront w owns columns 64w..64w+63.
// ---------------------------------------------------------------------------
struct HeadBwdBf16Args {
    int M, H, NH, NHP, rows;                   // rows per workgroup (multiple of 64)
    const uint16_t* hP; const float* dhead; const uint16_t* wh16;   // wh16: bf16 copy of Wh, [H][NH]
    uint16_t* dzR; uint16_t* dzP; float* partial;                    // partial: [blocks over rows][H*NH + NH]
};

// SPLIT: at most 128 columns, which two wavefronts have; the other two take the second 32 samples of a step instead of columns
// that do not exist (128 columns, 32768 samples 12.2 -> 10.0 us; the products of a step with their stores are two thirds of it)
template <bool SPLIT>
__global__ __launch_bounds__(WG) void head_backward_bf16(const HeadBwdBf16Args a)
{
    constexpr int LDT = WG + 8, MTS = SPLIT ? 1 : 2;                    // 32-sample tiles of a step that a wavefront has
    __shared__ __attribute__((aligned(16))) uint16_t tile[64 * LDT];   // [64 samples][256 columns] for the row-major copy
    __shared__ uint4 Ahl[2][64];                                       // dZ product, A operand per 32-sample tile
    __shared__ uint4 Bhl[2][2][64];                                    // dWh product, B operand per 32-sample tile and 16-sample step
    const int H = a.H, NH = a.NH, NHP = a.NHP;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, kg = lane >> 5;
    const int jb = blockIdx.y * WG, cw = SPLIT ? wave & 1 : wave, mt0 = SPLIT ? wave >> 1 : 0, jw = jb + cw * 64;
    const int m_begin = blockIdx.x * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    bf8 wB[2];
    bool live[2];
#pragma unroll
    for (int jt = 0; jt < 2; ++jt) live[jt] = jw + 32 * jt + l32 < H;
    // packed h of this wavefront's tiles (group g of 32-sample tile mt, samples 4kg..4kg+3) and, on the first wavefront, a
    // row of the head gradient per lane, asked for 64 samples ahead and the first of them ahead of everything else: a
    // workgroup has two or three such steps, so each load's round trip would be a good part of its time
    // (128 columns, 32768 samples 12.6 -> 12.0 us).  Wider layers pay for it with a wavefront per SIMD (two instead of three)
    // and are no slower but around 131072 samples (without / with, us: 256 columns 32768 samples 15.2 / 13.0, 131072 30.9 / 31.6,
    // 524288 104.4 / 101.6; 512 columns 19.6 / 18.2, 50.1 / 51.3, 194 / 188; 128-512 with five heads 262144 148 / 144)
    uint2 hq[MTS][2][4], hn[MTS][2][4];
    float dn[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    auto fetch = [&](int m0) {
#pragma unroll
        for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
            for (int jt = 0; jt < 2; ++jt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const size_t G = (size_t)((m0 + 32 * (mt0 + mt)) >> 3) + g;
                    hn[mt][jt][g] = live[jt] ? *reinterpret_cast<const uint2*>(a.hP + (G * H + jw + 32 * jt + l32) * 8 + 4 * kg)
                                             : make_uint2(0, 0);
                }
        if (tid < 64) {
            const float* dh = a.dhead + (size_t)(m0 + tid) * NHP;
            const float4 d0 = *reinterpret_cast<const float4*>(dh);
            dn[0] = d0.x; dn[1] = d0.y; dn[2] = d0.z; dn[3] = d0.w;
            if (NHP == 8) { const float4 d1 = *reinterpret_cast<const float4*>(dh + 4); dn[4] = d1.x; dn[5] = d1.y; dn[6] = d1.z; dn[7] = d1.w; }
        }
    };
    if (m_begin < m_end) fetch(m_begin);
#pragma unroll
    for (int jt = 0; jt < 2; ++jt) {
        const int j = jw + 32 * jt + l32;
        uint16_t w8[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w8[k] = (live[jt] && k < NH) ? a.wh16[(size_t)j * NH + k] : (uint16_t)0;
        const uint4 wv = make_uint4((uint32_t)w8[0] | ((uint32_t)w8[1] << 16), (uint32_t)w8[2] | ((uint32_t)w8[3] << 16),
                                    (uint32_t)w8[4] | ((uint32_t)w8[5] << 16), (uint32_t)w8[6] | ((uint32_t)w8[7] << 16));
        wB[jt] = *reinterpret_cast<const bf8*>(&wv);
    }
    f16v acc2[2];
#pragma unroll
    for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc2[jt][r] = 0.0f;
    float db[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // output columns 16..31 of the dWh product stay zero
    reinterpret_cast<uint4*>(Bhl)[tid] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (int m0 = m_begin; m0 < m_end; m0 += 64) {
#pragma unroll
        for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
            for (int jt = 0; jt < 2; ++jt)
#pragma unroll
                for (int g = 0; g < 4; ++g) hq[mt][jt][g] = hn[mt][jt][g];
        if (tid < 64) {
            float d[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) d[k] = dn[k];
            uint16_t hi[8], lo[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k >= NH) d[k] = 0.0f;
                db[k] += d[k];
                const uint32_t p = cvt_pk_bf16(d[k], 0.0f);
                hi[k] = (uint16_t)p;
                lo[k] = (uint16_t)cvt_pk_bf16(d[k] - bfu(hi[k]), 0.0f);
            }
            const int mt = tid >> 5, s = tid & 31;
            Ahl[mt][s] = make_uint4((uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16),
                                    (uint32_t)hi[4] | ((uint32_t)hi[5] << 16), (uint32_t)hi[6] | ((uint32_t)hi[7] << 16));
            Ahl[mt][32 + s] = make_uint4((uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16),
                                         (uint32_t)lo[4] | ((uint32_t)lo[5] << 16), (uint32_t)lo[6] | ((uint32_t)lo[7] << 16));
            const int g = s >> 3, r = s & 7, kgs = r >> 2, q = (g & 1) * 4 + (r & 3);
            uint16_t* Bp = reinterpret_cast<uint16_t*>(&Bhl[mt][g >> 1][0]);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                Bp[(kgs * 32 + k) * 8 + q] = hi[k];
                Bp[(kgs * 32 + 8 + k) * 8 + q] = lo[k];
            }
        }
        if (m0 + 64 < m_end) fetch(m0 + 64);
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MTS; ++mt) {
            const uint4 a1v = Ahl[mt0 + mt][lane];
            const bf8 a1 = *reinterpret_cast<const bf8*>(&a1v);
            const uint4 b20v = Bhl[mt0 + mt][0][lane], b21v = Bhl[mt0 + mt][1][lane];
            const bf8 b20 = *reinterpret_cast<const bf8*>(&b20v), b21 = *reinterpret_cast<const bf8*>(&b21v);
#pragma unroll
            for (int jt = 0; jt < 2; ++jt) {
                const uint4 x0 = make_uint4(hq[mt][jt][0].x, hq[mt][jt][0].y, hq[mt][jt][1].x, hq[mt][jt][1].y);
                const uint4 x1 = make_uint4(hq[mt][jt][2].x, hq[mt][jt][2].y, hq[mt][jt][3].x, hq[mt][jt][3].y);
                acc2[jt] = mfma_bf16(*reinterpret_cast<const bf8*>(&x0), b20, acc2[jt]);
                acc2[jt] = mfma_bf16(*reinterpret_cast<const bf8*>(&x1), b21, acc2[jt]);
                f16v acc1;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc1[r] = 0.0f;
                acc1 = mfma_bf16(a1, wB[jt], acc1);
                const int col = cw * 64 + 32 * jt + l32;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint32_t mw[2] = {hq[mt][jt][g].x, hq[mt][jt][g].y};
                    float o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float hv = bfu((uint16_t)((mw[q >> 1] >> ((q & 1) * 16)) & 0xffffu));
                        o[q] = hv > 0.0f ? acc1[4 * g + q] : 0.0f;
                    }
                    const uint32_t p01 = cvt_pk_bf16(o[0], o[1]), p23 = cvt_pk_bf16(o[2], o[3]);
                    const int row = 32 * (mt0 + mt) + 8 * g + 4 * kg;
                    if (a.dzR) {
                        tile[(row + 0) * LDT + col] = (uint16_t)p01; tile[(row + 1) * LDT + col] = (uint16_t)(p01 >> 16);
                        tile[(row + 2) * LDT + col] = (uint16_t)p23; tile[(row + 3) * LDT + col] = (uint16_t)(p23 >> 16);
                    }
                    if (live[jt]) {
                        const size_t G = (size_t)((m0 + 32 * (mt0 + mt)) >> 3) + g;
                        *reinterpret_cast<uint2*>(a.dzP + (G * H + jw + 32 * jt + l32) * 8 + 4 * kg) = make_uint2(p01, p23);
                    }
                }
            }
        }
        __syncthreads();
        // row-major copy (only where the tiled dX kernel reads it): 64 rows x 256 columns, 16-byte pieces
        if (a.dzR)
            for (int i = tid; i < 64 * (SPLIT ? WG / 16 : WG / 8); i += WG) {
                const int row = i / (SPLIT ? WG / 16 : WG / 8), c = (i % (SPLIT ? WG / 16 : WG / 8)) * 8;
                if (jb + c < H)
                    *reinterpret_cast<uint4*>(a.dzR + (size_t)(m0 + row) * H + jb + c) = *reinterpret_cast<const uint4*>(&tile[row * LDT + c]);
            }
    }
    __syncthreads();
    // dWh: rows j of the accumulator, columns k (hi parts) and 8+k (lo parts)
    float* S = reinterpret_cast<float*>(tile);                       // [256 columns j][16] (SPLIT: [2 sample tiles][128][16])
    if (l32 < 16) {
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                S[(wave * 64 + 32 * jt + 8 * (r >> 2) + 4 * kg + (r & 3)) * 16 + l32] = acc2[jt][r];
    }
    __syncthreads();
    float* out = a.partial + (size_t)blockIdx.x * ((size_t)H * NH + NH);
    if (jb + tid < H)
        for (int k = 0; k < NH; ++k) {
            float sum = S[tid * 16 + k] + S[tid * 16 + 8 + k];
            if (SPLIT) sum += S[(128 + tid) * 16 + k] + S[(128 + tid) * 16 + 8 + k];
            out[(size_t)(jb + tid) * NH + k] = sum;
        }
    if (blockIdx.y == 0) {
        __syncthreads();
        if (tid < 64) for (int k = 0; k < 8; ++k) S[tid * 8 + k] = db[k];
        __syncthreads();
        if (tid < NH) {
            float sum = 0.0f;
            for (int i = 0; i < 64; ++i) sum += S[i * 8 + tid];
            out[(size_t)H * NH + tid] = sum;
        }
    }
}

// ---------------------------------------------------------------------------
// dX = (dY W^T) masked.  dY row-major [M][N], W bf16 [K][N] (row i, reduction j
// contiguous), mask from packed h, output in both layouts.  128 x 128 tile,
// reduction staged through LDS 128 at a time.
// FIRST: the result is dZ_1 of the pendulum, which nothing else reads: a workgroup walks some tiles of rows and adds up
// dW_1[c][i] = sum_m o_c(m) dZ_1[m][i] for the three features and the bias in eight registers (binary32, dZ_1 unrounded).
// ---------------------------------------------------------------------------
struct GemmNtBf16Args {
    int M, K, N;
    const uint16_t* dyR;      // [M][N]
    const uint16_t* w16;      // [K][N]
    const uint16_t* hP;       // packed h_{l-1}: [M/8][K][8]
    uint16_t* dxR;            // [M][K], or null when no product below reads the row-major form
    uint16_t* dxP;            // [M/8][K][8]
    const float* dhead;       // TOP: [M][NHP] head gradient
    const uint32_t* maskTop;  // ReLU flags of h_l (relu_mask_index)
    const uint16_t* wh16;     // bf16 copy of Wh: [N][NH]
    int NH, NHP;
    const float* f0; const float* f1;   // FIRST: [M] stored angle and angular velocity
    float* first_partial;     // [nbx][4*K]
    int nbx, per;             // workgroups along the samples, tiles of 128 that each of them walks
};

// TOP, the layer under the heads: both products form dZ_L themselves from the head gradient, by the product of the head pass
// above (four MFMAs per 128 samples and wavefront), and it never reaches memory; dX takes the ReLU flag words for h_L, 1/8 of
// the bytes.  What bounds these products is memory's latency for few samples and its rate for many: a launch and a write and two
// reads of dZ_L less.  Every tile of 128 rows of dW and of dX forms its dZ_L again, which costs less than that at every width
// (head pass + products -> products, us, three heads: 128-128, 32768 samples 11.9 + 16.3 -> 19.3, 524288 79.9 + 134.0 -> 151.3;
// 512-128 11.9 + 32.8 -> 38.0, 79.6 + 408.8 -> 447.7; 128-512 22.0 + 26.6 -> 30.9, 302.5 + 323.2 -> 321.8; 512 samples
// 9.2 + 9.3 -> 12.0; whole steps 3 to 56 % faster).  Two wavefronts per SIMD are what makes it so: with 307 registers, one,
// 128-128 took 200 and 512-128 773 us.
// A thread's row of the head gradient as its two terms:
struct HeadRow {
    float d[8];
    __device__ __forceinline__ void load(const float* dhead, int NH, int NHP, int m, bool ok)
    {
        const float* p = dhead + (size_t)(ok ? m : 0) * NHP;
        const float4 d0 = *reinterpret_cast<const float4*>(p), d1 = *reinterpret_cast<const float4*>(p + (NHP == 8 ? 4 : 0));
        d[0] = d0.x; d[1] = d0.y; d[2] = d0.z; d[3] = d0.w; d[4] = d1.x; d[5] = d1.y; d[6] = d1.z; d[7] = d1.w;
#pragma unroll
        for (int k = 0; k < 8; ++k) d[k] = ok && k < NH ? d[k] : 0.0f;
    }
    __device__ __forceinline__ void terms(u4v& hi, u4v& lo) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            hi[k] = cvt_pk_bf16(d[2 * k], d[2 * k + 1]);
            lo[k] = cvt_pk_bf16(d[2 * k] - bfu((uint16_t)hi[k]), d[2 * k + 1] - bfu((uint16_t)(hi[k] >> 16)));
        }
    }
};

constexpr int NB_BK = 128;
constexpr int NB_LD = NB_BK + 8;        // row stride in bf16: 272 B, 16-byte aligned, 8 rows spread over all banks

template <bool TOP, bool FIRST>
__device__ __forceinline__ void gemm_nt_bf16_body(const GemmNtBf16Args& a, const int block)
{
    extern __shared__ uint4 smem4[];
    uint16_t* As = reinterpret_cast<uint16_t*>(smem4);          // [128][NB_LD] dY tile
    uint16_t* Bs = As + 128 * NB_LD;                            // [128][NB_LD] W tile
    u4v* Ahl = reinterpret_cast<u4v*>(Bs + 128 * NB_LD);        // TOP: [4 blocks of 32 samples][64] head gradient, A operand
    float* feat = reinterpret_cast<float*>(Ahl + (TOP ? 4 * 64 : 0));   // FIRST: [2][3 features][128 samples]
    int bx, it_;
    xcd_map(block, FIRST ? a.nbx : (a.M + 127) / 128, (a.K + 127) / 128, bx, it_);   // the i-tiles of one m-tile share dY
    const int i0 = it_ * 128;
    float gw[FIRST ? 2 : 1][4];                                  // FIRST: this lane's columns' sums of three features and one
#pragma unroll
    for (int tc = 0; tc < (FIRST ? 2 : 1); ++tc)
#pragma unroll
        for (int c = 0; c < 4; ++c) gw[tc][c] = 0.0f;
    auto row_tile = [&](const int mt_, float* ft) {
        int tid = threadIdx.x;
        if (FIRST) asm volatile("" : "+v"(tid));                     // or the addresses of a tile stay in registers across the loop
        const int lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1, l32 = lane & 31, kg = lane >> 5;
        const int m0 = mt_ * 128;
        float th = 0.0f, td = 0.0f;
        if (FIRST && tid >= 128) { const int m = m0 + tid - 128 < a.M ? m0 + tid - 128 : 0; th = a.f0[m]; td = a.f1[m]; }
        // loader: 128 rows x 16 pieces of 16 B = 2048 pieces per matrix, 8 per thread
        uint4 ra[TOP ? 1 : 8], rb[8];
        u4v wr;
        uint32_t fw[4];
        auto fetch = [&](int j0) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int p = q * WG + tid, row = p >> 4, kc = (p & 15) << 3;
                if (!TOP) ra[TOP ? 0 : q] = (m0 + row < a.M) ? *reinterpret_cast<const uint4*>(a.dyR + (size_t)(m0 + row) * a.N + j0 + kc) : make_uint4(0, 0, 0, 0);
                rb[q] = (i0 + row < a.K) ? *reinterpret_cast<const uint4*>(a.w16 + (size_t)(i0 + row) * a.N + j0 + kc) : make_uint4(0, 0, 0, 0);
            }
            if (TOP) {                                               // this wavefront's 32 columns of h_L: row of Wh, ReLU flags
                const int col = j0 + wave * 32 + l32;
                wr = head_row(a.wh16, a.NH, col);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) fw[mt] = a.maskTop[relu_mask_index(m0 + 32 * mt < a.M ? (size_t)(m0 >> 5) + mt : 0, kg, a.N, col)];
            }
        };
        HeadRow hr;
        if (TOP && tid < 128) hr.load(a.dhead, a.NH, a.NHP, m0 + tid, m0 + tid < a.M);
        fetch(0);
        // the ReLU masks: asked for with the first tile (in the epilogue, where they are used, they were a round trip of their own)
        uint2 hm[2][2][4];
        auto load_masks = [&]() {
#pragma unroll
            for (int tr = 0; tr < 2; ++tr)
#pragma unroll
                for (int tc = 0; tc < 2; ++tc)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int m = m0 + wm * 64 + tr * 32 + 8 * g + 4 * kg, i = i0 + wn * 64 + tc * 32 + l32;
                        hm[tr][tc][g] = m < a.M && i < a.K ? *reinterpret_cast<const uint2*>(a.hP + ((size_t)(m >> 3) * a.K + i) * 8 + (m & 7)) : make_uint2(0, 0);
                    }
        };
        if (!FIRST) load_masks();                                    // (FIRST: when the registers of the tiles are free)
        f16v acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        if (TOP) {
            if (tid < 128) hr.terms(Ahl[(tid >> 5) * 64 + (tid & 31)], Ahl[(tid >> 5) * 64 + 32 + (tid & 31)]);
            __syncthreads();
        }
        if (FIRST && tid >= 128) {                                   // as the forward pass read them
            float sn, cs;
            det_sincos(th, sn, cs);
            ft[tid - 128] = bfu(bf16_bits(cs)); ft[tid] = bfu(bf16_bits(sn)); ft[128 + tid] = bfu(bf16_bits(td));
        }
        const uint16_t* a_rd = As + (wm * 64 + l32) * NB_LD + 8 * kg;
        const uint16_t* b_rd = Bs + (wn * 64 + l32) * NB_LD + 8 * kg;
        for (int j0 = 0; j0 < a.N; j0 += NB_BK) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int p = q * WG + tid, row = p >> 4, kc = (p & 15) << 3;
                if (!TOP) *reinterpret_cast<uint4*>(As + row * NB_LD + kc) = ra[TOP ? 0 : q];
                *reinterpret_cast<uint4*>(Bs + row * NB_LD + kc) = rb[q];
            }
            if (TOP) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    f16v z;
#pragma unroll
                    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                    z = mfma_bf16(__builtin_bit_cast(bf8, Ahl[mt * 64 + lane]), __builtin_bit_cast(bf8, wr), z);
                    uint16_t* dst = As + (32 * mt + 4 * kg) * NB_LD + wave * 32 + l32;
#pragma unroll
                    for (int p = 0; p < 8; ++p) {                    // rows 8 (p / 2) + 4 kg + 2 (p % 2) and the next
                        const uint32_t v = cvt_pk_bf16(z[2 * p], z[2 * p + 1]) & mask_pair(fw[mt], p);
                        dst[(8 * (p >> 1) + 2 * (p & 1)) * NB_LD] = (uint16_t)v;
                        dst[(8 * (p >> 1) + 2 * (p & 1) + 1) * NB_LD] = (uint16_t)(v >> 16);
                    }
                }
            }
            __syncthreads();
            if (j0 + NB_BK < a.N) fetch(j0 + NB_BK);
            else if (FIRST) load_masks();
#pragma unroll
            for (int ks = 0; ks < NB_BK; ks += 16) {
                const bf8 a0 = *reinterpret_cast<const bf8*>(a_rd + ks);
                const bf8 a1 = *reinterpret_cast<const bf8*>(a_rd + 32 * NB_LD + ks);
                const bf8 b0 = *reinterpret_cast<const bf8*>(b_rd + ks);
                const bf8 b1 = *reinterpret_cast<const bf8*>(b_rd + 32 * NB_LD + ks);
                acc[0][0] = mfma_bf16(a0, b0, acc[0][0]);
                acc[0][1] = mfma_bf16(a0, b1, acc[0][1]);
                acc[1][0] = mfma_bf16(a1, b0, acc[1][0]);
                acc[1][1] = mfma_bf16(a1, b1, acc[1][1]);
            }
            __syncthreads();
        }
        if (FIRST) {
#pragma unroll
            for (int tr = 0; tr < 2; ++tr)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4* f = reinterpret_cast<const float4*>(ft + wm * 64 + tr * 32 + 8 * g + 4 * kg);
                    const float4 fc = f[0], fs = f[32], fd = f[64];
                    const float c4[4] = {fc.x, fc.y, fc.z, fc.w}, s4[4] = {fs.x, fs.y, fs.z, fs.w}, d4[4] = {fd.x, fd.y, fd.z, fd.w};
#pragma unroll
                    for (int tc = 0; tc < 2; ++tc)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t w = q < 2 ? hm[tr][tc][g].x : hm[tr][tc][g].y;
                            const float v = bfu((uint16_t)((w >> ((q & 1) * 16)) & 0xffffu)) > 0.0f ? acc[tr][tc][4 * g + q] : 0.0f;
                            float* z = gw[FIRST ? tc : 0];
                            z[0] = fmaf(c4[q], v, z[0]); z[1] = fmaf(s4[q], v, z[1]); z[2] = fmaf(d4[q], v, z[2]); z[3] += v;
                        }
                }
            return;
        }
        // epilogue.  Accumulator register group r/4 of lane (l32, kg) holds rows 8*(r/4) + 4*kg + 0..3 of
        // column l32: exactly half of one packed group of eight samples -> 8-byte mask loads and stores.
        uint16_t* Ts = As;                                           // [128][NB_LD] staging for the row-major copy
#pragma unroll
        for (int tr = 0; tr < 2; ++tr)
#pragma unroll
            for (int tc = 0; tc < 2; ++tc) {
                const int col = wn * 64 + tc * 32 + l32, i = i0 + col;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int rowl = wm * 64 + tr * 32 + 8 * g + 4 * kg;          // first of 4 consecutive rows
                    const int m = m0 + rowl;
                    const bool ok = m < a.M && i < a.K;
                    const uint32_t mw[2] = {hm[tr][tc][g].x, hm[tr][tc][g].y};
                    uint16_t o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float hv = bfu((uint16_t)((mw[q >> 1] >> ((q & 1) * 16)) & 0xffffu));
                        o[q] = bf16_bits(hv > 0.0f ? acc[tr][tc][4 * g + q] : 0.0f);
                        if (a.dxR) Ts[(rowl + q) * NB_LD + col] = o[q];
                    }
                    if (ok) *reinterpret_cast<uint2*>(a.dxP + ((size_t)(m >> 3) * a.K + i) * 8 + (m & 7)) =
                        make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
                }
            }
        if (!a.dxR) return;
        __syncthreads();
        for (int p = tid; p < 128 * 16; p += WG) {
            const int row = p >> 4, c = (p & 15) << 3;
            if (m0 + row < a.M && i0 + c < a.K)
                *reinterpret_cast<uint4*>(a.dxR + (size_t)(m0 + row) * a.K + i0 + c) = *reinterpret_cast<const uint4*>(Ts + row * NB_LD + c);
        }
    };
    if (!FIRST) { row_tile(bx, nullptr); return; }
    const int tiles = (a.M + 127) / 128, t0 = bx * a.per, t1 = t0 + a.per < tiles ? t0 + a.per : tiles;
    for (int t = t0; t < t1; ++t) row_tile(t, feat + (t & 1) * 384);
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1, l32 = lane & 31, kg = lane >> 5;
    // two lanes and two wavefronts have samples of a column each
    float* red = reinterpret_cast<float*>(As);                   // [2 wn][2 tc][4][32], of the second wavefront
#pragma unroll
    for (int tc = 0; tc < 2; ++tc)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float* z = gw[FIRST ? tc : 0];
            z[c] += __shfl_xor(z[c], 32, 64);
            if (wm == 1 && kg == 0) red[((wn * 2 + tc) * 4 + c) * 32 + l32] = z[c];
        }
    __syncthreads();
    if (wm == 0 && kg == 0) {
        float* out = a.first_partial + (size_t)bx * 4 * a.K + i0 + wn * 64 + l32;
#pragma unroll
        for (int tc = 0; tc < 2; ++tc)
#pragma unroll
            for (int c = 0; c < 4; ++c) out[(size_t)c * a.K + 32 * tc] = gw[FIRST ? tc : 0][c] + red[((wn * 2 + tc) * 4 + c) * 32 + l32];
    }
}
__global__ __launch_bounds__(WG) void gemm_nt_bf16(const GemmNtBf16Args a) { gemm_nt_bf16_body<false, false>(a, (int)blockIdx.x); }

typedef uint32_t u32x4_l __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// dW partials from packed operands.  LDS tiles [sample group][column][8]; every
// operand is one 16-byte read.  OBS: the first layer's x comes from the state
// snapshots (walls bit planes, agent cell, goal cell / Catch cells).
// ---------------------------------------------------------------------------
struct GemmTnBf16Args {
    int M, K, N, splits, rows, tiles_i;
    int obs_row0;             // first layer: row i of this product is observation feature obs_row0 + i
    const uint16_t* xP;       // packed [M/8][K][8], unused in the first layer
    const uint16_t* dyP;      // packed [M/8][N][8]
    float* partial;           // [splits][split_stride]: K x N partial of each split
    size_t split_stride;
    float* bias_out;          // [splits][bias_stride]: N column sums of each split, or null
    size_t bias_stride;
    ObsSrc obs;
    // agent-plane product only: chunks are blocks of env_block environments over all T time steps, and the sum of
    // dY over time is written to sP (two bfloat16 terms per entry) on the way; null: chunks are sample ranges
    uint16_t* sP;
    int T, env_block;
    // TOP: dyP is packed h_L; the head gradient, bf16 Wh [N][NH], and partial sums of the gradients of Wh and its bias
    const float* dhead; const uint16_t* wh16;
    int NH, NHP;
    float* head_partial;      // [splits][N*NH + NH]
};

constexpr int TB_G = 16;      // sample groups (of 8) per LDS stage: 128 samples

__device__ __forceinline__ uint4 obs_piece(const ObsSrc& o, int mg, int i, bool valid)
{
    // eight consecutive samples of cell i of a Catch board beyond first_layer.hip's size
    uint16_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = 0;
    if (valid) {
        const int m = mg * 8;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            int bc, pc;
            catch_obs_cells(o.env, o.s0[m + q], bc, pc);
            v[q] = (i == bc || i == pc) ? 0x3f80 : 0;
        }
    }
    return make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                      (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16));
}

template <bool OBS, bool TOP>
__device__ __forceinline__ void gemm_tn_bf16_body(const GemmTnBf16Args& a, const int tile, const int split)
{
    extern __shared__ uint4 smem4[];
    uint4* Xs = smem4;                       // [TB_G][128] pieces of 8 samples
    uint4* Ys = Xs + TB_G * 128;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, kg = lane >> 5;
    const int ti = tile % a.tiles_i, tj = tile / a.tiles_i;
    const int i0 = ti * 128, j0 = tj * 128;
    const int g_begin = (split * a.rows) >> 3;
    const int g_end = (split + 1) * a.rows < a.M ? g_begin + (a.rows >> 3) : a.M >> 3;
    // loader: TB_G groups x 128 columns = 2048 pieces per matrix, 8 per thread: piece p -> group p/128, column p%128
    uint4 rx[8], ry[8];
    auto fetch = [&](int g0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int p = q * WG + tid, g = g0 + (p >> 7), c = p & 127;
            const bool gok = g < g_end;
            if (OBS) rx[q] = gok ? obs_piece(a.obs, g, a.obs_row0 + i0 + c, i0 + c < a.K) : make_uint4(0, 0, 0, 0);
            else rx[q] = (gok && i0 + c < a.K) ? *reinterpret_cast<const uint4*>(a.xP + ((size_t)g * a.K + i0 + c) * 8) : make_uint4(0, 0, 0, 0);
            if (!TOP) ry[q] = (gok && j0 + c < a.N) ? *reinterpret_cast<const uint4*>(a.dyP + ((size_t)g * a.N + j0 + c) * 8) : make_uint4(0, 0, 0, 0);
        }
        if (TOP) {                                               // 32 columns per wavefront, in the order in which the product below gives dZ
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int g = g0 + 2 * q + kg;
                ry[q] = g < g_end ? *reinterpret_cast<const uint4*>(a.dyP + ((size_t)g * a.N + j0 + wave * 32 + l32) * 8) : make_uint4(0, 0, 0, 0);
            }
        }
    };
    // TOP: sample 16 j + 8 kg + 4 h + q of a block of 32 sits in row 8 (2 j + h) + 4 kg + q of the A operand, so that a lane's
    // accumulators are eight consecutive samples of each 16; the B operand of dWh has the two terms in columns 0 and 8 on
    u4v* Ahl = reinterpret_cast<u4v*>(Ys + TB_G * 128);          // [4][64]
    uint16_t* Bhl = reinterpret_cast<uint16_t*>(Ahl + 4 * 64);   // [8 steps][2 kg][16 columns][8]
    HeadRow hr;
    float db[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    f16v acc2;
    u4v wr;
    auto fetch_head = [&](int g0) { if (tid < 128) hr.load(a.dhead, a.NH, a.NHP, g0 * 8 + tid, g0 + (tid >> 3) < g_end); };
    auto forms = [&]() {
        if (tid >= 128) return;
        u4v hi, lo;
        hr.terms(hi, lo);
        const int s = tid & 31, row = 8 * (2 * (s >> 4) + ((s >> 2) & 1)) + 4 * ((s >> 3) & 1) + (s & 3);
        Ahl[(tid >> 5) * 64 + row] = hi; Ahl[(tid >> 5) * 64 + 32 + row] = lo;
        uint16_t* b = Bhl + (tid >> 3) * 128 + (tid & 7);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            b[k * 8] = (uint16_t)(hi[k >> 1] >> (16 * (k & 1))); b[(8 + k) * 8] = (uint16_t)(lo[k >> 1] >> (16 * (k & 1)));
            db[k] += hr.d[k];
        }
    };
    if (TOP) {
        fetch_head(g_begin);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc2[r] = 0.0f;
        wr = head_row(a.wh16, a.NH, j0 + wave * 32 + l32);
    }
    fetch(g_begin);
    if (TOP) {
        forms();
        fetch_head(g_begin + TB_G);
        __syncthreads();
    }
    f16v acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    float bsum = 0.0f;
    const bool live = (i0 + wm * 64 < a.K) && (j0 + wn * 64 < a.N);
    for (int g0 = g_begin; g0 < g_end; g0 += TB_G) {
#pragma unroll
        for (int q = 0; q < 8; ++q) { const int p = q * WG + tid; Xs[p] = rx[q]; if (!TOP) Ys[p] = ry[q]; }
        if (TOP) {
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) {
                f16v z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                z = mfma_bf16(__builtin_bit_cast(bf8, Ahl[blk * 64 + lane]), __builtin_bit_cast(bf8, wr), z);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int q = 2 * blk + j;
                    const uint32_t hw[4] = {ry[q].x, ry[q].y, ry[q].z, ry[q].w};
                    if (ti == 0) acc2 = mfma_bf16(__builtin_bit_cast(bf8, ry[q]), *reinterpret_cast<const bf8*>(Bhl + ((2 * q + kg) * 16 + (l32 & 15)) * 8), acc2);
                    uint32_t w[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[k] = cvt_pk_bf16(z[8 * j + 2 * k], z[8 * j + 2 * k + 1]) & positive_mask_pk(hw[k]);
                    Ys[(2 * q + kg) * 128 + wave * 32 + l32] = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
        }
        __syncthreads();
        if (g0 + TB_G < g_end) fetch(g0 + TB_G);
        if (TOP) { forms(); fetch_head(g0 + 2 * TB_G); }
        if (live) {
#pragma unroll
            for (int ks = 0; ks < TB_G; ks += 2) {                // one MFMA step = 16 samples = 2 groups
                const uint4 xa0 = Xs[(ks + kg) * 128 + wm * 64 + l32], xa1 = Xs[(ks + kg) * 128 + wm * 64 + 32 + l32];
                const uint4 yb0 = Ys[(ks + kg) * 128 + wn * 64 + l32], yb1 = Ys[(ks + kg) * 128 + wn * 64 + 32 + l32];
                const bf8 a0 = *reinterpret_cast<const bf8*>(&xa0), a1 = *reinterpret_cast<const bf8*>(&xa1);
                const bf8 b0 = *reinterpret_cast<const bf8*>(&yb0), b1 = *reinterpret_cast<const bf8*>(&yb1);
                acc[0][0] = mfma_bf16(a0, b0, acc[0][0]);
                acc[0][1] = mfma_bf16(a0, b1, acc[0][1]);
                acc[1][0] = mfma_bf16(a1, b0, acc[1][0]);
                acc[1][1] = mfma_bf16(a1, b1, acc[1][1]);
            }
        }
        if (ti == 0 && tid < 128) {
#pragma unroll 4
            for (int g = 0; g < TB_G; ++g) {
                const uint4 y = Ys[g * 128 + tid];
                const uint32_t yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                for (int q = 0; q < 8; ++q) bsum += bfu((uint16_t)((yw[q >> 1] >> ((q & 1) * 16)) & 0xffffu));
            }
        }
        __syncthreads();
    }
    float* out = a.partial + (size_t)split * a.split_stride;
    if (live) {
#pragma unroll
        for (int tr = 0; tr < 2; ++tr)
#pragma unroll
            for (int tc = 0; tc < 2; ++tc) {
                const int j = j0 + wn * 64 + tc * 32 + l32;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = i0 + wm * 64 + tr * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
                    if (i < a.K && j < a.N) out[(size_t)i * a.N + j] = acc[tr][tc][r];
                }
            }
    }
    if (ti == 0 && a.bias_out && tid < 128 && j0 + tid < a.N) a.bias_out[(size_t)split * a.bias_stride + j0 + tid] = bsum;
    if (TOP && ti == 0) {
        float* hout = a.head_partial + (size_t)split * ((size_t)a.N * a.NH + a.NH);
        float* S = reinterpret_cast<float*>(Xs);                 // [128 columns][16], then [2][8]
        if (l32 < 16) {
#pragma unroll
            for (int r = 0; r < 16; ++r) S[(wave * 32 + 8 * (r >> 2) + 4 * kg + (r & 3)) * 16 + l32] = acc2[r];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) db[k] += __shfl_xor(db[k], d, 64);
        if (lane == 0 && wave < 2) {
#pragma unroll
            for (int k = 0; k < 8; ++k) S[2048 + wave * 8 + k] = db[k];
        }
        __syncthreads();
        if (tid < 128)
            for (int k = 0; k < a.NH; ++k) hout[(size_t)(j0 + tid) * a.NH + k] = S[tid * 16 + k] + S[tid * 16 + 8 + k];
        if (tj == 0 && tid < a.NH) hout[(size_t)a.N * a.NH + tid] = S[2048 + tid] + S[2056 + tid];
    }
}
__global__ __launch_bounds__(WG) void gemm_tn_obs_bf16(const GemmTnBf16Args a) { gemm_tn_bf16_body<true, false>(a, (int)blockIdx.x, (int)blockIdx.y); }

// Both products of a layer that takes the 128-wide tiles, dW workgroups first.  They read the same dZ and neither fills the
// chip for long: as two launches one after the other they were mostly their own beginnings and ends (128-128, 32768 samples
// 9.8 + 11.2 -> 14.0 us).
template <bool TOP, bool FIRST>
__global__ __launch_bounds__(WG, 2) void gemm_tn_nt_bf16(const GemmTnBf16Args t, const GemmNtBf16Args n, const int tiles, const int tn_blocks)
{
    const int b = (int)blockIdx.x;
    if (b < tn_blocks) gemm_tn_bf16_body<false, TOP>(t, b % tiles, b / tiles);
    else gemm_nt_bf16_body<TOP, FIRST>(n, b - tn_blocks);
}

// The first layer of a maze with a 256 x 256 tile and eight wavefronts (two per SIMD, so one's LDS and
// global traffic overlaps the other's MFMAs): wavefront (wm, wn) owns rows 128*wm.., columns
// 64*wn.. of the tile, eight 32 x 32 accumulators, and every 16-byte read from LDS feeds 2 or 4
// MFMAs.  K and N multiples of 256.
constexpr int BIGWG = 512;
constexpr int TB_BG = 8;      // sample groups (of 8) per LDS stage: 64 samples

// XMODE: where the X operand comes from.  1: the agent plane of the
// maze observation, a one-hot of the agent cell, built in registers from the stage's 64 cell indices, which pass
// through LDS (64 rows x 128 columns per wavefront, so that a one-hot operand feeds four MFMAs: three instructions a word,
// four per MFMA, where a piece through LDS cost a 16-byte store, three reads and ten compares; what was most of its LDS
// time went that way: 16 x 16 maze, 512 columns, 524288 samples 162 -> 147 us, 256 columns, 131072 samples 37.8 -> 33.0;
// dZ read once at the rate of a copy is 95 us); 2: the wall plane of the maze observation (samples are environments,
// rows are cells), built from the stage's 64 x 8 wall words which pass through LDS the same way.
// Pipeline: LDS holds two stages.  While the MFMAs run on stage i, the same wavefronts put stage
// i + 1 into the other half -- its four pieces per thread go between the four MFMA steps, so
// the LDS stores and the vector work behind them (the one-hot, the sums) run in the shadow of the
// matrix cores -- and then ask for stage i + 3 into the registers just emptied: every load has two
// stages to arrive, and there is one barrier per stage.  Chunks are pairs of stages of 64 samples
// (a.rows % 128 == 0); the last one may be shorter and end after an odd stage.
// 1 (bfloat16) in the halves of w that equal c's, 0 in the others
__device__ __forceinline__ uint32_t one_where_equal(uint32_t w, uint32_t c)
{
    uint32_t r;
    const uint32_t one = 0x00010001u, bf1 = 0x3f803f80u, neg = 0xc080c080u;   // 0x3f80 - 0x3f80 * min(w ^ c, 1)
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(w ^ c), "v"(one));
    asm("v_pk_mad_u16 %0, %1, %2, %3" : "=v"(r) : "v"(r), "v"(neg), "v"(bf1));
    return r;
}
template <int XMODE>
__global__ __launch_bounds__(BIGWG) void gemm_tn_bf16_big(const GemmTnBf16Args a)
{
    extern __shared__ uint4 smem4[];         // [2 stages][X | Y][TB_BG][256] pieces of 8 samples
    __shared__ __attribute__((aligned(16))) uint16_t posL[4][64];   // XMODE 1: agent cells of the 64 samples of a stage
    __shared__ uint32_t wallsL[2][XMODE == 2 ? 8 : 1][64];   // XMODE 2: the eight wall words of the 64 environments of a stage
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int RT = XMODE == 1 ? 2 : 4, CT = 8 / RT;                  // 32 x 32 tiles of a wavefront
    const int wm = wave / (8 / CT), wn = wave % (8 / CT), l32 = lane & 31, kg = lane >> 5;
    int split, tile;
    xcd_map((int)blockIdx.x, a.splits, a.tiles_i * (a.N / 256), split, tile);   // the tiles of one split share its samples
    const int ti = tile % a.tiles_i, tj = tile / a.tiles_i;
    const int i0 = ti * 256, j0 = tj * 256;
    // the last chunk may be shorter, and then end in the middle of a pair of stages
    const int n_stages = (a.rows < a.M - split * a.rows ? a.rows : a.M - split * a.rows) >> 6;
    const bool by_env = XMODE == 1 && a.sP != nullptr;
    // first sample group of stage i of this chunk.  Sample ranges: consecutive stages.  Blocks of environments: the 64
    // environments of one stage at t = 0 .. T-1, then the next 64 (so a thread meets every time step of its samples
    // in order and can add them up)
    auto stage_g0 = [&](int i) -> int {
        if (by_env) {
            const int p = i / a.T, t = i - p * a.T;
            return (t * a.obs.B + split * a.env_block + 64 * p) >> 3;
        }
        return ((split * a.rows) >> 3) + i * TB_BG;
    };
    // loader: thread = (column, parity of the sample group), four groups of the stage each
    const int lc = tid & 255, lg = tid >> 8;
    struct Set { u32x4_l y[TB_BG / 2]; uint32_t pos; };
    Set S0, S1;
    auto fetch = [&](Set& st, int i) {
        if (i >= n_stages) i = n_stages - 1;                     // past the end: re-read the last stage, never used
        const int g0 = stage_g0(i);
        // the cells first: they are needed one step before the rest of the set, and loads complete in issue order
        if (XMODE == 1) st.pos = a.obs.s0[(size_t)g0 * 8 + (tid & 63)];
        // wall words: thread = (environment of the stage, word); a stage never straddles the two halves of the 2B
        // samples (B is a multiple of 64)
        if (XMODE == 2) st.pos = a.obs.walls[(size_t)(tid & 7) * a.obs.B + (g0 * 8) % a.obs.B + (tid >> 3)];
#pragma unroll
        for (int q = 0; q < TB_BG / 2; ++q) {
            const int g = g0 + 2 * q + lg;
            st.y[q] = *reinterpret_cast<const u32x4_l*>(a.dyP + ((size_t)g * a.N + j0 + lc) * 8);
        }
    };
    float tsum[TB_BG / 2][8];                                    // by_env: sum over time of this thread's dY entries
#pragma unroll
    for (int q = 0; q < TB_BG / 2; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) tsum[q][e] = 0.0f;
    float bsum = 0.0f;
    const bool sums = ti == 0 && a.bias_out != nullptr;
    // piece q (sample group 2q + lg) of stage i, held in st, -> half nb of LDS; counted: a real stage (not the
    // repeat of the last one that the last step stores), whose dY entries go into the sums
    auto store_piece = [&](const Set& st, int i, int nb, int q, bool counted) {
        uint4* Xs = smem4 + nb * (2 * TB_BG * 256);
        uint4* Ys = Xs + TB_BG * 256;
        const int gl = 2 * q + lg;
        u32x4_l x;
        if (XMODE == 2) {
            const int c = a.obs_row0 + i0 + lc;                  // this thread's cell: bit c % 32 of wall word c / 32
            const u32x4_l w0 = *reinterpret_cast<const u32x4_l*>(&wallsL[i & 1][XMODE == 2 ? c >> 5 : 0][gl * 8]);
            const u32x4_l w1 = *reinterpret_cast<const u32x4_l*>(&wallsL[i & 1][XMODE == 2 ? c >> 5 : 0][gl * 8 + 4]);
            const uint32_t one = 0x3f80u;
            const int sh = c & 31;
            x[0] = (((w0[0] >> sh) & 1u) * one) | (((w0[1] >> sh) & 1u) * (one << 16));
            x[1] = (((w0[2] >> sh) & 1u) * one) | (((w0[3] >> sh) & 1u) * (one << 16));
            x[2] = (((w1[0] >> sh) & 1u) * one) | (((w1[1] >> sh) & 1u) * (one << 16));
            x[3] = (((w1[2] >> sh) & 1u) * one) | (((w1[3] >> sh) & 1u) * (one << 16));
            *reinterpret_cast<u32x4_l*>(&Xs[gl * 256 + lc]) = x;
        }
        *reinterpret_cast<u32x4_l*>(&Ys[gl * 256 + lc]) = st.y[q];
        // column sums in every workgroup (used only where `sums` holds; the workgroups that need them set the pace
        // anyway, and a branch on `sums` here would split the step into many basic blocks)
        const float keep = counted ? 1.0f : 0.0f;
        if (XMODE != 1) {
            float part = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) part += bfu((uint16_t)((st.y[q][e >> 1] >> ((e & 1) * 16)) & 0xffffu));
            bsum = fmaf(keep, part, bsum);
        }
        if (by_env) {
#pragma unroll
            for (int e = 0; e < 8; ++e) tsum[q][e] = fmaf(keep, bfu((uint16_t)((st.y[q][e >> 1] >> ((e & 1) * 16)) & 0xffffu)), tsum[q][e]);
        }
    };
    // by_env, after the last time step of a block of 64 environments (stage i): the sums leave as two bfloat16 terms,
    // hi in sample rows 0..B-1 and lo in rows B..2B-1 of a packed matrix with 2B samples
    auto flush_time_sum = [&](int i) {
        const int p = i / a.T;
        const size_t n = (size_t)(a.obs.B >> 3) * a.N;
#pragma unroll
        for (int q = 0; q < TB_BG / 2; ++q) {
            const size_t idx = (size_t)(((split * a.env_block + 64 * p) >> 3) + 2 * q + lg) * a.N + j0 + lc;
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                hi[w] = cvt_pk_bf16(tsum[q][2 * w], tsum[q][2 * w + 1]);
                lo[w] = cvt_pk_bf16(tsum[q][2 * w] - bfu((uint16_t)hi[w]), tsum[q][2 * w + 1] - bfu((uint16_t)(hi[w] >> 16)));
            }
            *reinterpret_cast<uint4*>(a.sP + idx * 8) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(a.sP + (n + idx) * 8) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
#pragma unroll
            for (int e = 0; e < 8; ++e) tsum[q][e] = 0.0f;
        }
    };
    uint32_t cell[RT];                                           // XMODE 1: the cells of this lane's rows, in both halves
#pragma unroll
    for (int t = 0; t < RT; ++t) cell[t] = (uint32_t)(a.obs_row0 + i0 + wm * 32 * RT + 32 * t + l32 - a.obs.env.rows * a.obs.env.cols) * 0x00010001u;
    f16v acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // MFMA step ks (16 samples = groups ks, ks + 1) on half cb of LDS
    auto compute_step = [&](int cb, int ks, int i) {
        const uint4* Xs = smem4 + cb * (2 * TB_BG * 256);
        const uint4* Ys = Xs + TB_BG * 256;
        bf8 av[RT], bv[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) bv[t] = *reinterpret_cast<const bf8*>(&Ys[(ks + kg) * 256 + wn * 32 * CT + 32 * t + l32]);
        if (XMODE == 1) {
            const u32x4_l p = *reinterpret_cast<const u32x4_l*>(&posL[i & 3][(ks + kg) * 8]);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                u32x4_l x;
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = one_where_equal(p[k], cell[t]);
                av[t] = __builtin_bit_cast(bf8, x);
            }
        } else {
#pragma unroll
            for (int t = 0; t < RT; ++t) av[t] = *reinterpret_cast<const bf8*>(&Xs[(ks + kg) * 256 + wm * 32 * RT + 32 * t + l32]);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[i][j] = mfma_bf16(av[i], bv[j], acc[i][j]);
    };
    // one step: the MFMAs of stage i on half i % 2 of LDS, stage i + 1 (held in `nxt`) into the other half piece by
    // piece between them; then `nxt` is refilled with stage i + 3 and the cells of stage i + 2 (held in `aft`) go to
    // LDS (XMODE 1: not where other wavefronts may still build stage i's one-hot from)
    auto step = [&](Set& nxt, const Set& aft, int i) {
        const int cb = i & 1;
        const bool counted = i + 1 < n_stages;
#pragma unroll
        for (int q = 0; q < TB_BG / 2; ++q) {
            store_piece(nxt, i + 1, cb ^ 1, q, counted);
            __builtin_amdgcn_sched_barrier(0);
            compute_step(cb, 2 * q, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (by_env && ti == 0 && counted && (i + 2) % a.T == 0) flush_time_sum(i + 1);
        if (XMODE == 1 && tid < 64) posL[(i + 2) & 3][tid] = (uint16_t)aft.pos;
        if (XMODE == 2) wallsL[cb][XMODE == 2 ? tid & 7 : 0][tid >> 3] = aft.pos;
        fetch(nxt, i + 3);
        __syncthreads();
    };
    // S0's loads strictly before S1's: the scheduler is otherwise free to issue S1's first, and then the wait-count
    // pass, which merges this state with the loop's own at the loop header, has to wait for every load in flight
    // there on every trip (loads complete in issue order), which would end the look-ahead
    fetch(S0, 0);
    __builtin_amdgcn_sched_barrier(0);
    fetch(S1, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (XMODE == 1) {
        if (tid < 64) { posL[0][tid] = (uint16_t)S0.pos; posL[1][tid] = (uint16_t)S1.pos; }
        __syncthreads();
    }
    if (XMODE == 2) {
        wallsL[0][XMODE == 2 ? tid & 7 : 0][tid >> 3] = S0.pos; wallsL[1][XMODE == 2 ? tid & 7 : 0][tid >> 3] = S1.pos;
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < TB_BG / 2; ++q) store_piece(S0, 0, 0, q, true);
    if (by_env && ti == 0 && a.T == 1) flush_time_sum(0);
    __builtin_amdgcn_sched_barrier(0);
    fetch(S0, 2);
    __syncthreads();
    // two steps per trip without a branch between them: with a conditional second step the wait-count pass gives up
    // counting in the same way
    int i = 0;
    for (; i + 1 < n_stages; i += 2) {
        step(S1, S0, i);
        step(S0, S1, i + 1);
    }
    if (i < n_stages) step(S1, S0, i);                       // an odd stage, outside the loop for the same reason
    float* out = a.partial + (size_t)split * a.split_stride;
#pragma unroll
    for (int tr = 0; tr < RT; ++tr)
#pragma unroll
        for (int tc = 0; tc < CT; ++tc) {
            const int j = j0 + wn * 32 * CT + tc * 32 + l32;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i0 + wm * 32 * RT + tr * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
                out[(size_t)i * a.N + j] = acc[tr][tc][r];
            }
        }
    if (sums) {
        // the two threads of a column (even and odd sample groups) add their sums in a fixed order
        float* red = reinterpret_cast<float*>(smem4);
        if (lg == 1) red[lc] = bsum;
        __syncthreads();
        if (lg == 0) a.bias_out[(size_t)split * a.bias_stride + j0 + lc] = bsum + red[lc];
    }
}

// ---------------------------------------------------------------------------
// Maze first layer.  The observation has three one-hot planes (paper section 2.1 style grid
// world: walls, agent, goal) and only the agent plane changes within an unroll, so
//   dW1[wall cell c]  = sum_b walls[b][c] * S[b],   S[b] = sum_t dZ1[t][b]   (B samples, not B*T)
//   dW1[agent cell c] = sum_m [pos_m == c] dZ1[m]                             (the only full-length product)
//   dW1[goal cell]    = db1 = sum_b S[b]  for the one goal cell, zero for the others
// S leaves as two bfloat16 terms (hi rows 0..B-1, lo rows B..2B-1 of a packed matrix with 2B
// samples) and the wall product runs over those 2B samples.  The agent product reads every dZ1
// entry anyway and writes S itself when its chunks are blocks of environments; time_sum_bf16 is
// the separate pass for batch sizes that do not divide that way.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void time_sum_bf16(const uint16_t* __restrict__ dzP, uint16_t* __restrict__ sP, int B, int T, int H)
{
    const size_t idx = (size_t)blockIdx.x * WG + threadIdx.x;          // (env group, column)
    const size_t n = (size_t)(B >> 3) * H;
    if (idx >= n) return;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 8
    for (int t = 0; t < T; ++t) {
        const uint4 v = *reinterpret_cast<const uint4*>(dzP + ((size_t)t * n + idx) * 8);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += bfu((uint16_t)((w[e >> 1] >> ((e & 1) * 16)) & 0xffffu));
    }
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        hi[q] = cvt_pk_bf16(s[2 * q], s[2 * q + 1]);
        lo[q] = cvt_pk_bf16(s[2 * q] - bfu((uint16_t)hi[q]), s[2 * q + 1] - bfu((uint16_t)(hi[q] >> 16)));
    }
    *reinterpret_cast<uint4*>(sP + idx * 8) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    *reinterpret_cast<uint4*>(sP + (n + idx) * 8) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// ---------------------------------------------------------------------------
// bf16 copies of the parameters the matrix cores read: same indexing (w16) and
// every weight matrix transposed (wt16: layers [N][K], heads [NH][HL]).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(WG) void refresh_bf16(const float* __restrict__ theta, uint16_t* __restrict__ w16,
                                                   uint16_t* __restrict__ wt16, const NetShape net)
{
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i >= net.P) return;
    const uint16_t v = bf16_bits(theta[i]);
    w16[i] = v;
    wt16[transposed_index(net, i)] = v;
}

hipError_t launch_refresh_bf16(anakin* h)
{
    const Layout& L = h->lay;
    hipLaunchKernelGGL(refresh_bf16, dim3((h->net.P + WG - 1) / WG), dim3(WG), 0, h->stream,
                       at<const float>(h, L.theta), at<uint16_t>(h, L.w_bf16), at<uint16_t>(h, L.wt_bf16), h->net);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// backward through all layers for a bf16 network
// ---------------------------------------------------------------------------
// A layer with K inputs and N outputs whose products run side by side in one launch (backward_bf16.hip), a workgroup per
// compute unit: chunks of the dW product at most, and row ranges of the dX product beside `splits` of them.
static bool bf16_dx_shape(int M, int K, int N) { return (N == 256 || N == 512) && K % 256 == 0 && M % 32 == 0; }
int bf16_dw_chunks(int M, int K, int N, bool top)
{
    const int tiles = (K / 256) * (N / 256), most = (top ? 144 : 128) / tiles, want = M / 512;
    if (most < 1) return 1;
    return most <= 64 || want >= most ? most : want > 64 ? want : 64;
}
int bf16_dx_ranges(int M, int K, int N, int splits)
{
    const int rest = 256 - splits * (K / 256) * (N / 256), most = rest / (K / 256) > 1 ? rest / (K / 256) : 1;
    return M / 32 < most ? M / 32 : most;
}

// Whether both products of layer l + 1 (reading dZ_l, l >= 1) run in that launch.  It reads and writes the packed layout
// only, so it is used only where the product below it (which reads its output) does too.
bool bf16_dx_resident(const NetShape& n, int M, int l)
{
    if (l < 1 || l >= n.L) return false;
    if (!bf16_dx_shape(M, n.dims[l], n.dims[l + 1])) return false;
    return l == 1 || bf16_dx_resident(n, M, l - 1);
}

// Whether the top layer's products form dZ_L themselves (no head pass, no dZ_L in memory): both sides of the layer
// multiples of 256, both products in one launch.
bool bf16_top_fused(const NetShape& n, int M)
{
    if (!n.bf16 || n.L < 2 || n.NH > 8) return false;
    if (n.dims[n.L] % 256 != 0 || n.dims[n.L - 1] % 256 != 0) return false;
    return bf16_dx_resident(n, M, n.L - 1);
}

// Whether a top layer in 128-wide tiles forms dZ_L in its products too (above at HeadRow: both sides)
bool bf16_top_fold(const NetShape& n)
{
    return n.bf16 && n.L >= 2 && n.NH <= 8 && (n.dims[n.L] % 256 != 0 || n.dims[n.L - 1] % 256 != 0);
}

// Whether the pendulum's first-layer gradient is summed in the dX product of a second and top layer in 128-wide tiles: a launch
// less, and dZ_1 is neither written nor read (steps, us, first layer apart and here: 128-128, 512 samples 41.4 and 38.3, 32768
// 99.0 and 94.5, 524288 266 and 238; 512-128 58.4 and 55.3, 177.0 and 168.6, 788 and 651; 128-256 46.0 and 43.9, 117.8 and 113.5).
// Under 512 outputs few samples lose by it (128-512, 512 samples 61.2 and 63.4, 8192 144.1 and 145.5, 32768 150.7 and 147.1):
// the walk's four turns per tile ask for the ReLU masks last.  A third layer's product has no registers left for the sums.
bool bf16_first_fold(const NetShape& n, const EnvDims& ed, int M)
{
    return ed.kind == ENV_PENDULUM && n.L == 2 && bf16_top_fold(n) && (n.dims[2] < 512 || M >= 32768);
}

hipError_t launch_backward_bf16(anakin* h)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    const int M = h->B * h->T;
    hipError_t e;
    auto dzR = [&](int l) { return at<uint16_t>(h, L.dz[l]); };
    auto dzP = [&](int l) { return at<uint16_t>(h, L.dz[l]) + (size_t)M * n.dims[l + 1]; };
    auto actP = [&](int l) { return at<uint16_t>(h, L.act[l]); };
    // dZ_l is kept sample-packed; the row-major copy exists only where the tiled dX kernel of layer l + 1 reads it
    auto needs_rows = [&](int l) { return l >= 1 && !bf16_dx_resident(n, M, l); };
    const bool top_fused = bf16_top_fused(n, M) && h->quanta[n.L - 1] == 128 && h->splits[n.L] == h->splits[n.L - 1] && h->head_fan == 1;
    const bool top_fold = bf16_top_fold(n) && h->quanta[n.L] == h->quanta[n.L - 1] && h->splits[n.L] == h->splits[n.L - 1] && h->head_fan == 1;
    const bool first_fold = top_fold && bf16_first_fold(n, h->env, M) && h->quanta[0] == 128;
    if (!top_fused && !top_fold) {   // heads
        HeadBwdBf16Args a;
        a.M = M; a.H = n.dims[n.L]; a.NH = n.NH; a.NHP = n.NHP;
        const int stage1 = h->splits[n.L] * h->head_fan;
        a.rows = chunk_rows(M, stage1, h->quanta[n.L]);
        a.hP = actP(n.L - 1); a.dhead = at<const float>(h, L.dhead);
        a.wh16 = at<const uint16_t>(h, L.w16_src) + n.wh_off;
        a.dzR = needs_rows(n.L - 1) ? dzR(n.L - 1) : nullptr; a.dzP = dzP(n.L - 1);
        a.partial = h->head_fan > 1 ? at<float>(h, L.head_stage) : at<float>(h, L.part[n.L]);
        {
            ProfScope prof(h, "head_backward");
            if (a.H <= 128) hipLaunchKernelGGL(head_backward_bf16<true>, dim3(stage1), dim3(WG), 0, h->stream, a);
            else hipLaunchKernelGGL(head_backward_bf16<false>, dim3(stage1, (a.H + WG - 1) / WG), dim3(WG), 0, h->stream, a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (h->head_fan > 1) {
            const int stride = a.H * a.NH + a.NH;
            ProfScope prof(h, "partial_reduce");
            e = launch_partial_reduce(at<const float>(h, L.head_stage), at<float>(h, L.part[n.L]), stride, h->head_fan,
                                      h->splits[n.L], h->stream);
            if (e != hipSuccess) return e;
        }
    }
    auto obs_src = [&]() {
        ObsSrc o;
        o.kind = h->env.kind; o.env = h->env; o.B = h->B;
        o.s0 = at<const uint32_t>(h, L.tr_s0); o.f0 = at<const float>(h, L.tr_f0);
        o.f1 = at<const float>(h, L.tr_f1); o.walls = at<const uint32_t>(h, L.walls);
        return o;
    };
    // dW partials of the first layer, whose x comes from the states; big: a plane of a maze in 256 x 256 tiles
    auto run_tn = [&](GemmTnBf16Args& t, bool big, const char* name) -> hipError_t {
        const int tile = big ? 256 : 128;
        t.tiles_i = (t.K + tile - 1) / tile;
        const int tiles = t.tiles_i * ((t.N + tile - 1) / tile);
        const dim3 grid = big ? dim3(tiles * t.splits) : dim3(tiles, t.splits);
        const size_t lds = (size_t)2 * (big ? 2 * TB_BG * 256 : TB_G * 128) * sizeof(uint4);   // 256-tile kernel: two stages
        // X operand of the 256-tile kernel: the agent plane (one-hot of the cell) or the wall plane
        const int cells = h->env.rows * h->env.cols;
        const bool agent = h->env.kind == ENV_MAZE && t.obs_row0 == cells && t.K == cells;
        if (big && !agent && !(h->env.kind == ENV_MAZE && t.obs_row0 == 0 && t.K == cells && h->B % 64 == 0)) return hipErrorInvalidValue;
        const auto kern = !big ? gemm_tn_obs_bf16 : agent ? gemm_tn_bf16_big<1> : gemm_tn_bf16_big<2>;
        const hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e2 != hipSuccess) return e2;
        ProfScope prof(h, name);
        hipLaunchKernelGGL(kern, grid, dim3(big ? BIGWG : WG), lds, h->stream, t);
        return hipGetLastError();
    };
    for (int l = n.L - 1; l >= 0; --l) {
        if (l == 0 && first_fold) continue;
        if (l == 0 && first_layer_split(h)) {
            const int H1 = n.dims[1], cells = h->env.rows * h->env.cols, plane = cells * H1;
            uint16_t* sP = at<uint16_t>(h, L.time_sum);
            float* pw = at<float>(h, L.part[0]);
            float* pa = pw + (size_t)plane * h->splits_w;
            float* pg = pa + (size_t)plane * h->splits[0];
            // the agent product adds dZ1 up over time on its way when its chunks can be blocks of 64 k environments
            const bool sum_in_product = h->B % (64 * h->splits[0]) == 0 && M % (h->splits[0] * 128) == 0;
            if (!sum_in_product) {
                ProfScope prof(h, "time_sum");
                hipLaunchKernelGGL(time_sum_bf16, dim3(((h->B >> 3) * H1 + WG - 1) / WG), dim3(WG), 0, h->stream,
                                   dzP(0), sP, h->B, h->T, H1);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            GemmTnBf16Args t;
            t.M = M; t.K = cells; t.N = H1; t.splits = h->splits[0]; t.rows = chunk_rows(M, t.splits, h->quanta[0]);
            t.obs_row0 = cells; t.xP = nullptr; t.dyP = dzP(0);
            t.partial = pa; t.split_stride = (size_t)plane; t.bias_out = nullptr; t.bias_stride = 0;
            t.obs = obs_src();
            t.sP = sum_in_product ? sP : nullptr; t.T = h->T; t.env_block = h->B / h->splits[0];
            if ((e = run_tn(t, true, "gemm_tn_agent")) != hipSuccess) return e;
            t.M = 2 * h->B; t.splits = h->splits_w; t.rows = chunk_rows(t.M, t.splits, 128);
            t.obs_row0 = 0; t.dyP = sP;
            t.partial = pw; t.bias_out = pg; t.bias_stride = (size_t)H1;
            t.sP = nullptr;
            if ((e = run_tn(t, true, "gemm_tn_walls")) != hipSuccess) return e;
            continue;
        }
        if (l == 0 && (first_onehot(h) || h->env.kind == ENV_PENDULUM)) {
            e = h->env.kind == ENV_PENDULUM ? launch_first_layer_pendulum_bf16(h) : launch_first_layer_onehot(h, true);
            if (e != hipSuccess) return e;
            continue;
        }
        GemmTnBf16Args t;
        t.M = M; t.K = n.dims[l]; t.N = n.dims[l + 1];
        t.splits = h->splits[l]; t.rows = chunk_rows(M, t.splits, h->quanta[l]);
        t.obs_row0 = 0;
        t.xP = l > 0 ? actP(l - 1) : nullptr;
        t.dyP = dzP(l);
        t.partial = at<float>(h, L.part[l]);
        t.split_stride = (size_t)t.K * t.N + t.N;
        t.bias_out = t.partial + (size_t)t.K * t.N; t.bias_stride = t.split_stride;
        t.obs = obs_src();
        t.sP = nullptr; t.T = h->T; t.env_block = 0;
        const bool fold = top_fold && l == n.L - 1;
        if (fold) {
            t.dyP = actP(l);
            t.dhead = at<const float>(h, L.dhead); t.wh16 = at<const uint16_t>(h, L.w16_src) + n.wh_off; t.NH = n.NH; t.NHP = n.NHP;
            t.head_partial = at<float>(h, L.part[n.L]);
        }
        const bool resident = bf16_dx_resident(n, M, l);         // both products, 256-wide tiles
        const bool big = l > 0 && t.K % 256 == 0 && t.N % 256 == 0;
        if (big) {
            const bool top = l == n.L - 1 && top_fused;
            BwdBf16Args u = {};
            u.M = M; u.K = t.K; u.N = t.N; u.NH = n.NH; u.NHP = n.NHP; u.splits = t.splits;
            u.ranges = resident ? bf16_dx_ranges(M, t.K, t.N, t.splits) : 0;
            u.rev = (n.L - 1 - l) % 2 == 0;
            u.xP = t.xP; u.dyP = t.dyP; u.hTop = actP(l); u.maskTop = at<const uint32_t>(h, L.mask[l]);
            // the mask of the layer below as flag words where the acting kernel writes them (every layer it runs
            // on the matrix cores; the first layer only at 512 columns)
            u.maskLo = (l - 1 >= 1 || n.dims[1] == 512) ? at<const uint32_t>(h, L.mask[l - 1]) : nullptr;
            u.dhead = at<const float>(h, L.dhead);
            u.wh16 = at<const uint16_t>(h, L.w16_src) + n.wh_off; u.w16 = at<const uint16_t>(h, L.w16_src) + n.w_off[l];
            u.dxP = dzP(l - 1);
            u.partial = t.partial; u.split_stride = t.split_stride;
            u.head_partial = at<float>(h, L.part[n.L]); u.head_stride = (size_t)t.N * n.NH + n.NH;
            ProfScope prof(h, !resident ? "gemm_tn" : top ? "gemm_tn_nt_top" : "gemm_tn_nt_256");
            if ((e = launch_backward_bf16_tiles(u, top, resident, h->stream)) != hipSuccess) return e;
        } else if (l == 0 && (e = run_tn(t, false, "gemm_tn_obs")) != hipSuccess) return e;
        if (l > 0 && !resident) {
            const bool both = !big;                              // one launch for both products
            GemmNtBf16Args g;
            g.M = M; g.K = n.dims[l]; g.N = n.dims[l + 1];
            g.dyR = dzR(l);
            g.w16 = at<const uint16_t>(h, L.w16_src) + n.w_off[l];
            g.hP = actP(l - 1);
            g.dxR = needs_rows(l - 1) ? dzR(l - 1) : nullptr;
            g.dxP = dzP(l - 1);
            if (fold) { g.dhead = t.dhead; g.maskTop = at<const uint32_t>(h, L.mask[l]); g.wh16 = t.wh16; g.NH = n.NH; g.NHP = n.NHP; }
            const bool first = first_fold && l == 1;
            g.nbx = first ? h->splits[0] : (M + 127) / 128;
            if (first) {
                g.f0 = at<const float>(h, L.tr_f0); g.f1 = at<const float>(h, L.tr_f1);
                g.first_partial = at<float>(h, L.part[0]); g.per = chunk_rows(M, h->splits[0], 128) / 128;
            }
            ProfScope prof(h, both ? "gemm_tn_nt" : "gemm_nt_mask");
            if (both) {
                t.tiles_i = (t.K + 127) / 128;
                const int tiles = t.tiles_i * ((t.N + 127) / 128), tn = tiles * t.splits;
                const size_t lds_t = (size_t)2 * TB_G * 128 * sizeof(uint4) + (fold ? 8192 : 0), lds_n = (size_t)2 * 128 * NB_LD * sizeof(uint16_t) + (fold ? 4096 : 0) + (first ? 3072 : 0);
                const size_t lds2 = lds_t > lds_n ? lds_t : lds_n;
                const auto kern = first ? gemm_tn_nt_bf16<true, true> : fold ? gemm_tn_nt_bf16<true, false> : gemm_tn_nt_bf16<false, false>;
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(kern, dim3(tn + g.nbx * ((g.K + 127) / 128)), dim3(WG), lds2, h->stream, t, g, tiles, tn);
            } else {
                const size_t lds2 = (size_t)2 * 128 * NB_LD * sizeof(uint16_t);
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_nt_bf16), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(gemm_nt_bf16, dim3(((g.M + 127) / 128) * ((g.K + 127) / 128)), dim3(WG), lds2, h->stream, g);
            }
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace ank
