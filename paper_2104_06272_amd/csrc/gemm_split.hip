// Backward GEMMs of fp32 hidden layers on the bf16 matrix instructions, without giving up fp32 precision (paper
// section 3.2: the backward pass is the expensive half of the update).
//
// A binary32 value is the exact sum of three bfloat16 terms, x = h + m + l (8 + 8 + 8 significand bits, each the
// previous remainder rounded to nearest: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|; the range of "exact": split_terms.h).  A
// product of two such values is nine bfloat16 products, each exact in binary32; the six with the largest factors
//     h h,  h m,  m h,  m m,  h l,  l h
// leave out 2^-24 |a b| at most and 5e-9 |a b| (2^-27.5) in the root mean square (m l, l m, l l), no more than the rounding
// error of ONE binary32 operation, and every sum is accumulated in binary32 by the matrix instruction exactly as before.
// v_mfma_f32_32x32x16_bf16 does 16 reduction steps in 32 cycles, v_mfma_f32_32x32x2_f32 two in 64: six of the former
// replace eight of the latter, a 2.67 times shorter matrix-core time for the same sums.  Relative error of whole update
// gradients over 2080 samples against binary64 on the same stored forward pass, worst region of eight nets: 1.4e-7 with
// these kernels, 1.3e-7 with the vector-ALU ones; hidden-layer regions 6.6e-8 to 9.5e-8 against 6.4e-8 to 9.4e-8
// (test_split_products_keep_binary32).
//
//   gemm_tn   partial[s][i][j] = sum over chunk s of x[m][i] dY[m][j]   (+ column sums of dY)
//   gemm_nt   dX[m][i] = (x[m][i] > 0) * sum_j dY[m][j] W[i][j]
//
// For the top hidden layer both form dY on the way in from the layer's forward activations and the head gradient
// (HeadFuse), and gemm_tn also sums the head matrix's gradient.  gemm_nt can keep dZ_1 on chip and add up the first
// layer's gradient itself (FirstFuse): the pendulum's three features on the vector ALU, a Catch board of up to 64 cells as a
// 0/1 operand of the matrix instruction (12 MFMAs more per 32 x 32 results of 6 N/16).  For Catch this took the launch that
// read dZ_1 again: 256-256, 81920 samples 114.0 us and 22.6 for the first layer -> 115.1 for all; 64-64, 1048576 samples,
// whole step 499 -> 416 us; 128-128, 65536 samples 106 -> 92; 128-64, 64 samples 34.9 -> 30.1 us.  More cells: below.
//
// Operand layout of v_mfma_f32_32x32x16_bf16: lane l feeds A[row l%32][k 8 (l/32) .. +7] and B[k ..][col l%32];
// accumulator register r is D[row 8 (r/4) + 4 (l/32) + r%4][col l%32].
//
// What bounds them: at 256 x 256 a sample costs 0.63 ns of matrix-core time for both products on the whole chip (six
// MFMAs per product, see above) and 2 to 3 KB of traffic, 0.4 to 0.5 ns at the rate of a copy.  Both products side by side,
// half the compute units each: 81920 samples 200 -> 110 us, 262144 samples (pendulum) 580 -> 310 us against the binary32
// kernels they replace.  The matrix-core time of these is 51 and 164 us at 2.4 GHz, but the clock is at 2.1 and 2.0 GHz under
// them: of the launch's cycles the matrix cores are busy in 0.55 (with the board's share) and 0.61, vector instructions issue
// in 0.42, and a wavefront with an instruction at hand waits in 0.44 of its cycles.  With every sample read from L2 (the
// first 4096 over and over) the launches take 2 to 3 % less, so memory is not what bounds them, although 967 MB are read past
// L2 where reading h1 and h2 once would be 537 (the dW and the dX workgroup of the same samples drift apart).
#include "split_terms.h"
#include "detmath.h"

namespace ank {

constexpr int SWG = 512;                // eight wavefronts, two per SIMD

// the vector instructions since the last scheduling barrier between the n MFMAs since then, V behind each
template <int V> __device__ __forceinline__ void spread(int n)
{
#pragma unroll
    for (int k = 0; k < n; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
}

__device__ __forceinline__ f16v_s mfma_s(u4v_s a, u4v_s b, f16v_s c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8_s, a), __builtin_bit_cast(bf8_s, b), c, 0, 0, 0);
}
// the six products: terms of a and of b.  b's small terms are done with first, so that the next stage's can take their registers
constexpr int PROD_A[6] = {0, 1, 0, 2, 1, 0};
constexpr int PROD_B[6] = {2, 1, 1, 0, 0, 0};

// ---------------------------------------------------------------------------
// dW.  A workgroup owns a TI x TJ tile of the product for one chunk of samples and keeps the accumulators in registers.
// X and dY stream through LDS 16 WK samples at a time, double buffered, already split and packed as operands: a thread
// reads eight consecutive samples of one column (64 lanes: 256 contiguous bytes per sample), splits them and stores three
// 16-byte pieces.  WI x WJ wavefronts share the tile, WK of them the samples of a stage.
// One barrier per stage: while the MFMAs run on one half of LDS the same wavefronts split the next stage's values (asked
// for a whole stage earlier) into the other half.
// ROT: the barrier stands before the last MFMAs of a stage, whose operands are in registers by then, so that the reads of the
// next stage's first operands run beside them; and the split's vector instructions stand one by one between MFMAs rather than
// by the dozen, since a wavefront whose partner on the SIMD waits at the barrier has only its own MFMAs to cover them.  Both
// products of 256 x 256 tiles take 5.54 -> 5.11 million cycles (pendulum, 262144 samples: 323 -> 310 us, the clock falling from
// 1.98 to 1.93 GHz as the matrix cores get busier; Catch, 81920: 112.1 -> 109.8).  The other tiles have fewer MFMAs a stage and
// lose as often as they gain (256-128, 65536 to 524288 samples 2 % slower; 64-128 with five heads, 524288 samples, 177 -> 358 us
// for want of registers).  256 x 256 with five heads gains too (mazes, without and with: 256-256, 81920 samples 124.6 and 120.5 us,
// 524288 749 and 728; 512-512, 40000 samples 213 and 208), with five instructions behind an MFMA: with seven, as the other heads
// have, one register went to scratch, at the same speed.
// ---------------------------------------------------------------------------
template <int WI, int WJ, int AI, int AJ, int WK, int HEADS, bool ROT>
__device__ __forceinline__ void gemm_tn_split_body(const GemmTnArgs& a, const int split, const int i0, const int j0)
{
    static_assert(WI * WJ * WK == 8, "eight wavefronts");
    constexpr int TI = 32 * WI * AI, TJ = 32 * WJ * AJ, S = 16 * WK, GR = 2 * WK;
    constexpr int XP = TI * GR / SWG, YP = TJ * GR / SWG;        // pieces (eight samples of a column) per thread and stage
    static_assert(XP * SWG == TI * GR && YP * SWG == TJ * GR, "whole pieces");
    extern __shared__ float4 smem_s[];
    u4v_s* lds = reinterpret_cast<u4v_s*>(smem_s);               // [2][ X: 3 x GR x TI | Y: 3 x GR x TJ ]
    constexpr int XN = 3 * GR * TI, HALF = XN + 3 * GR * TJ;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, kg = lane >> 5;
    const int wk = wave / (WI * WJ), wi = (wave % (WI * WJ)) / WJ, wj = wave % WJ;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    const int n_stages = (m_end - m_begin + S - 1) / S;
    const float* ysrc = HEADS ? a.hf.hl : a.dy;
    struct Set { float x[XP][8], y[YP][8], d[HEADS ? YP : 1]; };
    Set S0, S1;                                                   // raw values of two stages in flight
    constexpr int HN = HEADS ? HEADS : 1, HP = HEADS > 4 ? 8 : 4;   // heads in the sums; of a row of the head gradient
    float bsum[YP], gwh[HEADS ? YP : 1][HN], gbh = 0.0f, wh[HEADS ? YP : 1][HN];
#pragma unroll
    for (int q = 0; q < YP; ++q) bsum[q] = 0.0f;
    if (HEADS) {
#pragma unroll
        for (int q = 0; q < YP; ++q)
#pragma unroll
            for (int k = 0; k < HN; ++k) {
                gwh[HEADS ? q : 0][k] = 0.0f;
                const int j = j0 + (q * SWG + tid) % TJ;
                wh[HEADS ? q : 0][k] = (k < a.hf.NH && j < a.N) ? head_weight(a.hf, j, k) : 0.0f;
            }
    }
    // loads of stage s, plain: a value past the end of the chunk or of the matrix is some other sample's, and is dropped
    // where the set is stored (a select right behind a load would wait for it).  A group of eight samples is uniform in a
    // wavefront, so the row part of every address is scalar.
    auto fetch_x = [&](Set& st, int s, int q) {
        {
            const int p = q * SWG + tid, c = i0 + p % TI, m = m_begin + s * S + 8 * (__builtin_amdgcn_readfirstlane(p / TI));
            const float* src = a.x + (size_t)(m < m_end ? m : m_begin) * a.K;
            const uint32_t co = c < a.K ? c : 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) st.x[q][e] = (src + (size_t)e * a.K)[co];
        }
    };
    auto fetch_y = [&](Set& st, int s, int q) {
        {
            const int p = q * SWG + tid, c = j0 + p % TJ, m = m_begin + s * S + 8 * (__builtin_amdgcn_readfirstlane(p / TJ));
            const int mc = m < m_end ? m : m_begin;
            const float* src = ysrc + (size_t)mc * a.ldy;
            const uint32_t co = c < a.N ? c : 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) st.y[q][e] = (src + (size_t)e * a.ldy)[co];
            // the eight samples' head gradients, one value per lane: lane HP e + k holds output k of sample e
            if (HEADS) st.d[HEADS ? q : 0] = a.hf.dhead[(size_t)(mc + ((lane / HP) & 7)) * HP + (lane & (HP - 1))];
        }
    };
    // Putting stage s (held in st) into half b of LDS, in units of a dozen vector instructions that go between MFMAs:
    // four pairs per X piece, then per Y piece eight samples' head terms (HEADS) and four pairs.  The unit that completes
    // a piece stores it and asks for the same piece of stage s + 2.
    constexpr int UX = 4, UY = HEADS ? 12 : 4, UNITS = XP * UX + YP * UY;
    u4v_s tt[3];
    float yv[8], gw[HN], live = 1.0f;
    auto unit = [&](Set& st, int b, int s, int u, bool refill) {
        if (u < XP * UX) {
            const int q = u / UX, i = u % UX, p = q * SWG + tid, c = p % TI, g = p / TI;
            // a stage of one group pair is whole or not there at all (and then never multiplied); a longer one can end early
            const bool ok = WK == 1 || m_begin + s * S + 8 * __builtin_amdgcn_readfirstlane(g) < m_end;
            split_pair(ok ? st.x[q][2 * i] : 0.0f, ok ? st.x[q][2 * i + 1] : 0.0f, tt, i);
            if (i == UX - 1) {
#pragma unroll
                for (int k = 0; k < 3; ++k) lds[b * HALF + (k * GR + g) * TI + c] = tt[k];
                if (refill) fetch_x(st, s + 2, q);
            }
            return;
        }
        const int v = u - XP * UX, q = v / UY, i = v % UY, p = q * SWG + tid, c = p % TJ, g = p / TJ;
        if (i == 0) {
            live = m_begin + s * S + 8 * __builtin_amdgcn_readfirstlane(g) < m_end ? 1.0f : 0.0f;
            if (HEADS) gbh = fmaf(live, st.d[HEADS ? q : 0], gbh);
#pragma unroll
            for (int k = 0; k < HN; ++k) gw[k] = 0.0f;
        }
        if (HEADS && i < 8) {
            float d[HN];
#pragma unroll
            for (int k = 0; k < HN; ++k) d[k] = f_from_bits((uint32_t)__builtin_amdgcn_readlane((int)bits_from_f(st.d[HEADS ? q : 0]), HP * i + k));
            float o = wh[HEADS ? q : 0][0] * d[0];
#pragma unroll
            for (int k = 1; k < HN; ++k) o = fmaf(wh[HEADS ? q : 0][k], d[k], o);
            const float hv = st.y[q][i < 8 ? i : 0];
#pragma unroll
            for (int k = 0; k < HN; ++k) gw[k] = fmaf(hv, d[k], gw[k]);
            yv[i < 8 ? i : 0] = hv > 0.0f ? o : 0.0f;
            return;
        }
        const int j = HEADS ? i - 8 : i;
        if (!HEADS) { yv[2 * j] = st.y[q][2 * j]; yv[2 * j + 1] = st.y[q][2 * j + 1]; }
        split_pair(yv[2 * j], yv[2 * j + 1], tt, j);
        if (j == 3) {
#pragma unroll
            for (int k = 0; k < 3; ++k) lds[b * HALF + XN + (k * GR + g) * TJ + c] = tt[k];
            bsum[q] = fmaf(live, ((yv[0] + yv[1]) + (yv[2] + yv[3])) + ((yv[4] + yv[5]) + (yv[6] + yv[7])), bsum[q]);
            if (HEADS) {
#pragma unroll
                for (int k = 0; k < HN; ++k) gwh[HEADS ? q : 0][k] = fmaf(live, gw[k], gwh[HEADS ? q : 0][k]);
            }
            if (refill) fetch_y(st, s + 2, q);
        }
    };
    f16v_s acc[AI][AJ];
#pragma unroll
    for (int i = 0; i < AI; ++i)
#pragma unroll
        for (int j = 0; j < AJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    auto fetch = [&](Set& st, int s) {
#pragma unroll
        for (int q = 0; q < XP; ++q) fetch_x(st, s, q);
#pragma unroll
        for (int q = 0; q < YP; ++q) fetch_y(st, s, q);
    };
    const int xb = (2 * wk + kg) * TI + wi * AI * 32 + l32, yb = XN + (2 * wk + kg) * TJ + wj * AJ * 32 + l32;
    // One step: the MFMAs of stage s on half cb of LDS, stage s + 1 (held in nxt) into the other half, nxt refilled with stage
    // s + 3.  ROT: the last row of tiles of stage s - 1, whose operands are in registers, then all rows of stage s but the last.
    u4v_s av[2][3], bv[3][AJ];
#pragma unroll
    for (int k = 0; ROT && k < 3; ++k) {
        av[1][k] = u4v_s{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < AJ; ++j) bv[k][j] = u4v_s{0, 0, 0, 0};
    }
    static_assert(AI % 2 == 0, "the last row of tiles is in av[1]");
    auto step = [&](Set& nxt, int cb, int s) {
        const u4v_s* X = lds + cb * HALF + xb;
        const u4v_s* Y = lds + cb * HALF + yb;
        // A unit of the next stage's split behind every few MFMAs: an MFMA keeps the matrix core busy for 32 cycles and its
        // wavefront for 4.  As a phase of its own the split was not covered by the other wavefront of the SIMD, which sits
        // between the same two barriers.
        constexpr int NM = 6 * AI * AJ;
        int done = 0, last = 0;
        auto read_x = [&](int i) {
#pragma unroll
            for (int k = 0; k < 3; ++k) av[i & 1][k] = X[k * GR * TI + 32 * i];
        };
        auto read_y = [&](int k) {
#pragma unroll
            for (int j = 0; j < AJ; ++j) bv[k][j] = Y[k * GR * TJ + 32 * j];
        };
        if (!ROT) { read_y(2); read_x(0); read_y(1); read_y(0); }
#pragma unroll
        for (int v = 0; v < AI; ++v) {
            const int i = !ROT ? v : v == 0 ? AI - 1 : v - 1;
            if (ROT || v + 1 < AI) read_x(ROT ? v : v + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
#pragma unroll
                for (int j = 0; j < AJ; ++j) {
                    acc[i][j] = mfma_s(av[i & 1][PROD_A[pr]], bv[PROD_B[pr]][j], acc[i][j]);
                    const int n = (v * 6 + pr) * AJ + j + 1;
                    if (n * UNITS / NM > done) {
                        if (!ROT) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (; done < n * UNITS / NM; ++done) unit(nxt, cb ^ 1, s + 1, done, true);
                        if (ROT) spread<(HEADS > 4 ? 5 : HEADS ? 7 : 4)>(n - last);
                        __builtin_amdgcn_sched_barrier(0);
                        last = n;
                    }
                }
                if (ROT && v == 0 && (pr == 5 || PROD_B[pr] != PROD_B[pr < 5 ? pr + 1 : 5])) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_y(PROD_B[pr]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        __syncthreads();
    };
    // S0's loads strictly before S1's, so that the wait counters can tell the two sets apart at the loop header
    fetch(S0, 0);
    __builtin_amdgcn_sched_barrier(0);
    fetch(S1, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) unit(S0, 0, 0, u, true);
    __syncthreads();
    int s = 0;
    for (; s + 1 < n_stages; s += 2) {
        step(S1, 0, s);
        step(S0, 1, s + 1);
    }
    if (s < n_stages) step(S1, 0, s);
#pragma unroll
    for (int pr = 0; ROT && pr < 6; ++pr)
#pragma unroll
        for (int j = 0; j < AJ; ++j) acc[AI - 1][j] = mfma_s(av[1][PROD_A[pr]], bv[PROD_B[pr]][j], acc[AI - 1][j]);
    float* out = a.partial + (size_t)split * ((size_t)a.K * a.N + a.N);
    if (WK > 1) {
        // the wavefronts that took other samples of the stages hand their sums over
        float* red = reinterpret_cast<float*>(lds) + (size_t)(wave % (WI * WJ)) * (AI * AJ * 1024);
        constexpr int PART = WI * WJ * AI * AJ * 1024;
        static_assert((WK - 1) * PART * 4 <= 2 * HALF * 16, "the sums fit the stages' LDS");
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < AI; ++i)
#pragma unroll
                for (int j = 0; j < AJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[(wk - 1) * PART + ((i * AJ + j) * 16 + r) * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (wk == 0) {
#pragma unroll
            for (int w = 0; w < WK - 1; ++w)
#pragma unroll
                for (int i = 0; i < AI; ++i)
#pragma unroll
                    for (int j = 0; j < AJ; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] += red[w * PART + ((i * AJ + j) * 16 + r) * 64 + lane];
        }
        __syncthreads();
    }
    if (wk == 0) {
#pragma unroll
        for (int i = 0; i < AI; ++i)
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                const int col = j0 + wj * AJ * 32 + 32 * j + l32;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = i0 + wi * AI * 32 + 32 * i + 8 * (r >> 2) + 4 * kg + (r & 3);
                    if (row < a.K && col < a.N) out[(size_t)row * a.N + col] = acc[i][j][r];
                }
            }
    }
    if (i0 != 0) return;
    // column sums (and the head matrix's gradient): the GR threads of a column add up in ascending sample-group order
    float* red = reinterpret_cast<float*>(lds);                  // [GR][TJ] sums, then [HN][GR][TJ]
    float* redh = red + GR * TJ;
    float* redb = redh + (HEADS ? HN * GR * TJ : 0);             // [SWG / TJ][64]
#pragma unroll
    for (int q = 0; q < YP; ++q) {
        const int p = q * SWG + tid, c = p % TJ, g = p / TJ;
        red[g * TJ + c] = bsum[q];
        if (HEADS) {
#pragma unroll
            for (int k = 0; k < HN; ++k) redh[(k * GR + g) * TJ + c] = gwh[HEADS ? q : 0][k];
        }
    }
    // every wavefront holds the head-bias sums of the sample groups it loaded; one of each kind hands them over
    if (HEADS && j0 == 0) {
        if ((tid % TJ) < 64) redb[(tid / TJ) * 64 + lane] = gbh;
    }
    __syncthreads();
    if (tid < TJ && j0 + tid < a.N) {
        float s = 0.0f;
#pragma unroll
        for (int g = 0; g < GR; ++g) s += red[g * TJ + tid];
        out[(size_t)a.K * a.N + j0 + tid] = s;
        if (HEADS) {
            float* hout = a.hf.head_partial + (size_t)split * ((size_t)a.N * a.hf.NH + a.hf.NH) + (size_t)(j0 + tid) * a.hf.NH;
#pragma unroll
            for (int k = 0; k < HN; ++k) {
                float sk = 0.0f;
#pragma unroll
                for (int g = 0; g < GR; ++g) sk += redh[(k * GR + g) * TJ + tid];
                if (k < a.hf.NH) hout[k] = sk;
            }
        }
    }
    if (HEADS && j0 == 0 && tid < a.hf.NH) {
        float s = 0.0f;
        for (int g = 0; g < SWG / TJ; ++g)
            for (int e = 0; e < 8; ++e) s += redb[g * 64 + HP * e + tid];
        a.hf.head_partial[(size_t)split * ((size_t)a.N * a.hf.NH + a.hf.NH) + (size_t)a.N * a.hf.NH + tid] = s;
    }
}

// ---------------------------------------------------------------------------
// dX.  A workgroup walks a range of samples, TR = 32 MT WM rows at a time, for 32 WN output columns: wavefront (wm, wn)
// owns rows 32 MT wm.., columns 32 wn...  dY comes through LDS 32 reduction indices at a time, double buffered, split
// and packed by its loader (a thread reads 32 contiguous bytes of a row); the split weights stream from L2 straight into
// registers, two steps of 16 ahead.  The pipeline runs across row tiles.  N is a multiple of 64, M of 8.
// Memory is addressed through buffer descriptors, one row tile each: rows past M read zero and are not written, and a row
// costs one scalar instruction instead of eight.
// ---------------------------------------------------------------------------
constexpr int NTS_KC = 32;
constexpr int NTS_SEG = 3072;           // samples whose features are in LDS at a time: 36 KB (Catch 12, and up to 64 of board), within what the dW product takes anyway
enum : int { FIRST_NONE = 0, FIRST_PENDULUM = 1, FIRST_CATCH = 2 };
struct STrue { static constexpr bool value = true; };
struct SFalse { static constexpr bool value = false; };

typedef __amdgpu_buffer_rsrc_t rsrc_s;
// rows [row0, row0 + rows) of a [M][ld] array of floats, as far as they exist
__device__ __forceinline__ rsrc_s rows_rsrc(const float* p, int row0, int rows, int M, int ld)
{
    int have = M - row0 < rows ? M - row0 : rows;
    asm("" : "+s"(have));                                        // or min and max become one vector instruction, and the
                                                                 // descriptor, then in vector registers, a loop per access
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + (size_t)row0 * ld, 0, (uint32_t)(have > 0 ? have : 0) * (uint32_t)ld * 4u, 0x00020000);
}
__device__ __forceinline__ float buf_load1(rsrc_s r, uint32_t voff, uint32_t soff) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0)); }
__device__ __forceinline__ f4v_s buf_load4(rsrc_s r, uint32_t voff, uint32_t soff) { return __builtin_bit_cast(f4v_s, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0)); }
__device__ __forceinline__ void buf_store1(float v, rsrc_s r, uint32_t voff, uint32_t soff) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, 0); }

template <int WN, int MT, int HEADS, int FIRST, bool ROT>
__device__ __forceinline__ void gemm_nt_split_body(const GemmNtArgs& a, const int tile0, const int tile1, const int by, const int part)
{
    constexpr int WM = 8 / WN, TR = 32 * MT * WM, PITCH = TR + 2, AP = TR * 4 / SWG;
    constexpr bool CATCH = FIRST == FIRST_CATCH;
    constexpr int CT = CATCH ? 2 : 1;                            // Catch: tiles of 32 cells (first_fused_splits: at most 64)
    constexpr int MP = MT < 2 ? MT : 2;                     // row tiles per turn of the epilogue
    static_assert(AP * SWG == TR * 4 && MT % MP == 0, "whole pieces, whole turns");
    extern __shared__ float4 smem_s[];
    u4v_s* As = reinterpret_cast<u4v_s*>(smem_s);                 // [2][3 terms][4 groups of 8 j][PITCH]
    constexpr int HALF = 3 * 4 * PITCH;
    f4v_s* whs = reinterpret_cast<f4v_s*>(As + 2 * HALF);         // HEADS: [N] head weights of a unit, the first four
    float* wh5 = reinterpret_cast<float*>(whs + (HEADS ? a.N : 0));   // HEADS > 4: [N] the fifth
    float* obsS = wh5 + (HEADS > 4 ? a.N : 0);   // FIRST: [3][NTS_SEG] features of a segment's samples; Catch: [2][NTS_SEG] cells, 16 bits each
    uint16_t* cellS = reinterpret_cast<uint16_t*>(obsS);
    u4v_s* boardS = reinterpret_cast<u4v_s*>(obsS + NTS_SEG);     // Catch: [TR / 16][CT][64] the board as operand
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, kg = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int N = a.N, NC = N / NTS_KC;
    const int ib = by * WN + wn;                                  // block of 32 output columns
    const bool live = ib * 32 < a.K;
    const int i = (live ? ib : 0) * 32 + l32;
    if (tile0 >= tile1) return;
    if (HEADS) {
        for (int j = tid; j < N; j += SWG) {
            f4v_s v;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = k < a.hf.NH ? head_weight(a.hf, j, k) : 0.0f;
            whs[j] = v;
            if (HEADS > 4) wh5[j] = head_weight(a.hf, j, 4);
        }
    }
    // loader: thread = (row, group of eight j)
    const int lrow = tid >> 2, lg = tid & 3;
    struct Set { f4v_s raw[AP][2], d[HEADS ? AP : 1]; float d5[HEADS > 4 ? AP : 1]; };
    Set S0, S1;                                                   // dY of two steps in flight
    const float* ysrc = HEADS ? a.hf.hl : a.dy;
    const uint32_t yoff = ((uint32_t)lrow * (uint32_t)N + 8u * (uint32_t)lg) * 4u, doff = (uint32_t)lrow * (uint32_t)a.hf.NHP * 4u;
    auto fetch = [&](Set& st, int tile, int c, int q) {
        const rsrc_s ry = rows_rsrc(ysrc, tile * TR + q * (SWG / 4), SWG / 4, a.M, N);
        st.raw[q][0] = buf_load4(ry, yoff, c * (NTS_KC * 4));
        st.raw[q][1] = buf_load4(ry, yoff + 16, c * (NTS_KC * 4));
        if (HEADS) {
            const rsrc_s rd = rows_rsrc(a.hf.dhead, tile * TR + q * (SWG / 4), SWG / 4, a.M, a.hf.NHP);
            st.d[HEADS ? q : 0] = buf_load4(rd, doff, 0);
            if (HEADS > 4) st.d5[HEADS > 4 ? q : 0] = buf_load1(rd, doff + 16, 0);
        }
    };
    // chunk c of dY (held in st) into half b of LDS, in units of about ten vector instructions that go between MFMAs: per
    // piece eight head terms (HEADS) and four pairs; the last one stores the piece and asks for the same of step + 3
    constexpr int UY = HEADS ? 12 : 4, UNITS = AP * UY;
    u4v_s tt[3];
    float yv[8];
    f4v_s wv;
    float wv5 = 0.0f;
    auto unit = [&](Set& st, int b, int c, int u, int tile_n, int c_n) {
        const int q = u / UY, v = u % UY;
        if (HEADS && v < 8) {
            const f4v_s w = v == 0 ? whs[c * NTS_KC + 8 * lg] : wv, d = st.d[HEADS ? q : 0];
            const float w5 = HEADS > 4 ? (v == 0 ? wh5[c * NTS_KC + 8 * lg] : wv5) : 0.0f;
            if (v < 7) wv = whs[c * NTS_KC + 8 * lg + (v < 7 ? v + 1 : 0)];
            if (HEADS > 4 && v < 7) wv5 = wh5[c * NTS_KC + 8 * lg + (v < 7 ? v + 1 : 0)];
            const float h = st.raw[q][(v < 8 ? v : 0) >> 2][v & 3];
            float o = w[0] * d[0];
            o = fmaf(w[1], d[1], o); o = fmaf(w[2], d[2], o); o = fmaf(w[3], d[3], o);
            if (HEADS > 4) o = fmaf(w5, st.d5[HEADS > 4 ? q : 0], o);
            yv[v < 8 ? v : 0] = h > 0.0f ? o : 0.0f;
            return;
        }
        const int j = HEADS ? v - 8 : v;
        if (!HEADS) { yv[2 * j] = st.raw[q][j >> 1][(2 * j) & 3]; yv[2 * j + 1] = st.raw[q][j >> 1][(2 * j + 1) & 3]; }
        split_pair(yv[2 * j], yv[2 * j + 1], tt, j);
        if (j == 3) {
#pragma unroll
            for (int k = 0; k < 3; ++k) As[b * HALF + (k * 4 + lg) * PITCH + q * (SWG / 4) + lrow] = tt[k];
            fetch(st, tile_n, c_n, q);
        }
    };
    const u4v_s* wb = reinterpret_cast<const u4v_s*>(a.w3) + (size_t)(live ? ib : 0) * (N >> 4) * 3 * 64 + lane;
    u4v_s bw[2][3];
    auto load_b = [&](int d, int ks) {
#pragma unroll
        for (int k = 0; k < 3; ++k) bw[d][k] = wb[(ks * 3 + k) * 64];
    };
    // pendulum: cos, sin and angular velocity of the samples of a segment of tiles, a bf16 net's rounded as its forward pass
    // read them (outside the tile loop: the constants of
    // sine and cosine alone would take twenty scalar registers there)
    auto features = [&](int t0, int t1) {
        for (int u = tid; u < (t1 - t0) * TR; u += SWG) {
            int m = t0 * TR + u;
            m = m < a.M ? m : a.M - 1;
            if (CATCH) {
                const uint32_t w = a.ff.s0[m];
                cellS[u] = (uint16_t)(((w >> 8) & 0xffu) * (uint32_t)a.ff.cols + (w & 0xffu));
                cellS[NTS_SEG + u] = (uint16_t)((uint32_t)a.ff.paddle_row0 + ((w >> 16) & 0xffu));
                continue;
            }
            float sn, cs;
            det_sincos(a.ff.f0[m], sn, cs);
            float td = a.ff.f1[m];
            if (a.bf16) { cs = bf16_to_f(bf16_bits(cs)); sn = bf16_to_f(bf16_bits(sn)); td = bf16_to_f(bf16_bits(td)); }
            obsS[u] = cs; obsS[NTS_SEG + u] = sn; obsS[2 * NTS_SEG + u] = td;
        }
    };
    // Catch: the boards of a tile as the A operand of dW_1, for each 16 of its samples and 32 cells, an entry 1 where the ball or
    // the paddle is in the lane's cell; a lane half has the samples 4 kg.. and 8 + 4 kg.. of the sixteen, in the order in which
    // the accumulators of dX hold them
    auto boards = [&](int first) {
        typedef uint32_t u2v_s __attribute__((ext_vector_type(2)));
        for (int p = wave; p < TR / 16; p += SWG / 64) {
            const uint16_t* s = cellS + first + 16 * p + 4 * kg;
            const u2v_s b0 = *reinterpret_cast<const u2v_s*>(s), b1 = *reinterpret_cast<const u2v_s*>(s + 8);
            const u2v_s p0 = *reinterpret_cast<const u2v_s*>(s + NTS_SEG), p1 = *reinterpret_cast<const u2v_s*>(s + NTS_SEG + 8);
            const uint32_t ball[4] = {b0[0], b0[1], b1[0], b1[1]}, pad[4] = {p0[0], p0[1], p1[0], p1[1]}, one = 0x00010001u;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const uint32_t cell = (uint32_t)(32 * ct + l32) * 0x00010001u;
                u4v_s v;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t x, y;                                // 1 in a half whose cell is this lane's, else 0 (a saturating subtraction)
                    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(x) : "v"(one), "v"(ball[i] ^ cell));
                    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(y) : "v"(one), "v"(pad[i] ^ cell));
                    v[i] = (x | y) * 0x3f80u;
                }
                boardS[(p * CT + ct) * 64 + lane] = v;
            }
        }
    };
    float gw0 = 0.0f, gw1 = 0.0f, gw2 = 0.0f, gb = 0.0f;
    f16v_s acc1[CT];                                              // Catch: dW_1
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc1[ct][r] = 0.0f;
    f16v_s acc[MT];
    auto clear = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][r] = 0.0f;
    };
    const uint32_t kb = (uint32_t)a.K * 4u;
    const uint32_t xoff = (uint32_t)(4 * kg) * kb + (uint32_t)i * 4u;
    // a row's offset in its tile; worked out again wherever it is used (from a value the compiler cannot see through): the
    // 64 of them kept across the loop would not fit the scalar registers
    auto row_off = [&](uint32_t k4, int mt, int r) { return (uint32_t)((wm * MT + mt) * 32 + 8 * (r >> 2) + (r & 3)) * k4; };
    auto opaque = [](uint32_t k4) { asm volatile("" : "+s"(k4)); return k4; };
    float xm[MP][16];
    auto load_mask = [&](rsrc_s rx, int mt0) {
        const uint32_t k4 = opaque(kb);
#pragma unroll
        for (int u = 0; u < MP; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) xm[u][r] = buf_load1(rx, xoff, row_off(k4, mt0 + u, r));
    };
    // One step: the MFMAs of 32 reduction indices (chunk c) on half par of LDS; the next step's dY (chunk c + 1, held in
    // nxt) into the other half between them, nxt refilled with the step after next's successor; the weights of the same
    // half of the next step asked for.  LAST: the step that completes a tile also asks for the first ReLU masks.
    // ROT: the last six, whose operands are in registers, are left to the next step (CONT: a tile's first has none to finish).
    u4v_s av[2][3];
    auto read_a = [&](int par, int p) {
        const u4v_s* A = As + par * HALF + (wm * MT * 32) + l32;
#pragma unroll
        for (int k = 0; k < 3; ++k) av[p & 1][k] = A[(k * 4 + 2 * (p / MT) + kg) * PITCH + 32 * (p % MT)];
    };
    auto finish = [&]() {
#pragma unroll
        for (int pr = 0; pr < 6; ++pr) acc[MT - 1] = mfma_s(av[1][PROD_A[pr]], bw[1][PROD_B[pr]], acc[MT - 1]);
    };
    auto step = [&](auto CONT, auto LAST, Set& nxt, int par, int tile, int c) {
        const int cn = c + 1 < NC ? c + 1 : 0;
        const int t3 = c + 3 < NC ? tile : c + 3 < 2 * NC ? tile + 1 : tile + 2;   // (two steps a tile where N is 64)
        const int c3 = c + 3 - (t3 - tile) * NC;
        if (LAST.value) {
            load_mask(rows_rsrc(a.x, tile * TR, TR, a.M, a.K), 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the six MFMAs of a row tile are one dependent chain; the other wavefront of the SIMD fills its gaps
        constexpr int P0 = ROT && CONT.value ? -1 : 0, NP = 2 * MT - ROT, NM = 6 * (NP - P0);
        if (!ROT || CONT.value) read_a(par, 0);
        int done = 0, last = 0;
#pragma unroll
        for (int p = P0; p < NP; ++p) {
            const int q = p < 0 ? 2 * MT - 1 : p, ks = q / MT, mt = q % MT;
            if (p >= 0 && p + 1 < 2 * MT) read_a(par, p + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
                acc[mt] = mfma_s(av[q & 1][PROD_A[pr]], bw[ks][PROD_B[pr]], acc[mt]);
                const int n = (p - P0) * 6 + pr + 1;
                if (n * UNITS / NM > done) {
                    if (!ROT) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (; done < n * UNITS / NM; ++done) unit(nxt, par ^ 1, cn, done, t3, c3);
                    if (ROT) spread<4>(n - last);
                    __builtin_amdgcn_sched_barrier(0);
                    last = n;
                }
            }
            if (mt == MT - 1) {
                load_b(ks, p < 0 ? 2 * c + 1 : 2 * cn + ks);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
#pragma unroll
    for (int q = 0; q < AP; ++q) fetch(S0, tile0, 0, q);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < AP; ++q) fetch(S1, tile0, 1, q);
    __builtin_amdgcn_sched_barrier(0);
    load_b(0, 0); load_b(1, 1);
    clear();
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UNITS; ++u) unit(S0, 0, 0, u, NC == 2 ? tile0 + 1 : tile0, NC == 2 ? 0 : 2);
    __syncthreads();
    for (int seg = tile0; seg < tile1; seg += NTS_SEG / TR) {
    const int seg1 = FIRST == FIRST_NONE || tile1 - seg < NTS_SEG / TR ? tile1 : seg + NTS_SEG / TR;
    if (FIRST != FIRST_NONE) {
        if (seg > tile0) __syncthreads();                         // the last segment's are still read
        features(seg, seg1);
        __syncthreads();
    }
    for (int tile = seg; tile < seg1; ++tile) {
        if (ROT) read_a(0, 0);
        step(SFalse(), SFalse(), S1, 0, tile, 0);
        __syncthreads();
        for (int c = 1; c + 1 < NC; c += 2) {
            step(STrue(), SFalse(), S0, 1, tile, c);
            __syncthreads();
            step(STrue(), SFalse(), S1, 0, tile, c + 1);
            __syncthreads();
        }
        if (CATCH) boards((tile - seg) * TR);                     // (the last tile's are read before the barrier above)
        step(STrue(), STrue(), S0, 1, tile, NC - 1);
        __syncthreads();
        if (ROT) {
            finish();
            load_b(1, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const rsrc_s rx = rows_rsrc(a.x, tile * TR, TR, a.M, a.K), rd = rows_rsrc(a.dx, tile * TR, TR, a.M, a.K);
#pragma unroll
        for (int mp = 0; mp < MT; mp += MP) {
            float o[MP][16];
#pragma unroll
            for (int u = 0; u < MP; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[u][r] = xm[u][r] > 0.0f ? acc[mp + u][r] : 0.0f;   // rows past M read as zero
            if (mp + MP < MT) load_mask(rx, mp + MP);
            if (FIRST == FIRST_NONE) {
                if (live) {
                    const uint32_t k4 = opaque(kb);
#pragma unroll
                    for (int u = 0; u < MP; ++u)
#pragma unroll
                        for (int r = 0; r < 16; ++r) buf_store1(o[u][r], rd, xoff, row_off(k4, mp + u, r));
                }
            } else if (CATCH) {
#pragma unroll
                for (int u = 0; u < MP; ++u)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {                 // 16 samples: dZ_1 in three terms against the 0/1 board leaves nothing out
                        u4v_s t1[3];
#pragma unroll
                        for (int q = 0; q < 4; ++q) split_pair(o[u][8 * j + 2 * q], o[u][8 * j + 2 * q + 1], t1, q);
                        gb += ((o[u][8 * j] + o[u][8 * j + 1]) + (o[u][8 * j + 2] + o[u][8 * j + 3])) + ((o[u][8 * j + 4] + o[u][8 * j + 5]) + (o[u][8 * j + 6] + o[u][8 * j + 7]));
                        u4v_s b[CT];
#pragma unroll
                        for (int ct = 0; ct < CT; ++ct) b[ct] = boardS[(((wm * MT + mp + u) * 2 + j) * CT + ct) * 64 + lane];
#pragma unroll
                        for (int k = 2; k >= 0; --k)
#pragma unroll
                            for (int ct = 0; ct < CT; ++ct) acc1[ct] = mfma_s(b[ct], t1[k], acc1[ct]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            } else {
#pragma unroll
                for (int u = 0; u < MP; ++u)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float* f = obsS + (tile - seg) * TR + (wm * MT + mp + u) * 32 + 8 * g + 4 * kg;
                        const f4v_s f0 = *reinterpret_cast<const f4v_s*>(f), f1 = *reinterpret_cast<const f4v_s*>(f + NTS_SEG), f2 = *reinterpret_cast<const f4v_s*>(f + 2 * NTS_SEG);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float v = o[u][4 * g + q];
                            gw0 = fmaf(f0[q], v, gw0); gw1 = fmaf(f1[q], v, gw1); gw2 = fmaf(f2[q], v, gw2); gb += v;
                        }
                        if (g & 1) __builtin_amdgcn_sched_barrier(0);   // six reads at a time: all of them at once do not fit the registers
                    }
            }
        }
        clear();
    }
    if (FIRST == FIRST_NONE) break;
    }
    if (FIRST != FIRST_NONE && WM > 1) __syncthreads();           // the sums go where operands are read
    if (CATCH) {
        gb += __shfl_xor(gb, 32, 64);
        float* red = reinterpret_cast<float*>(As);                // WM > 1: the row groups add up in ascending order
        float* redb = red + (WM - 1) * WN * CT * 1024;
        static_assert(((WM - 1) * WN * (CT * 1024 + 32)) * 4 <= 2 * HALF * 16, "the sums fit the operands' LDS");
        if (WM > 1) {
            if (wm > 0) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[((wm - 1) * WN + wn) * (CT * 1024) + (ct * 16 + r) * 64 + lane] = acc1[ct][r];
                if (kg == 0) redb[((wm - 1) * WN + wn) * 32 + l32] = gb;
            }
            __syncthreads();
            if (wm == 0) {
#pragma unroll
                for (int w = 0; w < WM - 1; ++w) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc1[ct][r] += red[(w * WN + wn) * (CT * 1024) + (ct * 16 + r) * 64 + lane];
                    gb += redb[(w * WN + wn) * 32 + l32];
                }
            }
        }
        if (wm == 0 && live) {
            float* out = a.ff.partial + (size_t)part * ((size_t)a.ff.cells * a.K + a.K) + i;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int cell = 32 * ct + 8 * (r >> 2) + 4 * kg + (r & 3);
                    if (cell < a.ff.cells) out[(size_t)cell * a.K] = acc1[ct][r];
                }
            if (kg == 0) out[(size_t)a.ff.cells * a.K] = gb;
        }
    }
    if (FIRST == FIRST_PENDULUM) {
        gw0 += __shfl_xor(gw0, 32, 64); gw1 += __shfl_xor(gw1, 32, 64); gw2 += __shfl_xor(gw2, 32, 64); gb += __shfl_xor(gb, 32, 64);
        f4v_s* red = reinterpret_cast<f4v_s*>(As);                // WM > 1: the row groups add up in ascending order
        f4v_s v = {gw0, gw1, gw2, gb};
        if (WM > 1) {
            if (kg == 0) red[wave * 32 + l32] = v;
            __syncthreads();
            if (wm == 0 && kg == 0) {
#pragma unroll
                for (int w = 1; w < WM; ++w) v += red[(w * WN + wn) * 32 + l32];
            }
        }
        if (wm == 0 && kg == 0 && live) {
            float* out = a.ff.partial + (size_t)part * (4 * (size_t)a.K);
            out[i] = v[0]; out[(size_t)a.K + i] = v[1]; out[2 * (size_t)a.K + i] = v[2]; out[3 * (size_t)a.K + i] = v[3];
        }
    }
}

// both products of a layer in one launch: dW workgroups first, dX workgroups behind them
template <int WI, int WJ, int AI, int AJ, int WK, int WN, int MT, int HEADS, int FIRST>
__global__ __launch_bounds__(SWG) void gemm_tn_nt_split(const GemmTnArgs t, const GemmNtArgs n, const int tn_blocks, const int tiles_j,
                                                        const int nt_bx, const int tiles_per_block)
{
    constexpr bool ROT = WI * AI == 8;                            // tiles of 256 x 256
    int b = (int)blockIdx.x;
    if (b < tn_blocks) {
        const int tile = b % (t.tiles_i * tiles_j), split = b / (t.tiles_i * tiles_j);
        gemm_tn_split_body<WI, WJ, AI, AJ, WK, HEADS, ROT>(t, split, (tile % t.tiles_i) * 32 * WI * AI, (tile / t.tiles_i) * 32 * WJ * AJ);
        return;
    }
    b -= tn_blocks;
    constexpr int TR = 32 * MT * (8 / WN);
    const int tiles = (n.M + TR - 1) / TR, bx = b % nt_bx, by = b / nt_bx;
    int t0 = bx * tiles_per_block, t1 = t0 + tiles_per_block < tiles ? t0 + tiles_per_block : tiles;
    asm("" : "+s"(t0), "+s"(t1));                                 // (the division above is done in vector registers)
    gemm_nt_split_body<WN, MT, HEADS, FIRST, ROT>(n, t0, t1, by, bx);
}

template <int WI, int WJ, int AI, int AJ, int WK, int WN, int MT>
static hipError_t launch_split_tiles(GemmTnArgs t, const GemmNtArgs& n, int nt_blocks, hipStream_t s)
{
    constexpr int TI = 32 * WI * AI, TJ = 32 * WJ * AJ, TR = 32 * MT * (8 / WN), TC = 32 * WN;
    t.tiles_i = t.K / TI;
    const int tiles_j = t.N / TJ, tn = t.tiles_i * tiles_j * t.splits;
    const int tiles = (n.M + TR - 1) / TR, per = (tiles + nt_blocks - 1) / nt_blocks, bx = (tiles + per - 1) / per, by = (n.K + TC - 1) / TC;
    const size_t lds_tn = (size_t)2 * 3 * 2 * WK * (TI + TJ) * 16;
    const size_t lds_nt = (size_t)2 * 3 * 4 * (TR + 2) * 16 + (n.hf.hl ? n.N * (n.hf.NH > 4 ? 20 : 16) : 0) + (n.ff.f0 ? NTS_SEG * 12 : n.ff.s0 ? NTS_SEG * 4 + TR / 16 * 2048 : 0);
    const size_t lds = lds_tn > lds_nt ? lds_tn : lds_nt;
    // (five heads: the maze, whose first layer is no part of these products)
    auto kern = n.ff.f0 ? (t.hf.hl ? gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 4, FIRST_PENDULUM> : gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 0, FIRST_PENDULUM>)
              : n.ff.s0 ? (t.hf.hl ? gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 4, FIRST_CATCH> : gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 0, FIRST_CATCH>)
              : !t.hf.hl ? gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 0, FIRST_NONE>
              : t.hf.NH > 4 ? gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 5, FIRST_NONE> : gemm_tn_nt_split<WI, WJ, AI, AJ, WK, WN, MT, 4, FIRST_NONE>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(tn + bx * by), dim3(SWG), lds, s, t, n, tn, tiles_j, bx, per);
    return hipGetLastError();
}

// the tile sizes of split_tile_i / split_tile_j / split_nt_rows; stages of 16 samples, 32 or 64 where a tile has fewer
// pieces than threads, the wavefronts that the tile leaves over sharing a stage's samples
hipError_t launch_gemm_tn_nt_split(const NetShape& net, int l, const GemmTnArgs& t, const GemmNtArgs& n, int nt_blocks, hipStream_t s)
{
    const int ti = split_tile_i(net, l), tj = split_tile_j(net, l);
    if (net.split == 2) {
        if (ti == 128) return tj == 128 ? launch_split_tiles<2, 2, 2, 2, 2, 2, 1>(t, n, nt_blocks, s) : launch_split_tiles<2, 1, 2, 2, 4, 2, 1>(t, n, nt_blocks, s);
        return tj == 128 ? launch_split_tiles<1, 2, 2, 2, 4, 2, 1>(t, n, nt_blocks, s) : launch_split_tiles<1, 2, 2, 1, 4, 2, 1>(t, n, nt_blocks, s);
    }
    if (ti == 256) return launch_split_tiles<2, 4, 4, 2, 1, 8, 4>(t, n, nt_blocks, s);
    if (ti == 128) {
        if (split_nt_cols(net, l) == 256)
            return tj == 128 ? launch_split_tiles<2, 2, 2, 2, 2, 8, 4>(t, n, nt_blocks, s) : launch_split_tiles<2, 1, 2, 2, 4, 8, 4>(t, n, nt_blocks, s);
        return tj == 128 ? launch_split_tiles<2, 2, 2, 2, 2, 4, 2>(t, n, nt_blocks, s) : launch_split_tiles<2, 1, 2, 2, 4, 4, 2>(t, n, nt_blocks, s);
    }
    return tj == 128 ? launch_split_tiles<1, 2, 2, 2, 4, 2, 2>(t, n, nt_blocks, s) : launch_split_tiles<1, 2, 2, 1, 4, 2, 2>(t, n, nt_blocks, s);
}

}  // namespace ank
