// Both backward products of a bf16 layer in whole 256-wide tiles, side by side in one launch:
//   dW_l = h_{l-1}^T dZ_l              reduction over the M samples, one partial per chunk
//   dZ_{l-1} = (dZ_l W_l^T) masked     reduction over the N outputs
// with the head pass folded in where l is the top layer (dZ_L is then formed from the head gradient
// inside both products and never reaches memory).
//
// Why one launch: each product alone is limited by something the other leaves free.  A compute unit has about 32 KB
// of loads in flight, 45 GB/s of HBM latency (140 GB/s from L2); dW pulls 64 KB per 64 samples and tile, dX half of
// that, but writes its result.  A workgroup per compute unit for the whole launch, half of them dW and half dX, all
// walking the samples in stages of 32 in the same order: chunk c takes stages c, c + splits, ..., so that what is read
// and written together stands together in memory, and half as many partial sums of dW are written as with a chunk per
// compute unit.  Layers alternate between the two ends of the samples, so that a launch begins with what the one before
// wrote last (the last-level cache still holds it).
// Why loads straight into LDS: what goes through registers cost as many LDS stores (74 B per cycle) as the operands'
// reads (220) and half of the registers.  Stages are in flight 2 to 4 ahead, counted by hand (backward_bf16_order.h).
// dX needs dZ by rows where memory has eight samples per piece: the transposing LDS read hands out the operand, in an
// order of the features that W in registers follows; before, 2-byte stores turned each piece.
// Measured (768-512-512-512, 524288 samples; dW and dX before, both here, us): top layer 380 + 303 -> 557, middle one
// 295 + 285 -> 465, optimiser kernel 60.5 -> 52.7, the step 2216 -> 2000.  256-256, 262144 samples 168 + 68 -> 101;
// 512-512, 16384 samples 30 + 31 -> 35; 256-256, 512 samples 17.6 + 10.4 -> 15.5.
// What bounds them now, by the counters: the matrix cores are busy in 0.54 (top) and 0.61 (middle) of the cycles, and the
// clock stands at 1.9 GHz under both, as it does under the acting kernel (2.4 GHz nominal): 0.40 and 0.48 of the cores'
// peak.  1.44 and 1.68 GB are read past L2 and 0.57 written, 3.7 and 5.0 TB/s where a copy reaches 5.6: the middle layer is
// near the memory's rate.  Its reads are h, the flags and dZ_l twice: the dW and the dX workgroups of the same samples sit
// on different XCDs, and what the last-level cache serves of the second reading these counters do not see.
#include "gemm_bf16.h"
#include "backward_bf16_order.h"

namespace ank {

typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_c;
typedef __attribute__((address_space(3))) u4v lds_u4;
typedef __attribute__((address_space(3))) s4v lds_s4;
typedef __attribute__((address_space(3))) uint32_t lds_w;
typedef __attribute__((address_space(3))) float lds_f;
typedef __attribute__((address_space(3))) uint16_t lds_h;

namespace {

// Eight wavefronts, two per SIMD, 256 registers each: with four of twice the tile the wavefront's own waits leave its SIMD
// idle (dX alone 474 us instead of 387 on half of the compute units).
constexpr int BWD_WG = 512;
constexpr int LDS_ALL = 160 * 1024;

__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p; }
// One load of a wavefront from memory straight into LDS: 16 (4) bytes per lane from base + voff to the LDS byte address
// lds + 16 (4) * lane.  The compiler does not see these loads; wait_loads counts them.
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, const void* base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ void dma4(uint32_t lds, uint32_t voff, const void* base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(lds), "v"(voff), "s"(base) : "memory");
}
template <int OFF> __device__ __forceinline__ void store8(uint32_t voff, u2v v, const void* base)
{
    asm volatile("global_store_dwordx2 %0, %1, %2 offset:%3" : : "v"(voff), "v"(v), "s"(base), "n"(OFF) : "memory");
}
// all but the last N loads and stores of this wavefront are done, its LDS accesses too; then all wavefronts meet
template <int N> __device__ __forceinline__ void wait_loads_barrier()
{
    static_assert(N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}
__device__ __forceinline__ f16v zero16()
{
    f16v z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
    return z;
}
__device__ __forceinline__ f16v mma(u4v a, u4v b, f16v c) { return mfma_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c); }
// The same instruction with its result in ordinary registers (the compiler gives every MFMA of a function accumulation
// registers, and the tile of dW takes all of those), and with an operand that stays in accumulation registers.  It knows
// nothing of their latency: a result is read three MFMAs later at the earliest, or behind settle().
__device__ __forceinline__ void mma_new(f16v& d, u4v a, u4v b) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b)); }
__device__ __forceinline__ void mma_add(f16v& d, u4v a, u4v b) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b)); }
__device__ __forceinline__ void mma16_add(f4v& d, u4v a, u4v b) { asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b)); }
__device__ __forceinline__ void mma_new_w(f16v& d, u4v a, u4v w) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(w)); }
__device__ __forceinline__ void mma_add_w(f16v& d, u4v a, u4v w) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(w)); }
__device__ __forceinline__ void settle(f16v& d) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(d)); }
// both halves of a word of bfloat16 values added to c
__device__ __forceinline__ float add_pair(uint32_t w, float c)
{
    return c + (__builtin_bit_cast(float, w << 16) + __builtin_bit_cast(float, w & 0xffff0000u));
}
// where an operand's next stage begins; past the last one it stays there (what is loaded then is never used)
struct Cursor {
    const char* p; ptrdiff_t step;
    __device__ __forceinline__ void next(bool more) { p += more ? step : 0; }
};
// ---------------------------------------------------------------------------
// dW: one 256 x 256 tile of one chunk.  Wavefront (wm, wn) owns rows 128 wm.. and columns 64 wn.. of the tile, eight
// 32 x 32 accumulators.
// ---------------------------------------------------------------------------
// PARTS (top layer): how many halves of dWh of the tile's 256 columns this workgroup adds up.  SUMS: the column sums of dZ
template <bool TOP, int PARTS, bool SUMS>
__device__ __forceinline__ void dw_body(const BwdBf16Args& a, char* smem, const int split, const int ti, const int tj)
{
    using O = DwOrder<TOP, PARTS>;
    constexpr int STG = O::STG, NB = O::NB, NT = O::NT, DP = O::DP, D = O::D;
    constexpr int TST = 3072;                                              // top: mask words of 256 columns, head gradient
    constexpr int T0 = NB * STG, Z0 = T0 + NT * TST, A0 = Z0 + 2 * 16384, B0 = A0 + 3 * 1024, W0 = B0 + 3 * 1024, END = TOP ? W0 + 4096 : T0;
    static_assert(END <= LDS_ALL, "LDS");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3, l32 = lane & 31, kg = lane >> 5;
    const int i0 = ti * 256, j0 = tj * 256;
    const int total = a.M >> 5, n = (total - split + a.splits - 1) / a.splits;
    const uint32_t lds0 = lds_addr(smem);
    // loads: wavefront = (sample group of the stage, half of the 256 columns; PARTS = 1: of the 128 columns of h_L)
    const uint32_t vx = (uint32_t)((wave >> 1) * a.K + i0 + (wave & 1) * 128 + lane) * 16u;
    const uint32_t vy = (uint32_t)((wave >> 1) * a.N + j0 + (PARTS == 1 ? ti * 128 + (wave & 1) * 64 : (wave & 1) * 128) + lane) * 16u;
    // stage i of this chunk is stage i * splits + split of all samples, counted from the other end with a.rev
    const size_t st0 = (size_t)(a.rev ? total - 1 - split : split);
    const ptrdiff_t hop = a.rev ? -(ptrdiff_t)a.splits : (ptrdiff_t)a.splits;
    Cursor cx{reinterpret_cast<const char*>(a.xP) + st0 * 64 * a.K, hop * 64 * a.K};
    Cursor cy{reinterpret_cast<const char*>(TOP ? a.hTop : a.dyP) + st0 * 64 * a.N, hop * 64 * a.N};
    Cursor cm{reinterpret_cast<const char*>(a.maskTop + st0 * 2 * a.N + (size_t)(wave >> 2) * a.N + j0 + (wave & 3) * 64), hop * 8 * a.N};
    Cursor cd{reinterpret_cast<const char*>(a.dhead + (st0 * 32 + (wave & 3) * 8) * a.NHP), hop * 128 * a.NHP};
    int tslot = 0;                                                         // slot of the T ring that point_t's stage goes to
    auto load = [&](int slot, int k) {
        const uint32_t l = lds0 + (uint32_t)slot * STG + (uint32_t)(wave >> 1) * 4096u + (uint32_t)(wave & 1) * 2048u;
        if (k < 2) dma16(l + k * 1024u, vx + k * 1024u, cx.p);
        else if (k < DP) {
            if (PARTS == 1) dma16(lds0 + (uint32_t)slot * STG + 16384u + (uint32_t)wave * 1024u, vy, cy.p);
            else dma16(l + 16384u + (k - 2) * 1024u, vy + (k - 2) * 1024u, cy.p);
        } else {
            const uint32_t t = lds0 + T0 + (uint32_t)tslot * TST;
            if (k == DP) dma4(t + (uint32_t)wave * 256u, (uint32_t)lane * 4u, cm.p);        // mask words: (kg, quarter of the columns)
            else dma4(t + 2048u + (uint32_t)(wave & 3) * 256u, (uint32_t)(a.NHP == 8 ? lane : l32) * 4u, cd.p);   // eight rows of the head gradient; four wavefronts load what the others do
        }
    };
    f16v acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = zero16();
    f4v ex[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};      // dWh of 16 columns per part
    float bsum = 0.0f, dbsum = 0.0f;                                       // column sums
    // not the top layer: column tile t of a wavefront is tile (t + wm) % 2 of its 64 columns, so that the two wavefronts of a
    // column add up one tile each
    uint32_t ct[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) ct[t] = (uint32_t)(wn * 64 + ((TOP ? t : t + wm) & 1) * 32 + l32);
    const lds_c* const s3 = (const lds_c*)smem;
    const lds_c* const ldsx = s3 + (wm * 128 + l32) * 16 + kg * 4096;
    const lds_c* const ldsy0 = s3 + (TOP ? Z0 : 16384) + ct[0] * 16 + kg * 4096;
    const lds_c* const ldsy1 = s3 + (TOP ? Z0 : 16384) + ct[1] * 16 + kg * 4096;
    // operand k of step ks: 0 and 2 of dZ, the others of X; slot: of the loads (top: zs: of the formed dZ)
    struct Frag { u4v x[4], y[2]; };
    Frag F0, F1;
    auto rd = [&](Frag& f, int slot, int zs, int ks, int k) {
        const int o = slot * STG + ks * 8192, z = TOP ? zs * 16384 + ks * 8192 : o;
        if (k == 0) f.y[0] = *(const lds_u4*)(ldsy0 + z);
        else if (k == 2) f.y[1] = *(const lds_u4*)(ldsy1 + z);
        else f.x[k == 1 ? 0 : k - 2] = *(const lds_u4*)(ldsx + o + (k == 1 ? 0 : k - 2) * 512);
    };
    if constexpr (!TOP) {
        auto half = [&](const Frag& c, Frag& nx, int slot, int ks, bool ld, int lslot) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int i = s >> 1, j = s & 1;
                acc[i][j] = mma(c.x[i], c.y[j], acc[i][j]);
                if (s < 6) rd(nx, slot, 0, ks, s);
                if (ld && s >= 4) load(lslot, s - 4);
                if (SUMS && s < 4) bsum = add_pair(c.y[0][s], bsum);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int k = 0; k < D; ++k) load(b, k);
            cx.next(b + 1 < n); cy.next(b + 1 < n);
        }
        wait_loads_barrier<D * (NB - 1)>();
#pragma unroll
        for (int k = 0; k < 6; ++k) rd(F0, 0, 0, 0, k);
        int slot = 0;
        for (int i = 0; i < n; ++i) {
            const int nxt = slot + 1 == NB ? 0 : slot + 1;
            half(F0, F1, slot, 1, false, 0);
            wait_loads_barrier<O::LEFT>();
            half(F1, F0, nxt, 0, true, slot);
            cx.next(i + NB + 1 < n); cy.next(i + NB + 1 < n);
            slot = nxt;
        }
    } else {
        // dZ of a stage is formed by the eight wavefronts, 32 columns each, from the head gradient, in the layout the loads
        // give it otherwise.  Sample 16 j + 8 kg + 4 h + q of the stage sits in row 8 (2 j + h) + 4 kg + q of the A operand,
        // so that a lane's accumulators are eight consecutive samples of each step of 16.
        if (tid < 256) *reinterpret_cast<u4v*>(smem + W0 + tid * 16) = head_row(a.wh16, a.NH, j0 + tid);
        const int dm = (tid >> 3) & 31, dk = tid & 7;                      // head gradient: (sample of the stage, head output), the first four wavefronts
        const int drow = 8 * (2 * (dm >> 4) + ((dm >> 2) & 1)) + 4 * ((dm >> 3) & 1) + (dm & 3);
        const int draw = T0 + 2048 + (dm >> 3) * 256 + ((dm & 7) * a.NHP + (dk & (a.NHP - 1))) * 4;
        float raw = 0.0f;
        auto read_head = [&](int ts) { raw = *(const lds_f*)(s3 + ts * TST + draw); };
        auto forms = [&](int i, int p) {                                   // head gradient of stage i (raw) as both operands, place p
            if (wave >= 4) return;
            const float d = dk < a.NH ? raw : 0.0f;
            const uint16_t hi = (uint16_t)cvt_pk_bf16(d, 0.0f);
            const uint16_t lo = (uint16_t)cvt_pk_bf16(d - bf16_to_f(hi), 0.0f);
            lds_h* const A16 = (lds_h*)((lds_c*)smem + A0 + p * 1024);
            A16[drow * 8 + dk] = hi; A16[256 + drow * 8 + dk] = lo;
            if (PARTS) {
                lds_h* const B16 = (lds_h*)((lds_c*)smem + B0 + p * 1024) + ((dm >> 3) * 16 + dk) * 8 + (dm & 7);
                B16[0] = hi; B16[64] = lo;
                dbsum += i < n ? d : 0.0f;
            }
        };
        const lds_c* const ldsm = s3 + T0 + (wave * 32 + l32) * 4;
        lds_c* const ldsz = (lds_c*)smem + Z0 + (wave * 32 + l32) * 16 + kg * 4096;
        const lds_c* const ldsh = s3 + 16384 + (PARTS == 1 ? wave * 256 + (lane >> 4) * 2048 : wave * 512 + (lane >> 4) * 4096) + (lane & 15) * 16;
        f16v fz;
        uint32_t w0 = 0, w1 = 0;
        u4v fa, wc, z;
        auto form_words = [&](int ts) { w0 = *(const lds_w*)(ldsm + ts * TST); w1 = *(const lds_w*)(ldsm + ts * TST + 1024); };
        auto form_pair = [&](int p, bool counted) {                        // p: (step j, half h, pair of the half)
            const int j = p >> 2, h = (p >> 1) & 1, pr = p & 1, r = 4 * (2 * j + h) + 2 * pr;
            z[p & 3] = cvt_pk_bf16(fz[r], fz[r + 1]) & mask_pair(h ? w1 : w0, 4 * j + pr);
            if (SUMS) bsum = add_pair(z[p & 3] & (counted ? ~0u : 0u), bsum);
        };
        auto put = [&](int zs, int j) { *(lds_u4*)(ldsz + zs * 16384 + j * 8192) = z; };
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            tslot = b;
#pragma unroll
            for (int k = DP; k < D; ++k) load(0, k);
            cm.next(b + 1 < n); cd.next(b + 1 < n);
        }
        auto advance = [&](int i) { cx.next(i + 1 < n); cy.next(i + 1 < n); cm.next(i + 3 < n); cd.next(i + 3 < n); };   // from packet i to the next
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            tslot = b + 2;
#pragma unroll
            for (int k = 0; k < D; ++k) load(b, k);
            advance(b);
        }
        wait_loads_barrier<0>();
        for (int b = 0; b < 3; ++b) { read_head(b); forms(b, b); }
        __syncthreads();
        wc = *(const lds_u4*)(s3 + W0 + (wave * 32 + l32) * 16);
        for (int b = 0; b < 2; ++b) {                                      // stage 0, and the first half of stage 1
            fa = *(const lds_u4*)(s3 + A0 + b * 1024 + lane * 16);
            form_words(b);
            w0 >>= 2 * kg; w1 >>= 2 * kg;
            mma_new(fz, fa, wc);
            settle(fz);
#pragma unroll
            for (int p = 0; p < 4; ++p) form_pair(p, b < n);
            if (b == 0) {
                put(0, 0);
#pragma unroll
                for (int p = 4; p < 8; ++p) form_pair(p, true);
                put(0, 1);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; ++k) rd(F0, 0, 0, 0, k);
        int slot = 0, zs = 0, p0 = 0, p2 = 2, ts2 = 2, ts3 = 3;            // places of stage i: loads, dZ, head gradient; of i + 2 and i + 3
        tslot = 0;                                                         // T(i + NB + 2) goes where T(i) was
        u4v hx, hb;
        // half ks of a stage: the MFMAs of step ks with, between them, the operands of the next step, half of the work on dZ of
        // the stages to come, dWh of this stage, and in the second half the loads and the head gradient
        auto half = [&](const Frag& c, Frag& nx, int rslot, int rz, const int ks, int i) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                acc[s >> 1][s & 1] = mma(c.x[s >> 1], c.y[s & 1], acc[s >> 1][s & 1]);
                if (ks == 0) {
                    if (s == 0) put(zs ^ 1, 0);                            // stage i + 1: its first half was formed in the stage before
                    if (s == 4) put(zs ^ 1, 1);
                    if (PARTS && s == 5) hb = *(const lds_u4*)(s3 + B0 + p0 * 1024 + lane * 16);
                    if (PARTS && s == 6) hx = *(const lds_u4*)(ldsh + slot * STG);
                } else {
                    if (s == 0) { fa = *(const lds_u4*)(s3 + A0 + p2 * 1024 + lane * 16); form_words(ts2); }
                    if (s < D) load(slot, s);
                }
                if (s < 6) rd(nx, rslot, rz, 1 - ks, s);
                if (ks == 0) {
                    if (s < 4) form_pair(4 + s, i + 1 < n);
                    if (PARTS == 2 && s == 7) { mma16_add(ex[0], hx, hb); hx = *(const lds_u4*)(ldsh + slot * STG + 256); }
                } else {
                    if (PARTS && s == 1) mma16_add(ex[PARTS - 1], hx, hb);
                    if (s == 2) { mma_new(fz, fa, wc); w0 >>= 2 * kg; w1 >>= 2 * kg; }
                    if (s >= 5) form_pair(s - 5, i + 2 < n);
                    if (s == 7) form_pair(3, i + 2 < n);
                    if (s == 2) read_head(ts3);
                    if (s == 6) forms(i + 3, p0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int i = 0; i < n; ++i) {
            const int nxt = slot + 1 == NB ? 0 : slot + 1;
            half(F0, F1, slot, zs, 0, i);
            wait_loads_barrier<O::LEFT>();
            half(F1, F0, nxt, zs ^ 1, 1, i);
            advance(i + NB);
            slot = nxt; zs ^= 1;
            p2 = p0; p0 = p0 + 1 == 3 ? 0 : p0 + 1;
            ts2 = ts3; ts3 = ts3 + 1 == NT ? 0 : ts3 + 1; tslot = tslot + 1 == NT ? 0 : tslot + 1;
        }
    }
    wait_loads_barrier<0>();
    float* out = a.partial + (size_t)split * a.split_stride;
#pragma unroll
    for (int tr = 0; tr < 4; ++tr)
#pragma unroll
        for (int tc = 0; tc < 2; ++tc) {
            const int j = j0 + (int)ct[tc];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i0 + wm * 128 + tr * 32 + 8 * (r >> 2) + 4 * kg + (r & 3);
                out[(size_t)i * a.N + j] = acc[tr][tc][r];
            }
        }
    if (SUMS) {
        const float s = bsum + __shfl_xor(bsum, 32);                       // lanes kg = 0 and 1 hold half of the samples each
        if (kg == 0) out[(size_t)a.K * a.N + j0 + (TOP ? (uint32_t)(wave * 32 + l32) : ct[0])] = s;
    }
    if (PARTS) {
        float* hout = a.head_partial + (size_t)split * a.head_stride;
        const int jh = j0 + (PARTS == 1 ? ti * 128 : 0) + wave * 16 * PARTS;
#pragma unroll
        for (int c = 0; c < PARTS; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float s = ex[c][r] + __shfl(ex[c][r], (lane & 48) + ((lane + 8) & 15));   // hi and lo terms
                if ((lane & 15) < a.NH) hout[(size_t)(jh + c * 16 + 4 * (lane >> 4) + r) * a.NH + (lane & 15)] = s;
            }
        if (ti == 0 && tj == 0) {
            float* Sd = reinterpret_cast<float*>(smem);
            if (tid < 256) Sd[tid] = dbsum;
            __syncthreads();
            if (tid < a.NH) {
                float s = 0.0f;
                for (int m = 0; m < 32; ++m) s += Sd[m * 8 + tid];
                hout[(size_t)a.N * a.NH + tid] = s;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// dX: 256 output columns, one row range.  A wavefront keeps W of its 32 columns in registers (NR / 4 of them).
// ---------------------------------------------------------------------------
template <int NR, bool TOP, bool MASKW>
__device__ __forceinline__ void dx_body(const BwdBf16Args& a, char* smem, const int range, const int cb)
{
    using O = DxOrder<NR, TOP, MASKW>;
    constexpr int KS = O::KS, LA = O::LA, X = O::X, NY = O::NY, NL = O::NL, NT = O::NT, DL = O::DL, DM = O::DM, D = O::D, E0 = O::E0;
    constexpr int DY = NR * 64, LO = MASKW ? 2048 : 16384, TST = NR * 8 + 1024;
    constexpr int L0 = NY * DY, T0 = L0 + NL * LO, A0 = T0 + (TOP ? NT * TST : 0), END = A0 + (TOP ? 2 * 1024 : 0);
    static_assert(END <= LDS_ALL, "LDS");
    constexpr int TJ = NR / 256, FP = 16;                                  // TOP: 32-column tiles of dZ_L that a wavefront forms, slots between them
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kg = lane >> 5;
    const int total = a.M >> 5, n = (total - range + a.ranges - 1) / a.ranges;
    const int i0 = cb * 256 + wave * 32;                                   // this wavefront's columns
    const uint32_t lds0 = lds_addr(smem);
    const lds_c* const s3 = (const lds_c*)smem;
    // W: step s of the reduction covers features 16 s.., a lane's eight are 4 kg.. and 8 + 4 kg.. of them (the order in which the
    // transposing reads hand out dY)
    u4v w[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const uint16_t* p = a.w16 + (size_t)(i0 + l32) * NR + 16 * s + 4 * kg;
        const u2v lo = *reinterpret_cast<const u2v*>(p), hi = *reinterpret_cast<const u2v*>(p + 8);
        w[s][0] = lo[0]; w[s][1] = lo[1]; w[s][2] = hi[0]; w[s][3] = hi[1];
    }
    const size_t st0 = (size_t)(a.rev ? total - 1 - range : range);        // stages as in dw_body
    const ptrdiff_t hop = a.rev ? -(ptrdiff_t)a.ranges : (ptrdiff_t)a.ranges;
    Cursor cy{reinterpret_cast<const char*>(a.dyP) + st0 * 64 * NR, hop * 64 * NR};
    Cursor cl{MASKW ? reinterpret_cast<const char*>(a.maskLo + st0 * 2 * a.K) : reinterpret_cast<const char*>(a.xP) + st0 * 64 * a.K, hop * (MASKW ? 8 : 64) * a.K};
    Cursor cm{reinterpret_cast<const char*>(a.maskTop + st0 * 2 * NR), hop * 8 * NR};
    Cursor cd{reinterpret_cast<const char*>(a.dhead + (st0 * 32 + (wave & 3) * 8) * a.NHP), hop * 128 * a.NHP};
    char* out = reinterpret_cast<char*>(a.dxP) + st0 * 64 * a.K;           // the stage whose result is stored next
    const ptrdiff_t out_step = hop * 64 * a.K;
    // loads of dY: 16-byte piece (sample group g, feature n) goes to block n / 4 (256 bytes), place (g + n / 4) % 4, n % 4
    const uint32_t vdy = (uint32_t)((((lane >> 2) - (lane >> 4)) & 3) * NR + wave * (NR / 8) + 4 * (lane >> 4) + (lane & 3)) * 16u;
    const uint32_t vlo = (uint32_t)(kg * a.K + i0 + l32) * (MASKW ? 4u : 16u);
    const uint32_t vmt = NR == 512 ? (uint32_t)(wave * 64 + lane) * 4u : (uint32_t)(kg * NR + wave * 32 + l32) * 4u;
    const uint32_t vd = (uint32_t)(a.NHP == 8 ? lane : l32) * 4u;
    auto advance = [&](int p) { if (!TOP) cy.next(p + 1 < n); cl.next(p + 1 < n); if (TOP) { cm.next(p + 3 < n); cd.next(p + 3 < n); } };   // from packet p to the next
    int ls = 0, tsl = 0;                                                   // slots the next packet goes to
    auto load_t = [&](int k) {                                             // TOP: mask words of the wavefront's columns, rows of the head gradient
        const uint32_t t = lds0 + T0 + (uint32_t)tsl * TST;
        if (k < DM) dma4(t + (uint32_t)wave * NR + k * 256u, vmt + k * (NR * 4u), cm.p);
        else dma4(t + NR * 8u + (uint32_t)(wave & 3) * 256u, vd, cd.p);
    };
    auto load = [&](int k) {
        if (k < DL) {
            if (MASKW) dma4(lds0 + L0 + (uint32_t)ls * LO + (uint32_t)wave * 256u, vlo, cl.p);
            else dma16(lds0 + L0 + (uint32_t)ls * LO + (uint32_t)wave * 2048u + k * 1024u, vlo + (uint32_t)k * (uint32_t)a.K * 32u, cl.p);
        } else if (TOP) load_t(k - DL);
        else dma16(lds0 + (uint32_t)ls * DY + (uint32_t)wave * (DY / 8) + (uint32_t)(k - DL) * 1024u, vdy + (uint32_t)(k - DL) * 256u, cy.p);
    };
    // transposing reads of dY: a group of 16 lanes reads 4 features x 16 samples and hands each lane 4 features of one sample
    const int il = lane & 15, rg = 2 * ((lane >> 4) & 1) + ((il & 3) >> 1);
    const lds_c* const rd0 = s3 + kg * 256 + ((rg + kg) & 3) * 64 + (il >> 2) * 16 + (il & 1) * 8;
    const lds_c* const rd1 = s3 + (2 + kg) * 256 + ((rg + 2 + kg) & 3) * 64 + (il >> 2) * 16 + (il & 1) * 8;
    u4v fr[LA];
    auto rd = [&](int ks, int slot) {
        const u2v x = __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(rd0 + slot * DY + ks * 1024)));
        const u2v y = __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(rd1 + slot * DY + ks * 1024)));
        fr[ks % LA][0] = x[0]; fr[ks % LA][1] = x[1]; fr[ks % LA][2] = y[0]; fr[ks % LA][3] = y[1];
    };
    // result: rows 8 g + 4 kg + q of the stage, half of one packed group per g
    uint32_t vst[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) vst[g] = (uint32_t)(g * a.K + i0 + l32) * 16u + 8u * kg;
    struct Out { f16v acc; u2v m[4]; };                                    // a stage's result and its mask (one word: m[0][0])
    auto read_mask = [&](Out& o, int slot, int k) {
        const char* b = smem + L0 + slot * LO;
        if (MASKW) o.m[0][0] = *reinterpret_cast<const uint32_t*>(b + wave * 256 + lane * 4);
        else o.m[k] = *reinterpret_cast<const u2v*>(b + wave * 2048 + k * 512 + l32 * 16 + 8 * kg);
    };
    u2v pv;
    auto epi = [&](const Out& o, int k, char* base) {                      // word k & 1 of piece g = k >> 1; the second one stores
        const int g = k >> 1, h = k & 1, r = 4 * g + 2 * h;
        pv[h] = cvt_pk_bf16(o.acc[r], o.acc[r + 1]) & (MASKW ? mask_pair(o.m[0][0], 2 * g + h) : positive_mask_pk(o.m[g][h]));
        if (h) store8<0>(vst[g], pv, base);
    };
    // TOP: dZ_L of a stage, formed from the head gradient into the place the loads of dY have otherwise
    u4v wh[TOP ? TJ : 1], fa = {0u, 0u, 0u, 0u};
    uint32_t fw = 0;
    f16v fz = zero16();
    u2v fp;
    if (TOP) {
#pragma unroll
        for (int t = 0; t < TJ; ++t) wh[TOP ? t : 0] = head_row(a.wh16, a.NH, wave * (NR / 8) + 32 * t + l32);
    }
    const int dm = (tid >> 3) & 31, dk = tid & 7;
    const int draw = T0 + NR * 8 + (dm >> 3) * 256 + ((dm & 7) * a.NHP + (dk & (a.NHP - 1))) * 4;
    float raw = 0.0f;
    auto read_head = [&](int ts) { raw = *(const lds_f*)(s3 + ts * TST + draw); };
    auto forms = [&](int par) {                                            // the head gradient of a stage (raw) as (hi, lo) operand
        if (wave >= 4) return;
        const float d = dk < a.NH ? raw : 0.0f;
        const uint16_t hi = (uint16_t)cvt_pk_bf16(d, 0.0f);
        const uint16_t lo = (uint16_t)cvt_pk_bf16(d - bf16_to_f(hi), 0.0f);
        lds_h* const A16 = (lds_h*)((lds_c*)smem + A0 + par * 1024);
        A16[tid] = hi; A16[256 + tid] = lo;
    };
    uint32_t fo[4];                                                        // where group g of this lane's column goes inside its tile
#pragma unroll
    for (int g = 0; g < 4; ++g) fo[g] = (uint32_t)((wave * (NR / 32) + (l32 >> 2)) * 256 + ((g + (l32 >> 2)) & 3) * 64 + (l32 & 3) * 16 + 8 * kg);
    auto form_word = [&](int ts, int t) { fw = *reinterpret_cast<const uint32_t*>(smem + T0 + ts * TST + wave * NR + kg * (NR / 2) + (32 * t + l32) * 4); };
    auto form_pair = [&](int buf, int t, int p) {
        fp[p & 1] = cvt_pk_bf16(fz[2 * p], fz[2 * p + 1]) & mask_pair(fw, p);
        if (p & 1) *reinterpret_cast<u2v*>(smem + buf * DY + t * 2048 + fo[p >> 1]) = fp;
    };
    // what is put between the MFMAs of stage i: the operands LA steps ahead, the loads of packet i + X, the result of the
    // stage before (prev), the mask of this one, TOP: dZ_L of the next stage and the head gradient of the one after
    auto stage = [&](int i, int yslot, int ynext, int lslot, int ts1, int ts2, Out& cur, const Out& prev, bool first) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s == 0) mma_new_w(cur.acc, fr[0], w[0]); else mma_add_w(cur.acc, fr[s % LA], w[s]);
            if (s == O::WAIT_AT) { if (i >= X) wait_loads_barrier<O::LEFT>(); else wait_loads_barrier<O::LEFT_FIRST>(); }
            if (s + LA < KS) rd(s + LA, yslot); else rd(s + LA - KS, ynext);
            if (s < D) load(s);
            if (s < (MASKW ? 1 : 4)) read_mask(cur, lslot, s);
            if (s >= E0 && s < E0 + 8 && !first) epi(prev, s - E0, out);
            if (TOP) {
                const int t = s / FP < TJ ? s / FP : TJ - 1, u = s - t * FP;
                if (s == KS - LA + 1) fa = *reinterpret_cast<const u4v*>(smem + A0 + (i & 1) * 1024 + lane * 16);
                if (u == 0) form_word(ts1, t);
                if (u == 1) mma_new(fz, fa, wh[TOP ? t : 0]);
                if (u >= 4 && u < 12) form_pair(ynext, t, u - 4);
                if (s == KS - LA - 6) read_head(ts2);
                if (s == KS - LA - 2) forms(i & 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        advance(i + X);
        if (!first) out += out_step;
    };
    // beginning: the first packets, and stage 0 in its place
    if (TOP) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            tsl = b;
#pragma unroll
            for (int k = 0; k < DM + 1; ++k) load_t(k);
            cm.next(b + 1 < n); cd.next(b + 1 < n);
        }
    }
#pragma unroll
    for (int p = 0; p < X; ++p) {
        ls = p; tsl = p + 2;
#pragma unroll
        for (int k = 0; k < D; ++k) load(k);
        advance(p);
    }
    wait_loads_barrier<0>();
    if (TOP) {
        for (int b = 0; b < 2; ++b) { read_head(b); forms(b); }
        __syncthreads();
        fa = *reinterpret_cast<const u4v*>(smem + A0 + lane * 16);
#pragma unroll
        for (int t = 0; t < TJ; ++t) {
            mma_new(fz, fa, wh[TOP ? t : 0]);
            settle(fz);
            form_word(0, t);
#pragma unroll
            for (int p = 0; p < 8; ++p) form_pair(0, t, p);
        }
        fa = *reinterpret_cast<const u4v*>(smem + A0 + 1024 + lane * 16);
        __syncthreads();
    }
#pragma unroll
    for (int ks = 0; ks < LA; ++ks) rd(ks, 0);
    Out A, B;
    int ys = 0, lr = 0, t1 = 1, t2 = 2;
    ls = X; tsl = (X + 2) % NT;                                            // packet i + X goes to slot (i + X) % NL, T(i + X + 2) to (i + X + 2) % NT
    auto next = [&]() {
        ys = ys + 1 == NY ? 0 : ys + 1; lr = lr + 1 == NL ? 0 : lr + 1; ls = ls + 1 == NL ? 0 : ls + 1;
        t1 = t1 + 1 == NT ? 0 : t1 + 1; t2 = t2 + 1 == NT ? 0 : t2 + 1; tsl = tsl + 1 == NT ? 0 : tsl + 1;
    };
    auto yn = [&]() { return ys + 1 == NY ? 0 : ys + 1; };
    stage(0, ys, yn(), lr, t1, t2, A, B, true);
    next();
    int i = 1;
    for (; i + 1 < n; i += 2) {
        stage(i, ys, yn(), lr, t1, t2, B, A, false); next();
        stage(i + 1, ys, yn(), lr, t1, t2, A, B, false); next();
    }
    if (i < n) {
        stage(i, ys, yn(), lr, t1, t2, B, A, false);
        settle(B.acc);
#pragma unroll
        for (int k = 0; k < 8; ++k) epi(B, k, out);
    } else {
        settle(A.acc);
#pragma unroll
        for (int k = 0; k < 8; ++k) epi(A, k, out);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                       // no load into LDS outlives the workgroup
}

template <int NR, bool TOP, bool MASKW>
__global__ __launch_bounds__(BWD_WG, 1) void backward_bf16(const BwdBf16Args a)
{
    extern __shared__ uint4 smem4[];
    char* smem = reinterpret_cast<char*>(smem4);
    const int L = (int)blockIdx.x;
    int o, q;
    if (L < a.tn_blocks) {
        xcd_map(L, a.splits, a.tiles, o, q);                               // the tiles of a chunk share its samples
        const int ti = q % a.tiles_i, tj = q / a.tiles_i;
        if constexpr (!TOP) {
            if (ti == 0) dw_body<false, 0, true>(a, smem, o, ti, tj); else dw_body<false, 0, false>(a, smem, o, ti, tj);
        } else {
            if (a.tiles_i == 1) dw_body<true, 2, true>(a, smem, o, ti, tj);
            else if (ti == 0) dw_body<true, 1, true>(a, smem, o, ti, tj);
            else if (ti == 1) dw_body<true, 1, false>(a, smem, o, ti, tj);
            else dw_body<true, 0, false>(a, smem, o, ti, tj);              // (inputs of 768 and more)
        }
    } else {
        xcd_map(L - a.tn_blocks, a.ranges, a.K / 256, o, q);
        dx_body<NR, TOP, MASKW>(a, smem, o, q);
    }
}

template <int NR, bool TOP, bool MASKW>
hipError_t launch(const BwdBf16Args& a, int blocks, hipStream_t s)
{
    const void* fn = reinterpret_cast<const void*>(backward_bf16<NR, TOP, MASKW>);
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_ALL);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((backward_bf16<NR, TOP, MASKW>), dim3(blocks), dim3(BWD_WG), LDS_ALL, s, a);
    return hipGetLastError();
}

}  // namespace

// top: dZ_L from the head gradient.  dx: both products (N = 256 or 512), else dW alone.
hipError_t launch_backward_bf16_tiles(BwdBf16Args a, bool top, bool dx, hipStream_t s)
{
    a.tiles_i = a.K / 256; a.tiles = a.tiles_i * (a.N / 256); a.tn_blocks = a.splits * a.tiles;
    const int blocks = a.tn_blocks + (dx ? a.ranges * (a.K / 256) : 0);
    const bool mw = a.maskLo != nullptr;
    if (a.N == 512 && dx) {
        if (top) return mw ? launch<512, true, true>(a, blocks, s) : launch<512, true, false>(a, blocks, s);
        return mw ? launch<512, false, true>(a, blocks, s) : launch<512, false, false>(a, blocks, s);
    }
    if (top) return mw ? launch<256, true, true>(a, blocks, s) : launch<256, true, false>(a, blocks, s);
    return mw ? launch<256, false, true>(a, blocks, s) : launch<256, false, false>(a, blocks, s);
}

}  // namespace ank
