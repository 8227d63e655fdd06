// Gradient of the first layer for boards (paper section 3.1: the update differentiates through the policy network).  The
// observation of a grid environment is a 0/1 board with one or two cells set per changing plane, so dW_1 = X^T dZ_1 needs
// no X in memory: the board is rebuilt from the 4-byte state of a sample, as the 0/1 operand of the matrix instruction.
//
//   first_layer_onehot   Catch: rows = cells, two of them set per sample (fp32 boards of up to 64 cells above a second layer
//                        in whole 64-wide tiles: gemm_split.hip instead).  Maze: the agent's plane, one cell per sample,
//                        and the plane of walls, which is the same all through an unroll and so needs only
//                        S[b] = sum_t dZ_1[t][b]; the goal's plane has one cell that is always set: the column sums.
//
//   first_layer_pendulum_bf16   the pendulum's three features, bf16 matrix path (most nets of two layers with a 128-wide one:
//                               learn_bf16.hip's dX product instead)
//
// dZ_1 comes as binary32 rows (taken apart into three bfloat16 terms: every product with a 0/1 operand is exact and the
// accumulation is binary32, see split_terms.h) or as the sample-packed bfloat16 of the bf16 matrix path (one term).
#include "onehot.h"

namespace ank {

struct FirstOneHotArgs {
    int B, T, N, cells;
    int units, per;           // units of 16 samples, and how many of them a chunk has
    int tiles_wg;             // column tiles (of 32) per workgroup
    int cols, paddle_row0;    // Catch: board columns, first cell of the bottom row
    const void* dy;           // [M][N] binary32, or packed [M/8][N][8] bfloat16
    const uint32_t* s0;       // [M] states
    const uint32_t* walls;    // maze: [8][B]
    float* out;               // Catch: [splits][cells*N + N].  Maze: agent plane [splits][cells*N]
    float* walls_out;         // maze: [splits][cells*N]
    float* sums_out;          // maze: [splits][N]
};

// What a wavefront holds of one unit: eight samples (16 g' + 8 kg + 0..7) of its column, and their states.
template <bool PACKED> struct UnitDz;
template <> struct UnitDz<false> {
    float d[8];
    __device__ __forceinline__ void terms(u4v_s (&t)[3]) const { split_terms(d, t); }
    __device__ __forceinline__ void add_to(float (&s)[8]) const
    {
#pragma unroll
        for (int q = 0; q < 8; ++q) s[q] += d[q];
    }
};
template <> struct UnitDz<true> {
    u4v_s p;
    __device__ __forceinline__ void add_to(float (&s)[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { s[2 * i] += f_from_bits(p[i] << 16); s[2 * i + 1] += f_from_bits(p[i] & 0xffff0000u); }
    }
};

// Bound by reading dZ_1 once where the board is small (Catch 10 x 5, 256 columns, 81920 samples, 84 MB: 23.8 us, 24.2 as a
// kernel that shared the board operand through LDS), by the vector work of the board operand and the three terms where it
// has many tiles.  Before, boards of 64 cells or more were a dense product over all features, walls and goal included,
// or a scatter in LDS.  Maze 9 x 13, 128 columns, 23920 samples: 41.3 -> 13.5 us; 16 x 16, 512 columns, 276480 samples
// (566 MB): 3088 -> 224 us; Catch 16 x 12, 512 columns, 327680 samples: 1007 -> 225 us; Catch 12 x 7, 256 columns, 65536
// samples: 76.3 -> 23.6 us; Catch 10 x 5, 512 columns, 30000 samples (a batch that is no multiple of 64): 36.6 -> 18.2 us;
// bf16, Catch 12 x 12, 256 columns, 163840 samples: 93.5 -> 38 us; maze 8 x 8: 83.4 -> 25 us.
//
// A wavefront owns 32 columns and walks its chunk in units of 16 samples, one step of v_mfma_f32_32x32x16_bf16; lane
// (l32, kg) is cell l32 of a tile in the board operand and column l32 of dZ_1 in the other, samples 8 kg + 0..7 of the
// unit in both.  Wavefronts share nothing: no LDS, no barriers; a workgroup's column tiles stand side by side, so a unit's
// rows are read in whole lines.  Maze: units are 16 environments at one time step, walked through time; half of the
// wavefronts take the agent's plane, the others read the same rows (from the cache), add them up over time and multiply by
// the walls once per 16 environments.
template <int ENV, int NT, bool PACKED>
__global__ __launch_bounds__(ENV == ENV_MAZE ? 512 : 256, 2) void first_layer_onehot(const FirstOneHotArgs a)
{
    constexpr int DEPTH = PACKED ? 4 : 3;                        // units in flight per wavefront (4 and 5: no faster)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, kg = lane >> 5;
    const int N = a.N;
    const bool walls_role = ENV == ENV_MAZE && wave >= a.tiles_wg;
    const int j = (blockIdx.y * a.tiles_wg + (walls_role ? wave - a.tiles_wg : wave)) * 32 + l32;
    const int split = blockIdx.x;
    const int u0 = split * a.per, u1 = u0 + a.per < a.units ? u0 + a.per : a.units;
    // first sample of a unit: Catch 16 u; maze 16 (u / T) + B (u mod T)
    struct Pos { int g, t; };
    auto start = [&](int u) { Pos p; if (ENV == ENV_MAZE) { p.g = u / a.T; p.t = u - p.g * a.T; } else { p.g = u; p.t = 0; } return p; };
    auto advance = [&](Pos& p) { if (ENV == ENV_MAZE) { if (++p.t == a.T) { p.t = 0; ++p.g; } } else ++p.g; };
    auto sample = [&](const Pos& p) { return ENV == ENV_MAZE ? 16 * p.g + a.B * p.t : 16 * p.g; };
    uint32_t off[PACKED ? 1 : 8];
    if (PACKED) off[0] = (uint32_t)kg * (uint32_t)N + (uint32_t)j;
    else {
#pragma unroll
        for (int q = 0; q < (PACKED ? 1 : 8); ++q) off[q] = (uint32_t)(8 * kg + q) * (uint32_t)N + (uint32_t)j;
    }
    auto load = [&](UnitDz<PACKED>& z, int m) {
        if constexpr (PACKED) z.p = (reinterpret_cast<const u4v_s*>(a.dy) + (size_t)(m >> 3) * N)[off[0]];
        else {
            const float* base = reinterpret_cast<const float*>(a.dy) + (size_t)m * N;
#pragma unroll
            for (int q = 0; q < 8; ++q) z.d[q] = base[off[q]];
        }
    };
    auto load_states = [&](u4v_s (&s)[2], int m) {
        const u4v_s* p = reinterpret_cast<const u4v_s*>(a.s0 + m + 8 * kg);
        s[0] = p[0]; s[1] = p[1];
    };
    f16v_s acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
    float sums[8];                                               // Catch: column sums.  Walls: the time sum of 16 environments
#pragma unroll
    for (int q = 0; q < 8; ++q) sums[q] = 0.0f;
    float bias = 0.0f;
    const uint32_t idx2 = (uint32_t)l32 * 0x10001u;
    uint32_t ones = 0x10001u;
    asm("" : "+v"(ones));
    const int pad_tile = a.paddle_row0 >> 5;
    auto eight = [](const float (&s)[8]) { return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])); };
    auto store_plane = [&](float* out) {
        const uint32_t o = (uint32_t)(4 * kg) * (uint32_t)N + (uint32_t)j;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 32 * i + 8 * (r >> 2) + (r & 3);  // this lane's cell is row + 4 kg
                if (32 * i + 32 <= a.cells || row + 4 * kg < a.cells) (out + (size_t)row * N)[o] = acc[i][r];
            }
    };
    // every load is unconditional (past the end it reads the last unit again and the result is dropped), so that the waits
    // before a unit's products never cover the loads behind it
    Pos pf = start(u0 < a.units ? u0 : a.units - 1);
    int uf = u0;
    auto next_fetch = [&]() { if (uf + 1 < u1) { ++uf; advance(pf); } };
    if (walls_role) {
        if constexpr (ENV == ENV_MAZE) {
            UnitDz<PACKED> z[DEPTH];
#pragma unroll
            for (int k = 0; k < DEPTH; ++k) { load(z[k], sample(pf)); next_fetch(); }
            Pos pos = start(u0);
            for (int u = u0; u < u1; u += DEPTH) {
#pragma unroll
                for (int k = 0; k < DEPTH; ++k) {
                    if (u + k < u1) {
                        z[k].add_to(sums);
                        if (pos.t == a.T - 1 || u + k == u1 - 1) {          // the last time step of these environments here
                            bias += eight(sums);
                            u4v_s t[3];
                            split_terms(sums, t);
#pragma unroll
                            for (int q = 0; q < 8; ++q) sums[q] = 0.0f;
                            const uint32_t* wp = a.walls + 16 * pos.g + 8 * kg;
#pragma unroll
                            for (int i = 0; i < NT; ++i) {
                                const u4v_s* w4 = reinterpret_cast<const u4v_s*>(wp + (size_t)i * a.B);
                                const u4v_s wa = w4[0], wb = w4[1];
                                const uint32_t w[8] = {wa[0], wa[1], wa[2], wa[3], wb[0], wb[1], wb[2], wb[3]};
                                u4v_s x;
#pragma unroll
                                for (int e = 0; e < 4; ++e) x[e] = (((w[2 * e] >> l32) & 1u) | (((w[2 * e + 1] >> l32) & 1u) << 16)) * 0x3f80u;
                                acc[i] = mfma_f(x, t[2], acc[i]);            // smallest terms first
                                acc[i] = mfma_f(x, t[1], acc[i]);
                                acc[i] = mfma_f(x, t[0], acc[i]);
                            }
                        }
                        advance(pos);
                    }
                    load(z[k], sample(pf)); next_fetch();
                }
            }
            store_plane(a.walls_out + (size_t)split * a.cells * N);
            bias += __shfl_xor(bias, 32);
            if (kg == 0) a.sums_out[(size_t)split * N + j] = bias;
        }
        return;
    }
    UnitDz<PACKED> z[DEPTH];
    u4v_s st[DEPTH][2];
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) { const int m = sample(pf); load(z[k], m); load_states(st[k], m); next_fetch(); }
    for (int u = u0; u < u1; u += DEPTH) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            if (u + k < u1) {
                if (ENV == ENV_CATCH) z[k].add_to(sums);
                u4v_s t[3];
                if constexpr (PACKED) t[0] = z[k].p; else z[k].terms(t);
                const uint32_t s[8] = {st[k][0][0], st[k][0][1], st[k][0][2], st[k][0][3], st[k][1][0], st[k][1][1], st[k][1][2], st[k][1][3]};
                uint32_t c1[4], c2[4];                           // cells of two samples each, less this lane's
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t x = s[2 * e], y = s[2 * e + 1];
                    if (ENV == ENV_CATCH) {
                        const uint32_t col = (x & 0xffu) | ((y & 0xffu) << 16), row = ((x >> 8) & 0xffu) | (((y >> 8) & 0xffu) << 16);
                        const uint32_t pad = ((x >> 16) & 0xffu) | (y & 0xff0000u);
                        const us2_f w = {(uint16_t)a.cols, (uint16_t)a.cols}, b = {(uint16_t)a.paddle_row0, (uint16_t)a.paddle_row0};
                        c1[e] = __builtin_bit_cast(uint32_t, (us2_f)(__builtin_bit_cast(us2_f, row) * w + __builtin_bit_cast(us2_f, col))) ^ idx2;
                        c2[e] = __builtin_bit_cast(uint32_t, (us2_f)(__builtin_bit_cast(us2_f, pad) + b)) ^ idx2;
                    } else {
                        c1[e] = ((x & 0xffffu) | (y << 16)) ^ idx2;
                        c2[e] = 0xffffffffu;
                    }
                }
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    u4v_s x;
                    if (ENV == ENV_CATCH && i >= pad_tile) {     // tiles with cells of the bottom row
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = one_where_zero(min_pair(c1[e] ^ (0x200020u * (uint32_t)i), c2[e] ^ (0x200020u * (uint32_t)i)), ones);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = one_where_zero(c1[e] ^ (0x200020u * (uint32_t)i), ones);
                    }
                    if constexpr (!PACKED) {
                        acc[i] = mfma_f(x, t[2], acc[i]);        // smallest terms first
                        acc[i] = mfma_f(x, t[1], acc[i]);
                    }
                    acc[i] = mfma_f(x, t[0], acc[i]);
                }
            }
            const int m = sample(pf);
            load(z[k], m); load_states(st[k], m); next_fetch();
        }
    }
    if (ENV == ENV_CATCH) {
        float* out = a.out + (size_t)split * ((size_t)a.cells * N + N);
        store_plane(out);
        bias = eight(sums);
        bias += __shfl_xor(bias, 32);
        if (kg == 0) out[(size_t)a.cells * N + j] = bias;
    } else store_plane(a.out + (size_t)split * a.cells * N);
}

template <int NT>
static void launch_tiles(int nt, bool maze, bool packed, const FirstOneHotArgs& a, dim3 grid, dim3 block, hipStream_t s)
{
    if constexpr (NT > 1) if (nt < NT) return launch_tiles<NT - 1>(nt, maze, packed, a, grid, block, s);
    auto kern = maze ? (packed ? first_layer_onehot<ENV_MAZE, NT, true> : first_layer_onehot<ENV_MAZE, NT, false>)
                     : (packed ? first_layer_onehot<ENV_CATCH, NT, true> : first_layer_onehot<ENV_CATCH, NT, false>);
    hipLaunchKernelGGL(kern, grid, block, 0, s, a);
}

hipError_t launch_first_layer_onehot(anakin* h, bool packed)
{
    const Layout& L = h->lay;
    const NetShape& n = h->net;
    const int M = h->B * h->T;
    FirstOneHotArgs a;
    a.B = h->B; a.T = h->T; a.N = n.dims[1]; a.cells = h->env.rows * h->env.cols;
    a.units = M / 16; a.per = chunk_rows(M, h->splits[0], h->quanta[0]) / 16;
    const int tiles = a.N / 32;
    a.tiles_wg = tiles < 4 ? tiles : 4;
    a.cols = h->env.cols; a.paddle_row0 = (h->env.rows - 1) * h->env.cols;
    // packed dZ_1 follows the row-major copy
    a.dy = packed ? static_cast<const void*>(at<const uint16_t>(h, L.dz[0]) + (size_t)M * a.N) : static_cast<const void*>(at<const float>(h, L.dz[0]));
    a.s0 = at<const uint32_t>(h, L.tr_s0); a.walls = at<const uint32_t>(h, L.walls);
    const size_t plane = (size_t)a.cells * a.N;
    const bool maze = h->env.kind == ENV_MAZE;
    a.walls_out = at<float>(h, L.part[0]);                       // the pieces of launch_adam's regions
    a.out = maze ? a.walls_out + plane * h->splits[0] : a.walls_out;
    a.sums_out = a.out + plane * h->splits[0];
    const dim3 grid(h->splits[0], tiles / a.tiles_wg), block(a.tiles_wg * 64 * (maze ? 2 : 1));
    ProfScope prof(h, "first_layer_grad");
    launch_tiles<8>((a.cells + 31) / 32, maze, packed, a, grid, block, h->stream);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The pendulum in bf16: dW_1[c][j] = sum_m o_c(m) dZ_1[m][j] for o = (cos th, sin th, thd) rounded to bfloat16, and a
// fourth feature that is always 1, which gives the bias gradient.  A workgroup takes 128 columns and 256 samples at a
// time: a thread computes the features of one sample, which reach the matrix operand through LDS, while the block's 16
// packed pieces of dZ_1 per lane are on their way; wavefront w owns columns 32 w .. 32 w + 31.  Of the operand's 32 rows
// four mean something; the others repeat them and their sums are dropped.  Bound by reading dZ_1 (512 columns, 414720
// samples, 425 MB: 84 us, 5.1 TB/s; 675 as a dense product that computed a sample's sine and cosine once per feature and
// row of tiles.  256 columns, 163840 samples: 127.7 -> 17.0 us; 128 columns, 20480 samples: 18.7 -> 6.3 us).
// ---------------------------------------------------------------------------
struct FirstPendulumArgs {
    int N, M, rows;
    const uint16_t* dy;       // packed [M/8][N][8]
    const float* f0; const float* f1;
    float* out;               // [splits][3*N + N]
};
constexpr int FP_BLOCK = 256, FP_UNITS = FP_BLOCK / 16;

__global__ __launch_bounds__(FP_BLOCK) void first_layer_pendulum_bf16(const FirstPendulumArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t feat[2][4][FP_BLOCK];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, kg = lane >> 5;
    const int N = a.N, j = blockIdx.y * 128 + wave * 32 + l32, split = blockIdx.x;
    const int m_begin = split * a.rows, m_end = m_begin + a.rows < a.M ? m_begin + a.rows : a.M;
    const uint32_t off = (uint32_t)kg * (uint32_t)N + (uint32_t)j;
    f16v_s acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    feat[0][3][tid] = 0x3f80; feat[1][3][tid] = 0x3f80;
    int buf = 0;
    for (int m0 = m_begin; m0 < m_end; m0 += FP_BLOCK, buf ^= 1) {
        const int units = m_end - m0 < FP_BLOCK ? (m_end - m0) >> 4 : FP_UNITS;
        u4v_s p[FP_UNITS];
#pragma unroll
        for (int u = 0; u < FP_UNITS; ++u) {
            const int m = m0 + 16 * (u < units ? u : units - 1);  // past the end: the last piece again
            p[u] = (reinterpret_cast<const u4v_s*>(a.dy) + (size_t)(m >> 3) * N)[off];
        }
        const int ms = m0 + tid < m_end ? m0 + tid : m_end - 1;
        float sn, cs;
        det_sincos(a.f0[ms], sn, cs);
        feat[buf][0][tid] = bf16_bits(cs); feat[buf][1][tid] = bf16_bits(sn); feat[buf][2][tid] = bf16_bits(a.f1[ms]);
        __syncthreads();                                         // also: everybody is done with the other buffer
#pragma unroll
        for (int u = 0; u < FP_UNITS; ++u) {
            const u4v_s x = *reinterpret_cast<const u4v_s*>(&feat[buf][l32 & 3][16 * u + 8 * kg]);
            if (u < units) acc = mfma_f(x, p[u], acc);
        }
    }
    if (kg != 0) return;                                         // rows 0..3 of the sums
    float* out = a.out + (size_t)split * 4 * N + j;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(size_t)r * N] = acc[r];
}

hipError_t launch_first_layer_pendulum_bf16(anakin* h)
{
    const Layout& L = h->lay;
    FirstPendulumArgs a;
    a.N = h->net.dims[1]; a.M = h->B * h->T; a.rows = chunk_rows(a.M, h->splits[0], h->quanta[0]);
    a.dy = at<const uint16_t>(h, L.dz[0]) + (size_t)a.M * a.N;
    a.f0 = at<const float>(h, L.tr_f0); a.f1 = at<const float>(h, L.tr_f1);
    a.out = at<float>(h, L.part[0]);
    ProfScope prof(h, "first_layer_grad");
    hipLaunchKernelGGL(first_layer_pendulum_bf16, dim3(h->splits[0], a.N / 128), dim3(FP_BLOCK), 0, h->stream, a);
    return hipGetLastError();
}

}  // namespace ank
