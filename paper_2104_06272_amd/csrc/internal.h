// Host-side handle, device workspace layout and kernel argument blocks shared by
// the translation units of libanakin.  Nothing here is part of the public ABI.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <string>
#include <vector>
#include <hip/hip_runtime.h>
#include "env.h"
#include "../../include/anakin.h"

namespace ank {

constexpr int MAX_LAYERS = 4;
constexpr int MAX_REGIONS = MAX_LAYERS + 1;      // one (W,b) pair per hidden layer + the heads
constexpr int MAX_ADAM_REGIONS = MAX_REGIONS + 4; // the maze first layer of a bf16 net is reduced in five pieces
constexpr int WG = 256;                          // threads per workgroup everywhere

// network shape and parameter offsets (elements into theta)
struct NetShape {
    int D, A, NH, NHP, L;
    int dims[MAX_LAYERS + 2];                    // D, H1..HL
    int w_off[MAX_LAYERS], b_off[MAX_LAYERS], wh_off, bh_off;
    int P;
    int policy, bf16;
    int split;                                   // fp32, or bf16 off the bf16 matrix path: the dense products of wide layers run on split operands
};

// trajectory and env-state pointers (device)
struct TrajPtrs {
    uint32_t* s0; float* f0; float* f1; const uint32_t* walls;        // current env state; walls [8][B]
    uint32_t* tr_s0; float* tr_f0; float* tr_f1;                       // [T+1][B] state observed at t
    uint8_t* tr_act; float* tr_eps; float* tr_actf;                    // [T][B]
    float* tr_rew; uint8_t* tr_done;                                   // [T][B]
    float* tr_val;                                                     // [T+1][B]
    float* tr_head;                                                    // [T+1][B][NHP]
    float* act[MAX_LAYERS];                                            // [T*B][H_l] hidden activations
    uint32_t* mask[MAX_LAYERS];                                        // bf16 matrix-core path: which of them are positive, see relu_mask_index
};

// ReLU masks of the bf16 matrix-core path, written by the acting kernels beside the packed activations and read by
// the dX products of the update in place of the activations themselves (1/8 of the bytes).  One 32-bit word per
// (stage of 32 consecutive samples, half kg of the accumulator rows, column): [M/32][2][H].  Lane (column, kg) of a
// 32 x 32 MFMA accumulator tile holds rows 8g + 4kg + q (g, q = 0..3) as value r = 4g + q; bit relu_mask_bit(r) of
// its word says that this activation is positive.  (Values come in packed pairs; pair r/2 puts the flag of its low
// half in bit r/2 and of its high half in bit 16 + r/2, which costs the producer two instructions per pair.)
ANK_HD size_t relu_mask_index(size_t stage, int kg, int H, int col) { return (stage * 2 + (size_t)kg) * (size_t)H + (size_t)col; }
ANK_HD int relu_mask_bit(int r) { return (r >> 1) + 16 * (r & 1); }

struct RolloutArgs {
    EnvDims env;
    NetShape net;
    TrajPtrs tp;
    const float* theta;
    int B, T, ldx;
    int keep_acts;               // store hidden activations for the update (0: the update rebuilds them)
    int bootstrap;               // REPLAY: the state after the last step is evaluated too
    int maze_prefix;             // maze: the wall plane's share of the first layer is summed once per launch, in LDS
    uint64_t seed, gstep;
};

// position of parameter i in the copy that stores every weight matrix transposed
// (layers [N][K], heads [NH][HL]); biases keep their place
// Layout of the second bf16 copy of the parameters, the one the acting kernel feeds to
// v_mfma_f32_32x32x16_bf16 as the B operand.  A weight matrix W[K][N] with K % 16 == 0 and
// N % 32 == 0 is stored in operand tiles: for every block of 32 output columns and every
// step of 16 inputs, the 64 lanes' 16-byte pieces are adjacent (lane = 32*((k%16)/8) + n%32
// holds k%8 = 0..7), so one wavefront load is one contiguous KiB.  Other layer matrices are
// stored transposed ([N][K]); the head matrix as [NH][HL].
ANK_HD bool mfma_tiled(int K, int N) { return K % 16 == 0 && N % 32 == 0; }
ANK_HD int tiled_offset(int K, int k, int n)
{
    return (((n >> 5) * (K >> 4) + (k >> 4)) << 9) + (((((k & 15) >> 3) << 5) + (n & 31)) << 3) + (k & 7);
}
ANK_HD int transposed_index(const NetShape& n, int i)
{
    for (int l = 0; l < n.L; ++l) {
        const int K = n.dims[l], N = n.dims[l + 1], off = i - n.w_off[l];
        if (off >= 0 && off < K * N)
            return n.w_off[l] + (mfma_tiled(K, N) ? tiled_offset(K, off / N, off % N) : (off % N) * K + off / N);
    }
    const int off = i - n.wh_off, HL = n.dims[n.L];
    if (off >= 0 && off < HL * n.NH) return n.wh_off + (off % n.NH) * HL + off / n.NH;
    return i;
}

// Workgroup L of a 1-D grid runs on XCD L % 8 (round-robin dispatch) and each XCD has its own L2.
// Map L to (outer, inner) so that the n_inner workgroups sharing one `outer` (the same operand
// tile) run back to back on one XCD and the second reader hits in that L2.
__device__ __forceinline__ void xcd_map(int L, int n_outer, int n_inner, int& outer, int& inner)
{
    const int whole = (n_outer >> 3) << 3, full = whole * n_inner;
    if (L < full) { const int q = L >> 3; inner = q % n_inner; outer = (q / n_inner) * 8 + (L & 7); }
    else { const int r = L - full; outer = whole + r / n_inner; inner = r % n_inner; }
}

// Rows of a reduction over M samples that each of `splits` chunks takes: whole multiples of `quantum`, the last chunk
// whatever is left.  Every chunk count that pick_splits returns is reached exactly (no chunk is empty).
inline int chunk_rows(int M, int splits, int quantum)
{
    const int tiles = (M + quantum - 1) / quantum;
    return (tiles + splits - 1) / splits * quantum;
}

// state snapshots the first layer's input is rebuilt from (row m = t*B + b of the trajectory)
struct ObsLite { EnvDims env; const uint32_t* s0; const float* f0; const float* f1; };

// split-K partial sums of one parameter region (W_l followed by b_l, or Wh followed by bh)
struct Region { int start, count, splits; const float* partial; };

struct AdamArgs {
    Region reg[MAX_ADAM_REGIONS];
    int n_regions, P;
    float* theta; float* grad; float* m; float* v;
    uint16_t* w_bf16;            // bf16 copy of theta (same indexing), or null
    uint16_t* wt_bf16;           // bf16 copy with every weight matrix transposed, or null
    NetShape net;
    float lr, beta1, beta2, eps, bc1, bc2;
};

// Acting with the hidden matrices in the register file (rollout_pinned.hip).  A block is 128 inputs x 16 outputs of one
// layer, 32 registers of one wavefront; the blocks of 16 outputs follow one another in one wavefront.  Two words per block:
struct PinnedPlan {
    static constexpr int WAVES = 4, MAX_BLOCKS = 6;                                // wavefronts that compute the hidden layers
    enum : uint32_t { VALID = 1u, START = 2u, END = 4u, HALF = 8u, PAIR = 16u };   // first / last block of its outputs; 64 inputs only; with the next block, whose outputs are the next 16
    static constexpr int LAYER = 5, LGK = 7, LGN = 11, TILE = 15, KBLOCK = 20;     // bits: layer (2), log2 of its inputs (4), of its outputs (4), output / 16 (5), input / 128 (2)
    static constexpr int XOFF = 0, YOFF = 16;                                      // second word: LDS place of the layer's inputs and of these outputs, in 16 bytes (16 each)
    int NB;                               // blocks per wavefront (0: not applicable)
    uint32_t block[WAVES][MAX_BLOCKS][2];
};

struct Layout {
    size_t theta, grad, m, v, w_bf16, wt_bf16;
    size_t theta0, w0_bf16;      // copies of theta / w_bf16 taken before the first of several updates on one unroll
    size_t w_src, w16_src;       // where the backward kernels read weights: theta / w_bf16, or the copies
    size_t s0, f0, f1, walls;
    size_t tr_s0, tr_f0, tr_f1, tr_act, tr_eps, tr_actf, tr_rew, tr_done, tr_val, tr_head;
    size_t adv, ret, dhead;
    size_t act[MAX_LAYERS], dz[MAX_LAYERS];
    size_t mask[MAX_LAYERS];      // bf16 matrix-core path: ReLU masks, inside the unused upper half of act[l]
    size_t part[MAX_REGIONS];
    size_t w3[MAX_LAYERS];       // fp32 nets: weights of layer l as split operands of the dX product (split_weights)
    size_t head_stage;           // first-stage partials of the head gradient
    size_t time_sum;             // maze first layer of a bf16 net: dZ_1 summed over time, two bfloat16 terms, [2][B][H1]
    size_t loss_part;
    // decoupled acting and learning: the behaviour copy of the parameters the actor runs on, the second set of
    // trajectory records (the actor fills one set while the learner reads the other), and the learner's own
    // forward results on the stored unroll
    size_t theta_b, w_bf16_b, wt_bf16_b;                // bf16 nets: the actor's own rounded copies
    size_t alt_tr_s0, alt_tr_f0, alt_tr_f1, alt_tr_act, alt_tr_eps, alt_tr_actf, alt_tr_rew, alt_tr_done, alt_tr_val, alt_tr_head;
    size_t head_new, val_new, eps_new;
    size_t head_old;              // set while the loss is taken at a repeated forward pass: head outputs at acting time (0: none)
    size_t small_part;           // single-launch update of small nets: one whole gradient per workgroup, [workgroups][P]
    size_t counters;             // arrival counters of kernels whose last workgroup finishes the job (zero between launches)
    size_t path;                 // pathwise policy gradient: dL_path / d(mu, log_sigma) per sample, [T*B][2]
    size_t total;
};

}  // namespace ank

struct anakin {
    anakin_env_cfg env_cfg;
    anakin_net_cfg net_cfg;
    ank::EnvDims env;
    ank::NetShape net;
    int B, T;
    uint64_t seed, gstep;
    int adam_t;
    int have_traj;
    int mode;
    char* ws;
    size_t ws_bytes;
    char* scratch;                // base of tagged offsets (see SCRATCH_TAG); null outside anakin_learn_static
    int device;                   // the device the workspace lives on
    hipStream_t stream;
    ank::Layout lay;
    int TM;                       // envs per workgroup in the vector-ALU rollout kernel
    int TM_mfma;                  // envs per workgroup in the matrix-core rollout kernel (0: not applicable)
    int TM_res;                   // envs per workgroup in the weights-resident rollout kernel (0: not applicable)
    int wide;                    // groups of four environments per workgroup of the acting kernel of wide nets (0: not applicable)
    ank::PinnedPlan pinned;      // rollout kernel with hidden matrices of any widths in registers
    int splits[ank::MAX_REGIONS]; // split-K factor per parameter region
    int quanta[ank::MAX_REGIONS]; // rows of a region's chunks are multiples of this (chunk_rows)
    int loss_blocks;
    int metric_blocks;            // blocks of loss partials the last update wrote (0 before the first)
    int head_fan;                 // first-stage workgroups per split of the head-gradient pass
    int chunks_sequential;        // several updates per unroll: chunk k's gradient at the parameters after k updates (else at the acting ones)
    int n_updates;                // Adam updates per unroll (consecutive time chunks of the unroll), 1 by default
    int sub_splits[ank::MAX_REGIONS], sub_quanta[ank::MAX_REGIONS], sub_splits_w, sub_head_fan, sub_loss_blocks;   // split plan of one chunk
    int splits_w;                 // maze first layer of a bf16 net: split count of the wall-plane product (0: one product
                                  // over all observation rows); splits[0] is then the split count of the agent-plane product
    int bf16_path;                // the bf16 matrix-core kernels support this net
    int traj_packed;              // the stored unroll holds packed bf16 activations
    int traj_no_acts;             // the stored unroll holds no hidden activations (one-layer nets)
    int pathwise;                 // policy gradient through the environment instead of the score function (pendulum)
    int traj_decoupled;           // the stored unroll was collected by a decoupled step: behaviour parameters, no activations
    hipStream_t actor_stream;     // decoupled steps: the actor's stream (the caller's, or created on first use), and the fork/join events
    int actor_stream_owned;       // the library created actor_stream and destroys it
    hipEvent_t ev_fork, ev_join;
    std::string err;
    // optional per-kernel timing with events on the launch stream
    int prof_on;
    struct ProfPending { int name; hipEvent_t start, stop; };
    struct ProfTotal { std::string name; long long calls; double ms; };
    std::vector<ProfPending> prof_pending;
    std::vector<hipEvent_t> prof_pool;
    std::vector<ProfTotal> prof_totals;
};

namespace ank {

// An offset with this bit set is relative to the handle's update-scratch base instead of the workspace base
// (anakin_learn_static points the backward pass's scratch at the library's own static device array).
constexpr size_t SCRATCH_TAG = (size_t)1 << 62;
template <class T> inline T* at(const anakin* h, size_t off)
{
    return reinterpret_cast<T*>((off & SCRATCH_TAG) ? h->scratch + (off & ~SCRATCH_TAG) : h->ws + off);
}

// per-kernel timing: brackets one launch with two events when profiling is on
struct ProfScope {
    anakin* h; int idx;
    ProfScope(anakin* h_, const char* name);
    ~ProfScope();
};
hipError_t prof_resolve(anakin* h);

// kernel launchers (each enqueues on h->stream and returns the HIP status)
hipError_t launch_rollout(anakin* h);
hipError_t launch_rollout_behaviour(anakin* h);
hipError_t launch_replay_forward(anakin* h, bool bootstrap);
// time steps per workgroup of a replay: the steps do not depend on one another, so a batch that does not give every
// compute unit a tile is cut along time as well
inline int replay_segment(int tiles, int tend)
{
    int parts = 256 / tiles;
    if (parts < 1) parts = 1;
    if (parts > tend) parts = tend;
    return (tend + parts - 1) / parts;
}
hipError_t launch_pathwise(anakin* h);
bool pathwise_ok(const anakin* h);
hipError_t launch_returns(anakin* h);
bool scan_loss_ok(const anakin* h);          // returns and loss as one launch
hipError_t launch_scan_loss(anakin* h, bool vtrace);
hipError_t launch_vtrace_loss(anakin* h);
hipError_t launch_head_grad(anakin* h);
hipError_t launch_backward(anakin* h);
hipError_t launch_adam(anakin* h);
hipError_t launch_first_layer_grad(anakin* h);
hipError_t launch_adam_probe(float* base, int P, hipStream_t s);
hipError_t launch_learn_one_layer(anakin* h);
hipError_t launch_learn_catch_fused(anakin* h);
hipError_t launch_learn_small_fused(anakin* h);
bool small_fused_ok(const anakin* h);
size_t small_fused_part_bytes(const EnvDims& ed, const NetShape& ns, int B, int T);
bool catch_fused_ok(const anakin* h);
// single hidden layer on a one-hot or 3-feature observation: the update rebuilds the layer from the state
inline bool one_layer_shape(const NetShape& n, const EnvDims& ed) { return n.L == 1 && ed.kind != ENV_MAZE && !n.bf16 && n.dims[1] <= 128 && (size_t)128 * n.dims[0] * 4 + (size_t)n.dims[0] * n.dims[1] * 4 <= 64 * 1024; }
inline bool one_layer_fused(const anakin* h) { return one_layer_shape(h->net, h->env) && !(h->mode & ANAKIN_MODE_VALU_GEMM); }
// One-hidden-layer nets whose whole backward pass is one launch (learn_one.hip): those, and 256 units, which keep their
// activations in memory for the caller but are rebuilt all the same (Catch with the board in two tiles, 64 cells).  256
// units, before (head pass, first layer, their sums) and now: 524288 samples, Catch 10 x 5 360 us and 152, the pendulum 365 and
// 61; 1024 samples 11.3 and 8.6, 10.5 and 5.8; 8 x 8, whole steps, 64 samples 31.6 and 30.1, 16384 64.4 and 58.9, 524288 506 and 275.
inline bool one_layer_learn_shape(const NetShape& n, const EnvDims& ed) { return one_layer_shape(n, ed) || (n.L == 1 && !n.bf16 && n.dims[1] == 256 && (ed.kind == ENV_PENDULUM || (ed.kind == ENV_CATCH && n.dims[0] <= 64))); }
inline bool one_layer_learn(const anakin* h) { return one_layer_learn_shape(h->net, h->env) && !(h->mode & ANAKIN_MODE_VALU_GEMM); }
// Catch, 32 units: the launch that takes returns and loss too (learn_catch_fused) is a chain of T steps for each 256
// environments (54 us at T = 16), whatever their number up to two blocks of 256 a compute unit.  Three launches (learn_one_catch
// between loss and optimiser) grow with environments times steps, so the line between them falls with shorter unrolls
// (whole steps, three launches and one: T = 64, 49152 environments 261 and 286 us; T = 16, 49152 80.6 and 86.2, 65536 environments,
// update alone, 74.3 and 64.8; T = 8, 40960 49.1 and 52.7, 49152 53.4 and 53.2; T = 4, 32768 34.1 and 34.5, 34560 35.6 and 34.6,
// 49152 39.3 and 35.8; T = 2, 19200 26.5 and 27.3, 24576 28.1 and 26.0; T = 1, 16384 21.7 and 22.9, 19200 23.9 and 23.4,
// 24576 25.1 and 21.8).
inline int catch_fused_blocks(int T) { return T <= 2 ? 64 + 8 * T : T >= 16 ? 208 : 234 - 416 / T; }
inline bool catch_fused_shape(const NetShape& n, const EnvDims& ed, int B, int T) { return one_layer_shape(n, ed) && ed.kind == ENV_CATCH && n.dims[1] == 32 && B % 256 == 0 && B / 256 >= catch_fused_blocks(T); }
// its workgroups, whole blocks of 256 environments each (0: another launch)
inline int catch_fused_groups(const NetShape& n, const EnvDims& ed, int B, int T)
{
    if (!catch_fused_shape(n, ed, B, T)) return 0;
    int s = B / 256;
    while (s > 512 && s % 2 == 0) s /= 2;
    return s <= 1024 ? s : 0;
}
hipError_t launch_partial_reduce(const float* src, float* dst, int count, int fan, int splits, hipStream_t s);
hipError_t launch_rollout_bf16(anakin* h);
hipError_t launch_rollout_bf16_behaviour(anakin* h);
hipError_t launch_replay_bf16(anakin* h, bool bootstrap);
hipError_t launch_backward_bf16(anakin* h);
hipError_t launch_refresh_bf16(anakin* h);
int bf16_dw_chunks(int M, int K, int N, bool top);
int bf16_dx_ranges(int M, int K, int N, int splits);
bool bf16_top_fused(const NetShape& n, int M);
bool bf16_top_fold(const NetShape& n);
bool bf16_first_fold(const NetShape& n, const EnvDims& ed, int M);
bool bf16_dx_resident(const NetShape& n, int M, int l);
bool rollout_bf16_ok(const NetShape& net, const EnvDims& env, int B);
// the stored unroll was produced by the bf16 matrix-core kernels and the maze's first layer is two dense products, agent and walls
inline bool first_layer_split(const anakin* h) { return h->splits_w > 0 && h->traj_packed; }
// boards whose first-layer gradient comes from the one-hot kernel (first_layer.hip), in whichever form dZ_1 has
inline bool first_onehot_shape(const EnvDims& ed) { return ed.kind != ENV_PENDULUM && ed.rows * ed.cols <= 256; }
inline bool first_onehot(const anakin* h) { return first_onehot_shape(h->env) && !(h->mode & ANAKIN_MODE_VALU_GEMM) && !first_layer_split(h); }
hipError_t launch_first_layer_onehot(anakin* h, bool packed);
hipError_t launch_first_layer_pendulum_bf16(anakin* h);
// bf16 network running on the bf16 matrix path (packed bf16 activations) rather than on the fp32 kernels with rounded operands
inline bool bf16_mfma(const anakin* h) { return h->bf16_path && !(h->mode & (ANAKIN_MODE_CANONICAL_ACTING | ANAKIN_MODE_VALU_GEMM)); }
// both sides of layer l + 1 (l >= 1) are whole 64-wide tiles: its two products share a launch (gemm_split.hip)
inline bool split_gemm_shape(const NetShape& n, int l) { return n.split && l >= 1 && l < n.L && n.dims[l] % 64 == 0 && n.dims[l + 1] % 64 == 0; }
// tiles of the dW product: 256 x 256 where both sides allow it, else 128 or 64 on a side (128 x 256 as one tile spilled
// registers: 54 us for both products of a 128-256 net over 28 k samples, 35 as two tiles)
// n.split == 2 (few samples): tiles of 128 or 64 for dW and of 128 samples x 64 columns for dX, as long as the dX product
// has at most one of them per compute unit, samples x inputs <= 2^21.  The larger tiles need fewer passes over the operands
// but leave most units idle there: 256-256, 2048 samples 26.0 us with them, 16.5 with the small ones, 8192 samples 27.7
// and 25.7, 16384 34.0 and 39.1; 512-512, 512 samples 38.8 and 22.4, 4096 41.8 and 39.5, 8192 53.5 and 68.4; 256-256-256
// (two launches), 2048 samples 46.0 and 26.0.  Fewer inputs than 256: up to 8192 samples (64-64 12.9 and 11.0, 64-512 32.0
// and 23.5), 4096 where the larger tiles are no more than 128 x 128 (4096 samples 15.5 and 14.2, 8192 15.5 and 16.3).
inline bool split_tile_256(const NetShape& n, int l) { return n.split == 1 && n.dims[l] % 256 == 0 && n.dims[l + 1] % 256 == 0; }
inline int split_tile_i(const NetShape& n, int l) { return split_tile_256(n, l) ? 256 : n.dims[l] % 128 ? 64 : 128; }
inline int split_tile_j(const NetShape& n, int l) { return split_tile_256(n, l) ? 256 : n.dims[l + 1] % 128 ? 64 : 128; }
// the dX product: output columns and samples per tile (eight wavefronts, 32 columns each, or shared out over the samples)
inline int split_nt_cols(const NetShape& n, int l) { return n.split == 2 ? 64 : n.dims[l] % 256 == 0 ? 256 : split_tile_i(n, l); }
inline int split_nt_rows(const NetShape& n, int l) { return n.split == 1 && split_nt_cols(n, l) == 64 ? 256 : 128; }
// Compute units the dW and the dX product of such a layer get in their shared launch (their costs per sample are alike):
// chunks of the dW product per tile, and workgroups of the dX product along the samples per tile of output columns.
inline int split_tn_cap(const NetShape& n, int l) { const int c = 128 / ((n.dims[l] / split_tile_i(n, l)) * (n.dims[l + 1] / split_tile_j(n, l))); return c > 1 ? c : 1; }
inline int split_nt_blocks(const NetShape& n, int M, int l)
{
    const int c = 128 / (n.dims[l] / split_nt_cols(n, l)), cap = c > 1 ? c : 1;
    const int tiles = (M + split_nt_rows(n, l) - 1) / split_nt_rows(n, l), per = (tiles + cap - 1) / cap;
    return (tiles + per - 1) / per;
}
// the head pass folded into the top layer's products (a pass of its own for the maze's five heads: 128-64, 23920 samples
// 11.2 + 14.9 us against 18.4 with it folded in; whole steps of mazes of 64 to 512 units 5 to 16 % slower)
inline bool heads_fused_shape(const NetShape& n) { return n.NH <= 5 && split_gemm_shape(n, n.L - 1); }
// the first-layer gradient of the pendulum and of Catch boards of up to 64 cells rides in the epilogue of the dX product that
// forms dZ_1; returns the number of partials that kernel writes (its workgroups along the samples), else 0.  The pass of its own
// that it replaces reads dZ_1 once more: 20 % of the products' time at 256-256, more in narrower nets (67 nets and batches, whole
// steps, 1.00 to 1.32 times as fast).  128 cells would take 64 accumulators more of wavefronts that have 256 registers: 12 to 52
// bytes a lane in scratch in all but the 128-wide tiles, and twice the MFMAs; larger boards keep that pass.
inline int first_fused_splits(const NetShape& n, const EnvDims& ed, int M)
{
    const bool fits = ed.kind == ENV_PENDULUM || (ed.kind == ENV_CATCH && ed.rows * ed.cols <= 64);
    return fits && split_gemm_shape(n, 1) ? split_nt_blocks(n, M, 1) : 0;
}
int rollout_pick_tile(const NetShape& net, int B);
int rollout_pick_tile_mfma(const NetShape& net, const EnvDims& env, int B);
bool rollout_one_ok(const anakin* h);
hipError_t launch_rollout_one(anakin* h, const RolloutArgs& args, bool replay);
void rollout_pinned_plan(const NetShape& net, const EnvDims& env, int B, PinnedPlan& p);
hipError_t launch_pinned(anakin* h, const RolloutArgs& args);
int rollout_resident_width(const NetShape& net);
bool replay_resident_ok(const anakin* h, int samples);
hipError_t launch_replay_resident(anakin* h, const RolloutArgs& a, int samples);
bool vtrace_off_the_actor(const anakin* h, size_t lds);
bool rollout_small_ok(const anakin* h);
hipError_t launch_small(anakin* h, const RolloutArgs& args);
int rollout_wide_groups(const NetShape& net, const EnvDims& env, int B);
bool wide_before_pinned(const NetShape& net, int B);
hipError_t launch_wide(anakin* h, const RolloutArgs& args);
int rollout_resident_tile(const NetShape& net, int env_kind, int B);
size_t rollout_lds_bytes(const NetShape& net, const EnvDims& env, int TM, int* ldx);

}  // namespace ank
