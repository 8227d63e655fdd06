// Argument blocks of the dense-layer backward kernels (vector-ALU and
// matrix-core versions take the same ones).
#pragma once
#include "internal.h"

namespace ank {

// where the first layer's input comes from: the compact state snapshots
struct ObsSrc {
    int kind, B;
    EnvDims env;
    const uint32_t* s0; const float* f0; const float* f1;   // [T+1][B], row m = t*B + b
    const uint32_t* walls;                                   // [8][B]
};

// heads folded into the top hidden layer's products: dY is not read but formed on the way in,
//   dY[m][j] = (hl[m][j] > 0) * sum_a wh[j][a] dhead[m][a]
// from the layer's own forward activations hl, the per-sample head gradient and the head matrix
struct HeadFuse {
    const float* hl;      // [M][N] activations of the top hidden layer (null: dY is read from memory)
    const float* dhead;   // [M][NHP]
    const float* wh;      // [N][NH]
    int NH, NHP, bf16;    // bf16: wh is rounded to bfloat16
    float* head_partial;  // dW product only: [splits][N*NH + NH] partial sums of the head matrix and bias gradients
};

// first layer folded into the dX product that forms dZ_1, one partial per workgroup along the samples (dZ_1 itself is then not
// written: nothing else reads it).  Pendulum: dW_1[c][i] = sum_m o_c(m) dZ_1[m][i] for the three observation features
// o = (cos th, sin th, thd) of sample m.  Catch: the board's cells in place of the features.  db_1[i] = sum_m dZ_1[m][i].
struct FirstFuse {
    const float* f0; const float* f1;   // [M] stored angle and angular velocity (null: not the pendulum's)
    const uint32_t* s0;                 // [M] stored states (null: not Catch's)
    int cols, paddle_row0, cells;       // Catch: columns of the board, the bottom row's first cell, all cells
    float* partial;                     // [workgroups][features*K + K]
};
// dX[m][i] = (x[m][i] > 0) * sum_j dY[m][j] W[i][j];  W is [K][N] row-major (K = inputs, N = outputs)
struct GemmNtArgs {
    int M, K, N, bf16;
    HeadFuse hf;
    FirstFuse ff;
    const float* dy;      // [M][N]
    const float* w;       // [K][N]
    const float* x;       // [M][K] forward activations (relu mask)
    float* dx;            // [M][K]
    const void* w3;       // W as three bfloat16 terms in operand order (split_weights)
};

// weights of the layers whose dX product runs on split operands
struct SplitWeightsArgs { int n, bf16; int K[MAX_LAYERS], N[MAX_LAYERS]; const float* w[MAX_LAYERS]; void* out[MAX_LAYERS]; };

// partial[s][i][j] = sum over rows of chunk s of x[m][i] dY[m][j]; partial[s][K*N + j] = column sums of dY
struct GemmTnArgs {
    int M, K, N, ldy, bf16, splits, rows, tiles_i, use_obs;   // ldy: row stride of dy (>= N)
    HeadFuse hf;
    const float* x;       // [M][K], unused when use_obs
    const float* dy;      // [M][N]
    float* partial;       // [splits][K*N + N]
    ObsSrc obs;
};

// the head matrix as the products read it
__device__ __forceinline__ float head_weight(const HeadFuse& hf, int j, int k)
{
    const float x = hf.wh[(size_t)j * hf.NH + k];
    return hf.bf16 ? bf16_to_f(bf16_bits(x)) : x;
}

hipError_t launch_gemm_nt_valu(const GemmNtArgs& a, hipStream_t s);
hipError_t launch_gemm_tn_valu(GemmTnArgs a, hipStream_t s);
hipError_t launch_gemm_nt_mfma(const GemmNtArgs& a, hipStream_t s);
hipError_t launch_gemm_tn_mfma(GemmTnArgs a, hipStream_t s);
SplitWeightsArgs split_weights_args(const anakin* h);   // what the update's backward pass needs split (nothing: n = 0)
// both products of a layer whose sides are multiples of 64 (split_gemm_shape), on split operands (gemm_split.hip)
hipError_t launch_gemm_tn_nt_split(const NetShape& net, int l, const GemmTnArgs& t, const GemmNtArgs& n, int nt_blocks, hipStream_t s);

}  // namespace ank
