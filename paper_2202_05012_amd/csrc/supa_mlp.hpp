// supa_mlp.hpp -- arguments of the surrogate's matrix product kernels
// (supa_mlp.hip), shared with their C ABI (supa_surrogate_api.hip).
#pragma once
#include <stdint.h>

namespace supa {

// Arguments of the surrogate's matrix product (supa_mlp.hip).
struct GemmArgs {
    int M, N, K;
    const uint16_t *A;   // TA == 0: [M][lda] (row-major M x K); TA == 1: [K][lda] (K x M)
    const uint16_t *B;   // TB == 0: [K][ldb] (K x N);           TB == 1: [N][ldb] (N x K)
    int lda, ldb;
    const float *bias;   // [N] or null
    void *C;             // float [M][ldc] (EPI_F32, EPI_BIAS_F32) or bf16 [M][ldc]
    int ldc;
    uint16_t *pre;       // EPI_BIAS_GELU: pre-activation out; EPI_GELU_GRAD: in (bf16 [M][ldc])
    int k_chunk;         // > 0: block z covers K range [z k_chunk, (z+1) k_chunk) and writes
                         //   its partial product at C + z M ldc (EPI_F32); 0: all of K
    int split;           // EPI_GATE: columns from split on are log-variances
    float s_clamp;       // EPI_GATE: log-variance clamp
    const float *e0;     // EPI_GATE with counts: per row; a mean column counts as occupied when
    float cnt_scale;     //   mu > cnt_scale / e0[row] (null e0: no counts)
};

// Arguments of the fused forward pass (mlp_fused_kernel): an MLP of
// n_hidden GELU layers 256 wide on k_in inputs, then either the last hidden
// activations (n_out == 0) or a final linear layer of n_out outputs.
constexpr int MLP_FUSED_MAX_HIDDEN = 8;
struct MlpFusedArgs {
    int B, k_in, n_hidden, n_out;
    const uint16_t *x;   // bf16 [B][ldx], k_in columns
    int ldx;
    // layer l's weights transposed, bf16 [out][in]: in = k_in for l = 0, else
    // 256 with the input index permuted (the order the previous layer's
    // products leave the activations in registers)
    const uint16_t *wt[MLP_FUSED_MAX_HIDDEN + 1];
    const float *bias[MLP_FUSED_MAX_HIDDEN + 1];
    float *out;          // n_out > 0: float [B][ldo]
    int ldo;
    uint16_t *h;         // n_out == 0: bf16 [B][ldh], the last hidden activations
    int ldh;
};

// Arguments of a training step (supa_train.hip): n_hidden layers of 256 on
// k_in inputs, 2 D outputs (means, then log-variances); layer l of 0 ..
// n_hidden maps its input (x, or activations act[l - 1]) to the next.
struct TrainArgs {
    int B, n_hidden, k_in, D;
    const uint16_t *x;                                  // bf16 [B][ldx]
    int ldx;
    const float *img, *e0;                              // targets y_scale img / e0: [B][D], [B]
    float y_scale, s_clamp;
    int mse_mean;
    float lr, b1, b2, eps, c1, c2;                      // Adam (c1, c2: bias corrections)
    float *loss;                                        // the loss sum is added here
    const uint16_t *wb[MLP_FUSED_MAX_HIDDEN + 1];       // bf16 weights [in][out]
    uint16_t *wb_out[MLP_FUSED_MAX_HIDDEN + 1];         // the same, refreshed by Adam
    const float *bias[MLP_FUSED_MAX_HIDDEN + 1];
    float *p_w[MLP_FUSED_MAX_HIDDEN + 1], *m_w[MLP_FUSED_MAX_HIDDEN + 1], *v_w[MLP_FUSED_MAX_HIDDEN + 1];
    float *p_b[MLP_FUSED_MAX_HIDDEN + 1], *m_b[MLP_FUSED_MAX_HIDDEN + 1], *v_b[MLP_FUSED_MAX_HIDDEN + 1];
    // workspace (train_layout)
    uint16_t *act[MLP_FUSED_MAX_HIDDEN], *pre[MLP_FUSED_MAX_HIDDEN], *g[MLP_FUSED_MAX_HIDDEN];   // bf16 [B][256]
    uint16_t *dout;                                     // bf16 [B][ldd], 2 D columns, zeros beyond
    int ldd, Bp;                                        // Bp: rows of the gradients (B up to whole steps)
    uint16_t *wt[MLP_FUSED_MAX_HIDDEN + 1];             // bf16 weights [out][in]
    float *dw, *db;                                     // partial sums of the gradients
    int64_t dw_off[MLP_FUSED_MAX_HIDDEN + 1], db_off[MLP_FUSED_MAX_HIDDEN + 1];
    int tr_block[MLP_FUSED_MAX_HIDDEN + 2];             // first transpose block of each layer
    int wg_tiles[MLP_FUSED_MAX_HIDDEN + 1], wg_parts[MLP_FUSED_MAX_HIDDEN + 1], wg_rows[MLP_FUSED_MAX_HIDDEN + 1];
    int ad_block[2 * (MLP_FUSED_MAX_HIDDEN + 1) + 1];   // first Adam block of each tensor (W, b per layer)
};

}  // namespace supa
