// supa_train.hip -- one training step of the surrogate MLP for gfx950, for
// networks whose hidden layers are all 256 wide.
//
// Seven launches, in order:
//   transpose   bf16 weights [in][out] -> [out][in] (operands of the forward)
//   forward     every hidden layer of 32 rows per workgroup, activations
//               handed on through LDS, pre-activations and activations stored
//               for the backward
//   final       the output layer and the loss: a mean tile and the
//               log-variance tile of the same bins meet in one lane, so the
//               [B][2D] output is never written; leaves d loss / d out
//   input grad  d out W^T and GELU': the last hidden layer's gradient
//   backward    the hidden layers downwards, 32 rows per workgroup, through LDS
//   weight grad activations^T gradients of every layer in one launch, split
//               over the rows, and the bias gradients from the same tiles
//   adam        partial sums in order, then the step, of every tensor at once
// Every product is bf16 x bf16 accumulated in float32 by the matrix cores.
// What is rounded to bf16, and where, is as in the layer-by-layer products of
// supa_mlp.hip: weights, activations, pre-activations and gradients.  The
// products whose results are rounded use the same instruction, each sum over
// all of K in one accumulator in the same order (v_mfma_f32_16x16x32_bf16;
// operand: lane l holds row l & 15, k = 8 (l >> 4) .. + 8; result: column
// l & 15, rows 4 (l >> 4) .. + 4), so that no bf16 value differs from theirs
// by a rounding; the weight gradients, which stay float32, use
// v_mfma_f32_32x32x16_bf16 (row l & 31, k = 8 (l >> 5) .. + 8; column l & 31,
// row 8 (r >> 2) + 4 (l >> 5) + (r & 3)).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "supa_device.hpp"
#include "supa_mlp.hpp"

namespace supa {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4;

constexpr int W = 256;             // hidden width
constexpr int ROWS = 32;           // rows per workgroup of forward and backward
constexpr int PITCH = W + 8;       // LDS row of activations (bf16): rows 4 banks apart

__device__ __forceinline__ float bf_to_f(uint32_t h) { return __uint_as_float(h << 16); }

// two floats to a pair of bf16 (round to nearest even)
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float gelu_exact(float a) { return 0.5f * a * erfcf(-a * 0.707106781f); }

__device__ __forceinline__ float gelu_slope(float a) {
    return 0.5f * erfcf(-a * 0.707106781f) + a * 0.398942280f * __expf(-0.5f * a * a);
}

__device__ __forceinline__ floatx4_t mfma16(u32x4_t a, u32x4_t b, floatx4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                    0, 0, 0);
}

__device__ __forceinline__ floatx16_t mfma32(u32x4_t a, u32x4_t b, floatx16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                    0, 0, 0);
}

// All but this wave's latest N vector memory operations are done.  (The
// builtin, not inline assembly: the compiler then knows that copies into LDS
// have landed and adds no wait of its own before the tile is read.)
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

// The same, and every wave of the workgroup has got here.  (__syncthreads
// waits for all of a wave's operations, stores included.)
template <int N>
__device__ __forceinline__ void meet() {
    wait_vm<N>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr floatx16_t kZero16 = {};
constexpr floatx4_t kZero4 = {};
constexpr u32x4_t kNone = {};

}  // namespace

// ---------------------------------------------------------------------------
// Weights transposed, every layer in one launch: 64 x 64 tiles through LDS,
// 16-byte reads and writes (both dimensions are multiples of 8).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) train_transpose_kernel(TrainArgs a) {
    __shared__ uint16_t t[64][72];
    int l = 0;
    while (l < a.n_hidden && (int)blockIdx.x >= a.tr_block[l + 1]) ++l;
    const int in = l == 0 ? a.k_in : W, out = l == a.n_hidden ? 2 * a.D : W;
    const int tile = (int)blockIdx.x - a.tr_block[l], tn = (out + 63) / 64;
    const int k0 = tile / tn * 64, n0 = tile % tn * 64;
    for (int c = threadIdx.x; c < 512; c += 256) {
        const int k = c >> 3, n = (c & 7) * 8;
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (k0 + k < in && n0 + n < out) v = *(const u32x4_t *)(a.wb[l] + (int64_t)(k0 + k) * out + n0 + n);
        *(u32x4_t *)&t[k][n] = v;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < 512; c += 256) {
        const int n = c >> 3, k = (c & 7) * 8;
        if (k0 + k >= in || n0 + n >= out) continue;
        uint32_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (uint32_t)t[k + 2 * q][n] | ((uint32_t)t[k + 2 * q + 1][n] << 16);
        *(u32x4_t *)(a.wt[l] + (int64_t)(n0 + n) * in + k0 + k) = u32x4_t{v[0], v[1], v[2], v[3]};
    }
}

// All waves' LDS accesses are done (their loads and stores to memory need not be).
__device__ __forceinline__ void meet_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------
// Hidden layers forward: 32 rows per workgroup, so that a batch of 8,192 rows
// covers the 256 CUs; wave w takes outputs 32 w .. + 32 of all rows.  A wave's
// weights are its own (no two waves share an element), so they come straight
// from memory into registers in operand layout, the next layer's while this
// one's activations are evaluated; the activations pass to the other waves
// through LDS.  Bound by latency (four layers in a row) and by erfc.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(512) train_forward_kernel(TrainArgs a) {
    __shared__ __attribute__((aligned(16))) uint16_t X[2][ROWS][PITCH];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
    const int m0 = blockIdx.x * ROWS + lc, n0 = 32 * wave + lc;      // + 16 j, + 16 i
    u32x4_t w[2][8], x[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int k = 32 * kk + 8 * lq, m = m0 + 16 * i;
            w[i][kk] = x[i][kk] = kNone;
            if (k < a.k_in) {
                w[i][kk] = *(const u32x4_t *)(a.wt[0] + (int64_t)(n0 + 16 * i) * a.k_in + k);
                if (m < a.B) x[i][kk] = *(const u32x4_t *)(a.x + (int64_t)m * a.ldx + k);
            }
        }
    for (int l = 0; l < a.n_hidden; ++l) {
        const int ks = l == 0 ? (a.k_in + 31) / 32 : 8;
        floatx4_t acc[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            if (kk < ks) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(w[i][kk], x[j][kk], acc[i][j]);
            }
        if (l + 1 < a.n_hidden) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kk = 0; kk < 8; ++kk)
                    w[i][kk] = *(const u32x4_t *)(a.wt[l + 1] + (int64_t)(n0 + 16 * i) * W + 32 * kk + 8 * lq);
        }
        uint16_t(*Xo)[PITCH] = X[l & 1];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int f = 32 * wave + 16 * i + 4 * lq;
            const floatx4_t bv = *(const floatx4_t *)(a.bias[l] + f);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int m = m0 + 16 * j;
                float v[4], y[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[q] = acc[i][j][q] + bv[q];
                    y[q] = gelu_exact(v[q]);
                }
                const uint2 pv = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
                const uint2 yv = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
                if (m < a.B) {
                    *(uint2 *)(a.pre[l] + (int64_t)m * W + f) = pv;
                    *(uint2 *)(a.act[l] + (int64_t)m * W + f) = yv;
                }
                *(uint2 *)&Xo[lc + 16 * j][f] = yv;
            }
        }
        // one barrier per layer: the other buffer was last read before this one's writes
        meet_lds();
        if (l + 1 < a.n_hidden) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) x[j][kk] = *(const u32x4_t *)&Xo[lc + 16 * j][32 * kk + 8 * lq];
        }
    }
}

// ---------------------------------------------------------------------------
// Output layer, loss and its gradient.  A workgroup of eight waves takes 256
// rows (32 per wave, all of K = 256 in registers) through a range of tiles
// of 64 bins: the tile's 64 mean rows and 64 log-variance rows of W^T stream
// through LDS (two buffers copied straight into LDS, the layout of the gate
// kernel in supa_mlp.hip), and the products leave both outputs of a bin in
// the same lane, which turns them into the gradient pair at once.  Bound by
// the images read and the gradients written (4 + 4 bytes per bin).
// ---------------------------------------------------------------------------
constexpr int FT_BINS = 64, FT_ROWS = 256;
constexpr int XG_M = 64, XG_K = 128, XG_STEP = 64;      // input gradient: rows, inputs, outputs per step
typedef uint16_t FtTile[2 * FT_BINS][W];

__device__ __forceinline__ void ft_issue(const TrainArgs &a, int t, FtTile &T, float *Bt, int wave, int lane) {
    // chunk group g = wave (chunks 4 g .. + 4 of every row), copy q: rows 16 q .. + 16
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int row = 16 * q + (lane >> 2);
        const int c = 4 * wave + ((lane & 3) ^ ((row >> 2) & 3));
        // rows past the last bin repeat it (their results are not used)
        const int bin = min(t * FT_BINS + (row & 63), a.D - 1);
        const uint16_t *src = a.wt[a.n_hidden] + (int64_t)(bin + (row >= FT_BINS ? a.D : 0)) * W + c * 8;
        __builtin_amdgcn_global_load_lds(
            src, (__attribute__((address_space(3))) void *)((char *)&T[0][0] + 8192 * wave + 1024 * q), 16, 0, 0);
    }
    if (wave < 2) {
        const int bin = min(t * FT_BINS + lane, a.D - 1);
        __builtin_amdgcn_global_load_lds(a.bias[a.n_hidden] + bin + (wave ? a.D : 0),
                                         (__attribute__((address_space(3))) void *)(Bt + 64 * wave), 4, 0, 0);
    }
}

// The tile's products with this wave's 32 rows, and the loss: bins 16 i + 4 lq
// .. + 4 of rows 16 j + lc, means in mu[i][j], log-variances in lv[i][j].
__device__ __forceinline__ float ft_loss(const TrainArgs &a, int t, const FtTile &T, const float *Bt,
                                         const u32x4_t (&h)[2][8], int lc, int lq, int m0, const float (&e0)[2],
                                         const float (&ie0)[2], float inv_n) {
    // the targets, in flight during the products
    floatx4_t y[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int bin = t * FT_BINS + 16 * i + 4 * lq, m = m0 + 16 * j;
            y[i][j] = kZero4;
            if (m < a.B && bin < a.D) y[i][j] = *(const floatx4_t *)(a.img + (int64_t)m * a.D + bin);
        }
    floatx4_t mu[4][2], lv[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mu[i][j] = lv[i][j] = kZero4;
    // a row's chunks are permuted by bits 2, 3 of the row: the same for every block of 16 rows
    const char *base = (const char *)&T[0][0] + 64 * lc + 16 * (lq ^ (lc >> 2));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4_t wm = *(const u32x4_t *)(base + 8192 * kk + 1024 * i);
            const u32x4_t wv = *(const u32x4_t *)(base + 8192 * kk + 1024 * (i + 4));
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                mu[i][j] = mfma16(wm, h[j][kk], mu[i][j]);
                lv[i][j] = mfma16(wv, h[j][kk], lv[i][j]);
            }
        }
    // the targets and the next tile's copies have arrived (before this tile's
    // stores are issued, which nobody waits for at the tile's end)
    wait_vm<0>();
    asm volatile("" ::: "memory");
    float l = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = 16 * i + 4 * lq, bin = t * FT_BINS + o;
        const floatx4_t bm = *(const floatx4_t *)&Bt[o], bs = *(const floatx4_t *)&Bt[64 + o];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + 16 * j;
            float dm[4], ds[4], lj = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float sr = lv[i][j][q] + bs[q];
                const float s = __builtin_amdgcn_fmed3f(sr, -a.s_clamp, a.s_clamp);
                // (y_scale img) / e0 correctly rounded, from the rounded
                // reciprocal (Markstein's two fused steps; an e0 or target
                // that is zero, infinite or no number as in a division)
                const float yn = y[i][j][q] * a.y_scale;
                const float y0 = yn * ie0[j];
                const float yq = __builtin_amdgcn_div_fixupf(fmaf(fmaf(-y0, e0[j], yn), ie0[j], y0), e0[j], yn);
                const float r = yq - (mu[i][j][q] + bm[q]);
                const float ie = __expf(-s);
                const float e2 = r * r * ie;
                lj += 0.5f * (s + e2);
                dm[q] = -r * (a.mse_mean ? 1.0f : ie) * inv_n;
                ds[q] = fabsf(sr) <= a.s_clamp ? 0.5f * (1.0f - e2) * inv_n : 0.0f;
            }
            if (m < a.Bp && bin < a.D) {             // rows past the batch: zeros
                const bool in = m < a.B;
                l += in ? lj : 0.0f;
                uint16_t *d = a.dout + (int64_t)m * a.ldd + bin;
                *(uint2 *)d = make_uint2(in ? pack2(dm[0], dm[1]) : 0u, in ? pack2(dm[2], dm[3]) : 0u);
                *(uint2 *)(d + a.D) = make_uint2(in ? pack2(ds[0], ds[1]) : 0u, in ? pack2(ds[2], ds[3]) : 0u);
            }
        }
    }
    return l;
}

__global__ void __launch_bounds__(512) train_final_kernel(TrainArgs a, int tiles_per_block) {
    __shared__ __attribute__((aligned(1024))) FtTile T0, T1;
    __shared__ __attribute__((aligned(16))) float B0[128], B1[128];
    __shared__ float part[8];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
    const int m0 = blockIdx.x * FT_ROWS + 32 * wave + lc;
    const int tiles = (a.D + FT_BINS - 1) / FT_BINS;
    const int t0 = blockIdx.y * tiles_per_block, t1 = min(tiles, t0 + tiles_per_block);
    if (t0 >= t1) return;
    ft_issue(a, t0, T0, B0, wave, lane);
    u32x4_t h[2][8];
    float e0[2], ie0[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = m0 + 16 * j;
        e0[j] = m < a.B ? a.e0[m] : 1.0f;
        ie0[j] = 1.0f / e0[j];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            h[j][kk] = kNone;
            if (m < a.B) h[j][kk] = *(const u32x4_t *)(a.act[a.n_hidden - 1] + (int64_t)m * W + 32 * kk + 8 * lq);
        }
    }
    // the columns that pad the gradient's rows to whole K steps
    const int pad = (a.D + XG_STEP / 2 - 1) / (XG_STEP / 2) * XG_STEP - 2 * a.D;
    if (blockIdx.y == 0 && pad > 0)
        for (int q = lane; q < 32 * pad; q += 64) {
            const int m = blockIdx.x * FT_ROWS + 32 * wave + q / pad;
            if (m < a.B) a.dout[(int64_t)m * a.ldd + 2 * a.D + q % pad] = 0;
        }
    const float inv_n = 1.0f / (float)((int64_t)a.B * a.D);
    float l = 0.0f;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int t = t0; t < t1; t += 2) {
        // (distinct LDS variables: reads of one tile need not wait for the copy into the other)
        if (t + 1 < t1) ft_issue(a, t + 1, T1, B1, wave, lane);
        l += ft_loss(a, t, T0, B0, h, lc, lq, m0, e0, ie0, inv_n);
        meet<63>();
        if (t + 1 < t1) {
            if (t + 2 < t1) ft_issue(a, t + 2, T0, B0, wave, lane);
            l += ft_loss(a, t + 1, T1, B1, h, lc, lq, m0, e0, ie0, inv_n);
            meet<63>();
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) part[wave] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.0f;
        for (int q = 0; q < 8; ++q) s += part[q];
        atomicAdd(a.loss, s);
    }
}

// ---------------------------------------------------------------------------
// d out W^T times GELU': 64 rows x 128 inputs per workgroup (8,192 rows: 256
// workgroups), wave tiles of 32 x 32, the whole reduction over the outputs in
// order, K steps of 64 copied straight into LDS, three steps ahead in four
// buffers (distinct LDS variables, so that reads of one need not wait for the
// copies into the others; one barrier per step).  The weights come from the
// transposed copy, whose rows [out] are 512 bytes: a step's rows of the
// matrix as stored lie 4 D bytes apart, all in one L2 channel when that is a
// multiple of 4 KB (the gradient's rows are padded for the same reason), and
// reading them across rows is what ds_read_b64_tr_b16 does.  Gradient chunk c
// (16 bytes) of row r sits at c ^ ((r >> 1) & 7), weight chunk c of output n at
// c ^ tr_swizzle(n): no two lanes of a read's group share a bank.
// ---------------------------------------------------------------------------
struct XgTile {
    char w[XG_STEP * 2 * XG_K], g[XG_M * 2 * XG_STEP];
};

__device__ __forceinline__ int tr_swizzle(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }

__device__ __forceinline__ void xg_issue(const TrainArgs &p, int m0, int k0, int step, XgTile &T, int wave, int lane) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        // four outputs (256 bytes each) per instruction; past the last output
        // the gradient holds zeros: any weight will do
        const int blk = 2 * wave + q, r = 4 * blk + (lane >> 4);
        const int n = min(step * XG_STEP + r, 2 * p.D - 1);
        const uint16_t *src = p.wt[p.n_hidden] + (int64_t)n * W + k0 + 8 * ((lane & 15) ^ tr_swizzle(r));
        __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(&T.w[0] + 1024 * blk), 16, 0, 0);
    }
    const int r = 8 * wave + (lane >> 3);
    const uint16_t *src = p.dout + (int64_t)min(m0 + r, p.B - 1) * p.ldd + step * XG_STEP + 8 * ((lane & 7) ^ ((r >> 1) & 7));
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(&T.g[0] + 1024 * wave), 16, 0, 0);
}

__device__ __forceinline__ void xg_step(XgTile &T, floatx4_t (&acc)[2][2], int wk, int wm, int lc, int lq) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        u32x4_t x[2], y[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = (wk >> 3) + 2 * i + ((lc >> 1) & 1), j = lc >> 2;
            short4_t v[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_short4 *)(&T.w[0] + 256 * (32 * kk + 8 * lq + 4 * h + j) + 16 * (c ^ ((j << 1) | h)) + 8 * (lc & 1)));
            struct { short4_t a, b; } two = {v[0], v[1]};
            x[i] = __builtin_bit_cast(u32x4_t, two);
            const int rm = wm + 16 * i + lc;
            y[i] = *(const u32x4_t *)(&T.g[0] + 128 * rm + 16 * ((4 * kk + lq) ^ ((rm >> 1) & 7)));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(x[i], y[j], acc[i][j]);
    }
}

__global__ void __launch_bounds__(512) train_input_grad_kernel(TrainArgs p) {
    __shared__ __attribute__((aligned(1024))) XgTile T0, T1, T2, T3;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
    const int m0 = blockIdx.x * XG_M, k0 = blockIdx.y * XG_K;
    const int wk = (wave & 3) * 32, wm = (wave >> 2) * 32;
    const int steps = (2 * p.D + XG_STEP - 1) / XG_STEP;
    floatx4_t acc[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}};
    // step s: this wave's copies of it have landed once at most those of the
    // two later steps (three instructions each) are outstanding; after the
    // barrier everyone's have, and everyone has left the buffer of step s - 1.
    // Every stage of the main loop issues (past the end the last step again):
    // with a condition around it the compiler waits for everything.
#define XG_STAGE(S, CUR, FREE)                                                    \
    meet<6>();                                                                    \
    xg_issue(p, m0, k0, min((S) + 3, steps - 1), FREE, wave, lane);               \
    xg_step(CUR, acc, wk, wm, lc, lq);
    xg_issue(p, m0, k0, 0, T0, wave, lane);
    xg_issue(p, m0, k0, min(1, steps - 1), T1, wave, lane);
    xg_issue(p, m0, k0, min(2, steps - 1), T2, wave, lane);
    int s = 0;
    for (; s + 4 <= steps; s += 4) {
        XG_STAGE(s, T0, T3)
        XG_STAGE(s + 1, T1, T0)
        XG_STAGE(s + 2, T2, T1)
        XG_STAGE(s + 3, T3, T2)
    }
    meet<0>();
    if (s < steps) xg_step(T0, acc, wk, wm, lc, lq);
    if (s + 1 < steps) xg_step(T1, acc, wk, wm, lc, lq);
    if (s + 2 < steps) xg_step(T2, acc, wk, wm, lc, lq);
#undef XG_STAGE
    const int H = p.n_hidden;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + wm + 16 * j + lc, f = k0 + wk + 16 * i + 4 * lq;
            uint2 gv = make_uint2(0u, 0u);           // rows past the batch: zeros
            if (m < p.B) {
                const uint2 pv = *(const uint2 *)(p.pre[H - 1] + (int64_t)m * W + f);
                gv = make_uint2(
                    pack2(acc[i][j][0] * gelu_slope(bf_to_f(pv.x & 0xffffu)), acc[i][j][1] * gelu_slope(bf_to_f(pv.x >> 16))),
                    pack2(acc[i][j][2] * gelu_slope(bf_to_f(pv.y & 0xffffu)), acc[i][j][3] * gelu_slope(bf_to_f(pv.y >> 16))));
            }
            *(uint2 *)(p.g[H - 1] + (int64_t)m * W + f) = gv;
        }
}

// ---------------------------------------------------------------------------
// Hidden layers backward, 32 rows per workgroup (see the forward): g <-
// (g W^T) GELU' from the last hidden layer's gradient down to the first.
// Wave w takes inputs 32 w .. + 32; its weight rows [in][out] are contiguous
// in the reduction as they are stored.  The next layer's weights and
// preactivations are read while this one's are used, and no wave waits for its
// stores at a barrier (8,192 rows, 3 layers: 34 -> 29.6 us; the forward's
// barriers without that wait 34 -> 33.3).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(512) train_backward_kernel(TrainArgs a) {
    __shared__ __attribute__((aligned(16))) uint16_t X[2][ROWS][PITCH];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
    const int m0 = blockIdx.x * ROWS + lc, k0 = 32 * wave + lc;
    u32x4_t x[2][8];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            x[j][kk] = kNone;
            if (m0 + 16 * j < a.B)
                x[j][kk] = *(const u32x4_t *)(a.g[a.n_hidden - 1] + (int64_t)(m0 + 16 * j) * W + 32 * kk + 8 * lq);
        }
    // a layer's weights and preactivations, read while the layer before it is evaluated
    u32x4_t w[2][8];
    uint2 pre[2][2];
    auto read_weights = [&](int l) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                w[i][kk] = *(const u32x4_t *)(a.wb[l] + (int64_t)(k0 + 16 * i) * W + 32 * kk + 8 * lq);
    };
    auto read_pre = [&](int l) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                pre[i][j] = make_uint2(0u, 0u);
                if (m0 + 16 * j < a.B)
                    pre[i][j] = *(const uint2 *)(a.pre[l - 1] + (int64_t)(m0 + 16 * j) * W + 32 * wave + 16 * i + 4 * lq);
            }
    };
    if (a.n_hidden > 1) {
        read_weights(a.n_hidden - 1);
        read_pre(a.n_hidden - 1);
    }
    for (int l = a.n_hidden - 1; l >= 1; --l) {
        // gradient of hidden layer l - 1 from that of layer l (weights wb[l])
        floatx4_t acc[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(w[i][kk], x[j][kk], acc[i][j]);
        if (l > 1) read_weights(l - 1);
        uint16_t(*Xo)[PITCH] = X[l & 1];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int m = m0 + 16 * j, f = 32 * wave + 16 * i + 4 * lq;
                uint2 gv = make_uint2(0u, 0u);
                if (m < a.B) {
                    const uint2 pv = pre[i][j];
                    gv = make_uint2(pack2(acc[i][j][0] * gelu_slope(bf_to_f(pv.x & 0xffffu)),
                                          acc[i][j][1] * gelu_slope(bf_to_f(pv.x >> 16))),
                                    pack2(acc[i][j][2] * gelu_slope(bf_to_f(pv.y & 0xffffu)),
                                          acc[i][j][3] * gelu_slope(bf_to_f(pv.y >> 16))));
                }
                *(uint2 *)(a.g[l - 1] + (int64_t)m * W + f) = gv;          // (zeros past the batch)
                *(uint2 *)&Xo[lc + 16 * j][f] = gv;
            }
        if (l > 1) {
            read_pre(l - 1);
            meet_lds();
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) x[j][kk] = *(const u32x4_t *)&Xo[lc + 16 * j][32 * kk + 8 * lq];
        }
    }
}

// ---------------------------------------------------------------------------
// Weight and bias gradients of every layer in one launch: dW[k][n] = sum over
// rows of act[m][k] g[m][n], 256 inputs x 128 outputs per workgroup over a
// range of rows (float partial sums, added in order by the Adam kernel).
// Both operands are stored rows first, so the reduction runs across rows of
// the LDS tiles: ds_read_b64_tr_b16 hands each lane four rows of its column
// (two reads make an operand), which replaces a transposing store of single
// bf16.  Chunk c of row m sits at c ^ tr_swizzle(m): the four rows of a
// transposing read fall on different banks.  K steps of 64 rows are copied
// straight into LDS two steps ahead in three buffers (a step takes less time
// than a load from memory).  Gradient rows past the batch are zeros (their
// producers write them), so whatever stands beside them adds nothing; columns
// past a layer's inputs or outputs repeat others and are not stored.  The
// bias gradients are summed from the gradient tiles in passing.  A part has up
// to some thousand rows, too many for one float accumulator: every three steps
// (192 rows) the sums move to a second set of registers.  Root mean square
// error against float64, 8,192 rows, 10,240 outputs: 4.9e-8 (2,752 rows in one
// accumulator 1.6e-7; the layer-by-layer products, 1,184 rows, 8.2e-8), in
// 70.0 us against 69.5.
// ---------------------------------------------------------------------------
constexpr int WG_N = 128, WG_K = 64;

struct WgTile {
    char a[WG_K * 512], g[WG_K * 256];
};

struct WgJob {
    const uint16_t *act, *g;
    int lda, ldg, in, out, n0;
};

__device__ __forceinline__ void wg_issue(const WgJob &J, int B, int m0, WgTile &T, int wave, int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {                      // two rows of activations per instruction
        const int blk = 4 * wave + q, m = 2 * blk + (lane >> 5), k = 8 * ((lane & 31) ^ tr_swizzle(m));
        const uint16_t *src = J.act + (int64_t)min(m0 + m, B - 1) * J.lda + (k < J.in ? k : 0);
        __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(&T.a[0] + 1024 * blk), 16, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {                      // four rows of the gradient
        const int blk = 2 * wave + q, m = 4 * blk + (lane >> 4), n = J.n0 + 8 * ((lane & 15) ^ tr_swizzle(m));
        const uint16_t *src = J.g + (int64_t)(m0 + m) * J.ldg + (n < J.out ? n : 0);
        __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(&T.g[0] + 1024 * blk), 16, 0, 0);
    }
}

// operand of 32 columns from col0 (a multiple of 32), rows 16 kk .. + 16, of a
// tile with PB bytes per row
template <int PB>
__device__ __forceinline__ u32x4_t wg_operand(char *T, int col0, int kk, int lane) {
    const int j = (lane & 15) >> 2, lh = lane >> 5;
    const int c = (col0 >> 3) + 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
    short4_t v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int m = 16 * kk + 8 * lh + 4 * h + j;
        // (one offset: the compiler follows few steps back to the LDS variable, and
        // reads it cannot place wait for every copy in flight)
        const int at = PB * m + 16 * (c ^ ((j << 1) | h)) + 8 * (lane & 1);
        v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(T + at));
    }
    struct { short4_t a, b; } two = {v[0], v[1]};
    return __builtin_bit_cast(u32x4_t, two);
}

// Sums of a range of rows: of the products (inputs 32 i, outputs 32 j) and of
// the gradient.
struct WgSums {
    floatx16_t w[2][2];
    float b[8];
};

__device__ __forceinline__ void wg_clear(WgSums &S) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) S.w[i][j] = kZero16;
#pragma unroll
    for (int q = 0; q < 8; ++q) S.b[q] = 0.0f;
}

// adds S to T and clears it
__device__ __forceinline__ void wg_fold(WgSums &T, WgSums &S) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) T.w[i][j] += S.w[i][j];
#pragma unroll
    for (int q = 0; q < 8; ++q) T.b[q] += S.b[q];
    wg_clear(S);
}

// the operands of 16 rows
struct WgOps {
    u32x4_t x[2], y[2];
};

__device__ __forceinline__ void wg_read(WgTile &T, WgOps &O, int kk, int wk, int wn, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) O.x[i] = wg_operand<512>(&T.a[0], wk + 32 * i, kk, lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) O.y[j] = wg_operand<256>(&T.g[0], wn + 32 * j, kk, lane);
}

__device__ __forceinline__ void wg_mul(WgSums &S, const WgOps &O) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) S.w[i][j] = mfma32(O.x[i], O.y[j], S.w[i][j]);
}

// A step's products and bias sums; `meanwhile` runs while its first operands are
// on their way (left to itself the compiler issues the copies of a later step
// first, and reads no operand ahead: 74 us instead of 70 for the kernel).
template <typename F>
__device__ __forceinline__ void wg_step(WgTile &T, WgSums &S, int wk, int wn, int lane, F &&meanwhile) {
    WgOps p, q;
    wg_read(T, p, 0, wk, wn, lane);
    wg_read(T, q, 1, wk, wn, lane);
    __builtin_amdgcn_sched_barrier(0);
    meanwhile();
    wg_mul(S, p);
    wg_read(T, p, 2, wk, wn, lane);
    wg_mul(S, q);
    wg_read(T, q, 3, wk, wn, lane);
    // bias: this thread's chunk (of 16) of two rows
    u32x4_t v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int m = ((int)threadIdx.x >> 4) + 32 * r;
        const int at = 256 * m + 16 * (((int)threadIdx.x & 15) ^ tr_swizzle(m));
        v[r] = *(const u32x4_t *)(&T.g[0] + at);
    }
    wg_mul(S, p);
    wg_mul(S, q);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            S.b[2 * t] += bf_to_f(v[r][t] & 0xffffu);
            S.b[2 * t + 1] += bf_to_f(v[r][t] >> 16);
        }
}

__global__ void __launch_bounds__(512) train_weight_grad_kernel(TrainArgs a) {
    __shared__ __attribute__((aligned(1024))) WgTile T0, T1, T2;
    __shared__ __attribute__((aligned(16))) float bsum[32][WG_N];      // 160 KB with the tiles: all of a CU's LDS
    // the output layer's blocks first (the longest), then the others
    int l = a.n_hidden;
    int b = blockIdx.x;
    for (; l > 0 && b >= a.wg_tiles[l] * a.wg_parts[l]; --l) b -= a.wg_tiles[l] * a.wg_parts[l];
    const int tile = b % a.wg_tiles[l], part = b / a.wg_tiles[l];
    WgJob J;
    J.in = l == 0 ? a.k_in : W;
    J.out = l == a.n_hidden ? 2 * a.D : W;
    J.act = l == 0 ? a.x : a.act[l - 1];
    J.lda = l == 0 ? a.ldx : W;
    J.g = l == a.n_hidden ? a.dout : a.g[l];
    J.ldg = l == a.n_hidden ? a.ldd : W;
    J.n0 = tile * WG_N;
    const int m_begin = part * a.wg_rows[l], m_end = min(a.B, m_begin + a.wg_rows[l]);
    const int steps = (m_end - m_begin + WG_K - 1) / WG_K;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lc = lane & 31, lh = lane >> 5;
    const int wk = (wave >> 1) * 64, wn = (wave & 1) * 64;
    WgSums sum, acc;             // of the rows before the latest few steps, and of these
    wg_clear(sum);
    wg_clear(acc);
    // (see train_input_grad_kernel; six copy instructions per wave and step)
    auto none = [] {};
    auto issue = [&](int step, WgTile &T) { wg_issue(J, a.B, m_begin + WG_K * min(step, steps - 1), T, wave, lane); };
    issue(0, T0);
    issue(1, T1);
    int s = 0;
    for (; s + 3 <= steps; s += 3) {
        meet<6>();
        wg_step(T0, acc, wk, wn, lane, [&] {
            issue(s + 2, T2);
            wg_fold(sum, acc);
        });
        meet<6>();
        wg_step(T1, acc, wk, wn, lane, [&] { issue(s + 3, T0); });
        meet<6>();
        wg_step(T2, acc, wk, wn, lane, [&] { issue(s + 4, T1); });
    }
    meet<0>();
    if (s < steps) wg_step(T0, acc, wk, wn, lane, none);
    if (s + 1 < steps) wg_step(T1, acc, wk, wn, lane, none);
    wg_fold(sum, acc);
    float *out = a.dw + a.dw_off[l] + (int64_t)part * J.in * J.out;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = wk + 32 * i + 8 * (r >> 2) + 4 * lh + (r & 3), n = J.n0 + wn + 32 * j + lc;
                if (k < J.in && n < J.out) out[(int64_t)k * J.out + n] = sum.w[i][j][r];
            }
    // bias: thread t holds the sums of chunk t & 15 over rows t >> 4 (of each
    // 32); these are added in pairs
    *(floatx4_t *)&bsum[threadIdx.x >> 4][8 * (threadIdx.x & 15)] = floatx4_t{sum.b[0], sum.b[1], sum.b[2], sum.b[3]};
    *(floatx4_t *)&bsum[threadIdx.x >> 4][8 * (threadIdx.x & 15) + 4] = floatx4_t{sum.b[4], sum.b[5], sum.b[6], sum.b[7]};
    __syncthreads();
    if (threadIdx.x < WG_N && J.n0 + (int)threadIdx.x < J.out) {
        float t[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) t[q] = bsum[q][threadIdx.x];
#pragma unroll
        for (int w = 16; w > 0; w >>= 1)
#pragma unroll
            for (int q = 0; q < w; ++q) t[q] += t[q + w];
        a.db[a.db_off[l] + (int64_t)part * J.out + J.n0 + threadIdx.x] = t[0];
    }
}

// ---------------------------------------------------------------------------
// Adam (Kingma & Ba 2015) on every tensor in one launch: the gradient's
// partial sums in order, moments, weights, and the weights' bf16 copy.  Four
// elements per thread (every tensor's size is a multiple of 8).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) train_adam_kernel(TrainArgs a) {
    int t = 0;
    while ((int)blockIdx.x >= a.ad_block[t + 1]) ++t;
    const int l = t >> 1, is_b = t & 1;
    const int in = l == 0 ? a.k_in : W, out = l == a.n_hidden ? 2 * a.D : W;
    const int64_t n = is_b ? out : (int64_t)in * out;
    const int64_t i = ((int64_t)((int)blockIdx.x - a.ad_block[t]) * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    const float *part = is_b ? a.db + a.db_off[l] : a.dw + a.dw_off[l];
    float *pp = is_b ? a.p_b[l] : a.p_w[l], *pm = is_b ? a.m_b[l] : a.m_w[l], *pv = is_b ? a.v_b[l] : a.v_w[l];
    floatx4_t g = *(const floatx4_t *)(part + i);
    for (int z = 1; z < a.wg_parts[l]; ++z) g += *(const floatx4_t *)(part + (int64_t)z * n + i);
    floatx4_t m = *(const floatx4_t *)(pm + i), v = *(const floatx4_t *)(pv + i), p = *(const floatx4_t *)(pp + i);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        m[q] = a.b1 * m[q] + (1.0f - a.b1) * g[q];
        v[q] = a.b2 * v[q] + (1.0f - a.b2) * g[q] * g[q];
        p[q] -= a.lr * (m[q] / a.c1) / (sqrtf(v[q] / a.c2) + a.eps);
    }
    *(floatx4_t *)(pm + i) = m;
    *(floatx4_t *)(pv + i) = v;
    *(floatx4_t *)(pp + i) = p;
    if (!is_b) *(uint2 *)(a.wb_out[l] + i) = make_uint2(pack2(p[0], p[1]), pack2(p[2], p[3]));
}

// ---------------------------------------------------------------------------
// Host side: sizes, workspace layout, launches.
// ---------------------------------------------------------------------------
static size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Fills the derived sizes of `a` (B, n_hidden, k_in, D given) and, with a base
// address, its workspace pointers; returns the workspace's bytes.
size_t train_layout(TrainArgs &a, char *base) {
    size_t used = 0;
    auto take = [&](size_t bytes) -> char * {
        char *p = base ? base + used : nullptr;
        used += al(bytes);
        return p;
    };
    const int H = a.n_hidden;
    const int64_t N = 2 * (int64_t)a.D;
    // gradient rows up to whole K steps of the weight gradients (zeros past the batch)
    a.Bp = (a.B + WG_K - 1) / WG_K * WG_K;
    const size_t rows = (size_t)a.Bp;
    for (int l = 0; l < H; ++l) {
        a.act[l] = (uint16_t *)take((size_t)a.B * W * 2);
        a.pre[l] = (uint16_t *)take((size_t)a.B * W * 2);
        a.g[l] = (uint16_t *)take(rows * W * 2);
    }
    // rows of the gradient: whole K steps, and an odd number of 256-byte units
    // when they are long, so that equal columns of consecutive rows lie in
    // different L2 channels (at 20 KB, a multiple of 4 KB, all in one)
    a.ldd = (int)((N + XG_STEP - 1) / XG_STEP * XG_STEP);
    if (a.ldd >= 1024) a.ldd = ((a.ldd + 127) / 128 | 1) * 128;
    a.dout = (uint16_t *)take(rows * a.ldd * 2);
    int64_t off_w = 0, off_b = 0;
    int tr = 0, ad = 0;
    for (int l = 0; l <= H; ++l) {
        const int64_t in = l == 0 ? a.k_in : W, out = l == H ? N : W;
        a.wt[l] = (uint16_t *)take((size_t)in * out * 2);
        a.tr_block[l] = tr;
        tr += (int)((in + 63) / 64 * ((out + 63) / 64));
        // weight gradients: tiles x parts fill the chip for the output layer,
        // 512 rows per part for the small ones
        a.wg_tiles[l] = (int)((out + WG_N - 1) / WG_N);
        int want = l == H ? std::max(1, 240 / a.wg_tiles[l]) : 16;
        want = std::max(1, std::min(want, (a.B + 511) / 512));
        a.wg_rows[l] = ((a.B + want - 1) / want + WG_K - 1) / WG_K * WG_K;
        a.wg_parts[l] = (a.B + a.wg_rows[l] - 1) / a.wg_rows[l];
        a.dw_off[l] = off_w;
        off_w += a.wg_parts[l] * in * out;
        a.db_off[l] = off_b;
        off_b += a.wg_parts[l] * out;
        a.ad_block[2 * l] = ad;
        ad += (int)((in * out + 1023) / 1024);
        a.ad_block[2 * l + 1] = ad;
        ad += (int)((out + 1023) / 1024);
    }
    a.tr_block[H + 1] = tr;
    a.ad_block[2 * (H + 1)] = ad;
    a.dw = (float *)take((size_t)off_w * 4);
    a.db = (float *)take((size_t)off_b * 4);
    return used;
}

hipError_t launch_train(const TrainArgs &a, hipStream_t s) {
    const int H = a.n_hidden;
    hipLaunchKernelGGL(train_transpose_kernel, dim3(a.tr_block[H + 1]), dim3(256), 0, s, a);
    hipLaunchKernelGGL(train_forward_kernel, dim3((a.B + ROWS - 1) / ROWS), dim3(512), 0, s, a);
    // one workgroup per CU holds two tiles: split the bins until every CU has one
    const int rb = (a.B + FT_ROWS - 1) / FT_ROWS, tiles = (a.D + FT_BINS - 1) / FT_BINS;
    const int split = std::max(1, std::min(tiles, (256 + rb - 1) / rb)), per = (tiles + split - 1) / split;
    hipLaunchKernelGGL(train_final_kernel, dim3(rb, (tiles + per - 1) / per), dim3(512), 0, s, a, per);
    hipLaunchKernelGGL(train_input_grad_kernel, dim3((a.B + XG_M - 1) / XG_M, W / XG_K), dim3(512), 0, s, a);
    if (H > 1) hipLaunchKernelGGL(train_backward_kernel, dim3(a.Bp / ROWS), dim3(512), 0, s, a);
    int blocks = 0;
    for (int l = 0; l <= H; ++l) blocks += a.wg_tiles[l] * a.wg_parts[l];
    hipLaunchKernelGGL(train_weight_grad_kernel, dim3(blocks), dim3(512), 0, s, a);
    hipLaunchKernelGGL(train_adam_kernel, dim3(a.ad_block[2 * (H + 1)]), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace supa
