// supa_judge.hip -- the surrogate's judge on the GPU: exact 1-D Wasserstein
// distances between two samples of equal size, column by column (the
// distance of the paper's section "Performance Analysis of Generative
// Models", here between the simulator's per-layer quantities and those of
// surrogate + fallback), and the occupied-cell counts of per-layer images.
//
// For two samples a, b of n values each, W1(a, b) = (1/n) sum_i |a_(i) - b_(i)|
// with a_(i), b_(i) the order statistics.  Each column of both samples is
// sorted by a stable least-significant-digit radix sort of its float keys,
// both samples' columns in the same launches: the keys column by column, then
// four passes of 8 bits (per pass: digit counts per tile of 8192 keys, then
// every key to its place, ranked within its tile in input order with wave
// ballots and gathered by digit in LDS, so that it leaves in runs); then one
// kernel sums
// |a_(i) - b_(i)| per column in double, by fixed blocks summed in order, so
// the result does not depend on scheduling.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "supa_device.hpp"

namespace supa {

constexpr int RS_THREADS = 512;
constexpr int RS_WAVES = RS_THREADS / 64;
constexpr int RS_ITEMS = 16;                     // keys per thread of a tile
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;   // keys per tile
constexpr int RS_DIGITS = 256;
// up to this many tiles per column a scatter sums the tiles' counts itself
// (n = 1M: 123 tiles, 30 KB read per workgroup from the L2); beyond, one
// kernel per pass turns the counts into starts first
constexpr int RS_SUM_TILES = 128;

// float -> unsigned key with the same order (negative values reversed)
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The columns to sort: of up to two row-major samples of `cols` columns each;
// column q of the sort is column q % cols of sample q / cols.  Key buffers
// hold column q at q * stride.
struct SortSrc {
    const float *x[2];
    int64_t ld[2];
    int cols;
    int64_t n, stride;
};

// keys column by column: 256 rows x up to 32 columns per block through LDS
// (rows are read as they lie, each column is written in runs of 256 keys)
__global__ void __launch_bounds__(256) rs_keys(SortSrc S, uint32_t *keys) {
    __shared__ uint32_t t[32][257];
    const int64_t r0 = (int64_t)blockIdx.x * 256;
    const int c0 = blockIdx.y * 32, nc = min(32, S.cols - c0);
    const int rows = (int)min<int64_t>(256, S.n - r0);
    const float *x = S.x[blockIdx.z] + r0 * S.ld[blockIdx.z] + c0;
    // i / nc by a multiplication (exact for the few bits of i; nc > 1), eight rows' worth in flight
    const uint32_t inv = nc > 1 ? 0xffffffffu / (uint32_t)nc + 1u : 0u;
    const int64_t ld = S.ld[blockIdx.z];
#pragma unroll 8
    for (int i = threadIdx.x; i < rows * nc; i += 256) {
        const int r = nc > 1 ? (int)__umulhi((uint32_t)i, inv) : i, c = i - r * nc;
        t[c][r] = float_key(x[r * ld + c]);
    }
    __syncthreads();
    uint32_t *out = keys + ((int64_t)blockIdx.z * S.cols + c0) * S.stride + r0;
    if ((int)threadIdx.x < rows)
        for (int c = 0; c < nc; ++c) out[c * S.stride + threadIdx.x] = t[c][threadIdx.x];
}

// digit counts of each tile: hist[(column * tiles + tile) * 256 + digit].
// Sixteen copies of the counters (a few digits take most keys of a float's
// top byte or of whole numbers), the copies a word apart in the banks.
__global__ void __launch_bounds__(RS_THREADS) rs_hist(const uint32_t *keys, int64_t n, int64_t stride, int shift,
                                                      uint32_t *hist) {
    __shared__ uint32_t h[16][RS_DIGITS + 1];
    for (int q = threadIdx.x; q < 16 * (RS_DIGITS + 1); q += RS_THREADS) (&h[0][0])[q] = 0u;
    __syncthreads();
    const uint32_t *k = keys + blockIdx.y * stride;
    const int64_t j0 = (int64_t)blockIdx.x * RS_TILE;
    uint32_t *mine = h[threadIdx.x & 15];
    uint4 v[RS_ITEMS / 4];
#pragma unroll
    for (int q = 0; q < RS_ITEMS / 4; ++q) {
        const int64_t j = j0 + 4 * (q * RS_THREADS + (int64_t)threadIdx.x);
        // (columns start on 256 bytes and are whole 16-byte groups long)
        if (j < n) v[q] = *(const uint4 *)(k + j);
    }
#pragma unroll
    for (int q = 0; q < RS_ITEMS / 4; ++q) {
        const int64_t j = j0 + 4 * (q * RS_THREADS + (int64_t)threadIdx.x);
        const uint32_t e[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j + u < n) atomicAdd(&mine[(e[u] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < RS_DIGITS) {
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += h[q][threadIdx.x];
        hist[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * RS_DIGITS + threadIdx.x] = t;
    }
}

// Exclusive sum over the first 256 threads of a block (all threads call).
__device__ __forceinline__ uint32_t rs_excl256(uint32_t v, uint32_t *part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (w < 4 && lane == 63) part[w] = incl;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) before += q < w ? part[q] : 0u;
    __syncthreads();
    return before + incl - v;
}

// many tiles: one block per column turns the counts into starts (in place)
__global__ void __launch_bounds__(256) rs_scan(uint32_t *hist, int nt) {
    __shared__ uint32_t part[4];
    uint32_t *h = hist + (int64_t)blockIdx.x * nt * RS_DIGITS + threadIdx.x;
    uint32_t tot = 0;
    for (int t = 0; t < nt; ++t) tot += h[(int64_t)t * RS_DIGITS];
    uint32_t run = rs_excl256(tot, part);
    for (int t = 0; t < nt; ++t) {
        const uint32_t v = h[(int64_t)t * RS_DIGITS];
        h[(int64_t)t * RS_DIGITS] = run;
        run += v;
    }
}

// Every key of a tile to its place: its digit's start in the column for this
// tile + its rank among the tile's keys of that digit, in input order.  Each
// wave ranks its 1,024 consecutive keys by itself (64 at a time, the lanes of
// equal digit from eight ballots, the counts so far in LDS words of the wave's
// own), so the tile takes a handful of barriers; the keys are gathered by
// digit in LDS and leave in runs of consecutive places.
__global__ void __launch_bounds__(RS_THREADS) rs_scatter(const uint32_t *keys, int64_t n, int64_t stride, int shift,
                                                         const uint32_t *hist, bool starts, uint32_t *out) {
    __shared__ uint32_t cnt[RS_WAVES][RS_DIGITS];
    __shared__ uint32_t stage[RS_TILE];
    __shared__ uint32_t first[RS_DIGITS], gbase[RS_DIGITS], part[4], half[2][RS_DIGITS];
    const int T = blockIdx.x, nt = gridDim.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t *k0 = keys + blockIdx.y * stride;
    const int64_t j0 = (int64_t)T * RS_TILE;
    const int m = (int)min<int64_t>(RS_TILE, n - j0);
    uint32_t k[RS_ITEMS];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = w * (64 * RS_ITEMS) + 64 * r + lane;
        k[r] = i < m ? k0[j0 + i] : 0u;
    }
    for (int q = lane; q < RS_DIGITS; q += 64) cnt[w][q] = 0u;
    // this tile's start of each digit: keys of smaller digits + keys of the
    // digit in earlier tiles (the tiles' counts summed by two halves)
    const uint32_t *hc = hist + (int64_t)blockIdx.y * nt * RS_DIGITS;
    uint32_t tot = 0, before = 0;
    {
        const int d = threadIdx.x & 255, hf = threadIdx.x >> 8;
        if (starts) {
            if (hf == 0) gbase[d] = hc[(int64_t)T * RS_DIGITS + d];
        } else {
            for (int t = hf; t < nt; t += 2) {
                const uint32_t v = hc[(int64_t)t * RS_DIGITS + d];
                tot += v;
                before += t < T ? v : 0u;
            }
            if (hf == 1) {
                half[0][d] = tot;
                half[1][d] = before;
            }
        }
    }
    __syncthreads();
    if (!starts) {
        if (threadIdx.x < RS_DIGITS) {
            tot += half[0][threadIdx.x];
            before += half[1][threadIdx.x];
        }
        const uint32_t ex = rs_excl256(threadIdx.x < RS_DIGITS ? tot : 0u, part);
        if (threadIdx.x < RS_DIGITS) gbase[threadIdx.x] = ex + before;
    }
    uint32_t rank[RS_ITEMS];
    uint32_t *mine = cnt[w];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const bool valid = w * (64 * RS_ITEMS) + 64 * r + lane < m;
        const uint32_t d = (k[r] >> shift) & 255u;
        // the lanes of equal digit: per bit, those whose bit is this lane's
        // (x: the bit in every position; 0x90 = a & ~(b ^ c): four vector
        // instructions per bit)
        const uint64_t in = __ballot(valid);
        uint32_t lo = (uint32_t)in, hi = (uint32_t)(in >> 32);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int x = (int)(d << (31 - b)) >> 31;
            const uint64_t q = __ballot(x < 0);
            lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)q, (uint32_t)x, 0x90);
            hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(q >> 32), (uint32_t)x, 0x90);
        }
        const uint32_t ahead = lanes_below(((uint64_t)hi << 32) | lo);
        const uint32_t prev = mine[d];
        rank[r] = prev + ahead;
        asm volatile("" ::: "memory");             // every lane has read before the first of a digit adds
        if (valid && ahead == 0u) mine[d] = prev + (uint32_t)(__popc(lo) + __popc(hi));
        asm volatile("" ::: "memory");
    }
    __syncthreads();
    // per digit: where each wave's keys start among the tile's, then the tile's digits in order
    uint32_t run = 0;
    if (threadIdx.x < RS_DIGITS) {
#pragma unroll
        for (int q = 0; q < RS_WAVES; ++q) {
            const uint32_t c = cnt[q][threadIdx.x];
            cnt[q][threadIdx.x] = run;
            run += c;
        }
    }
    const uint32_t ex = rs_excl256(threadIdx.x < RS_DIGITS ? run : 0u, part);
    if (threadIdx.x < RS_DIGITS) first[threadIdx.x] = ex;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const uint32_t d = (k[r] >> shift) & 255u;
        if (w * (64 * RS_ITEMS) + 64 * r + lane < m) stage[first[d] + cnt[w][d] + rank[r]] = k[r];
    }
    __syncthreads();
    uint32_t *o = out + blockIdx.y * stride;
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = r * RS_THREADS + (int)threadIdx.x;
        if (i < m) {
            const uint32_t v = stage[i], d = (v >> shift) & 255u;
            o[gbase[d] + ((uint32_t)i - first[d])] = v;
        }
    }
}

// per column: partial sums of |a_(i) - b_(i)| over fixed blocks of rows
constexpr int W1S_THREADS = 256;
constexpr int W1S_ROWS = W1S_THREADS * 16;

__global__ void __launch_bounds__(W1S_THREADS) w1_sorted_partials(const uint32_t *ka, const uint32_t *kb, int64_t n,
                                                                   int64_t stride, double *part) {
    __shared__ double sh[W1S_THREADS / 64];
    const int blk = blockIdx.x, c = blockIdx.y, nb = gridDim.x;
    double s = 0.0;
    for (int q = 0; q < 16; ++q) {
        const int64_t i = (int64_t)blk * W1S_ROWS + q * W1S_THREADS + threadIdx.x;
        if (i < n) {
            const float a = key_float(ka[c * stride + i]), b = key_float(kb[c * stride + i]);
            s += fabs((double)a - (double)b);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < W1S_THREADS / 64; ++q) t += sh[q];
        part[(int64_t)c * nb + blk] = t;
    }
}

// one wave per column: the block partials in order, divided by n
__global__ void w1_sorted_final(const double *part, int nb, int64_t n, int cols, double *w1) {
    const int c = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= cols) return;
    double s = 0.0;
    for (int b = lane; b < nb; b += 64) s += part[(int64_t)c * nb + b];
    // fixed butterfly: the same result on every run
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) w1[c] = s / (double)n;
}

// sorted values back to floats, column-major [cols][n]
__global__ void keys_to_floats(const uint32_t *k, int64_t n, int64_t stride, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[blockIdx.y * n + i] = key_float(k[blockIdx.y * stride + i]);
}

// cnt[r][l] = number of q < g with img[r][l * g + q] > thr
__global__ void occupied_counts(int64_t rows, int L, int g, const float *img, float thr, float *cnt) {
    const int64_t rl = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (rl >= rows * L) return;
    const float *p = img + rl * g;
    int m = 0;
    for (int q = lane; q < g; q += 64) m += p[q] > thr ? 1 : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m += __shfl_xor(m, off, 64);
    if (lane == 0) cnt[rl] = (float)m;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int64_t rs_tiles(int64_t n) { return (n + RS_TILE - 1) / RS_TILE; }
static int64_t rs_stride(int64_t n) { return (n + 63) / 64 * 64; }

// bytes of workspace for sorting `cols` columns of n keys (two key buffers
// and the digit counts)
size_t sort_work_bytes(int64_t n, int cols) {
    const size_t keys = (size_t)cols * rs_stride(n) * 4;
    const size_t hist = (size_t)cols * RS_DIGITS * rs_tiles(n) * 4;
    return 2 * ((keys + 255) & ~(size_t)255) + ((hist + 255) & ~(size_t)255);
}

// sorts the columns of `samples` (1 or 2) row-major matrices x[q] (ld[q]) of n
// rows and `cols` columns each; work: sort_work_bytes(n, samples * cols);
// returns the buffer holding the result, column q * cols + c at the returned
// stride
hipError_t launch_sort_columns(int samples, const float *const *x, const int64_t *ld, int64_t n, int cols, void *work,
                               uint32_t **sorted, int64_t *stride, hipStream_t s) {
    SortSrc S{};
    for (int q = 0; q < samples; ++q) {
        S.x[q] = x[q];
        S.ld[q] = ld[q];
    }
    S.cols = cols;
    S.n = n;
    S.stride = *stride = rs_stride(n);
    const size_t keys_b = (((size_t)samples * cols * S.stride * 4) + 255) & ~(size_t)255;
    uint32_t *src = (uint32_t *)work, *dst = (uint32_t *)((char *)work + keys_b);
    uint32_t *hist = (uint32_t *)((char *)work + 2 * keys_b);
    const int nt = (int)rs_tiles(n);
    const dim3 grid(nt, samples * cols);
    const bool starts = nt > RS_SUM_TILES;
    hipLaunchKernelGGL(rs_keys, dim3((unsigned)((n + 255) / 256), (cols + 31) / 32, samples), dim3(256), 0, s, S, src);
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 8 * pass;
        hipLaunchKernelGGL(rs_hist, grid, dim3(RS_THREADS), 0, s, src, n, S.stride, shift, hist);
        if (starts) hipLaunchKernelGGL(rs_scan, dim3(samples * cols), dim3(256), 0, s, hist, nt);
        hipLaunchKernelGGL(rs_scatter, grid, dim3(RS_THREADS), 0, s, src, n, S.stride, shift, hist, starts, dst);
        std::swap(src, dst);
    }
    *sorted = src;
    return hipGetLastError();
}

hipError_t launch_w1_sorted(const uint32_t *ka, const uint32_t *kb, int64_t n, int64_t stride, int cols, double *part,
                            double *w1, hipStream_t s) {
    const int nb = (int)((n + W1S_ROWS - 1) / W1S_ROWS);
    hipLaunchKernelGGL(w1_sorted_partials, dim3(nb, cols), dim3(W1S_THREADS), 0, s, ka, kb, n, stride, part);
    hipLaunchKernelGGL(w1_sorted_final, dim3((cols + 3) / 4), dim3(256), 0, s, part, nb, n, cols, w1);
    return hipGetLastError();
}

int64_t w1_sorted_partial_words(int64_t n, int cols) { return (int64_t)cols * ((n + W1S_ROWS - 1) / W1S_ROWS); }

hipError_t launch_keys_to_floats(const uint32_t *k, int64_t n, int64_t stride, int cols, float *out, hipStream_t s) {
    if (n <= 0 || cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(keys_to_floats, dim3((unsigned)((n + 255) / 256), cols), dim3(256), 0, s, k, n, stride, out);
    return hipGetLastError();
}

hipError_t launch_occupied_counts(int64_t rows, int L, int g, const float *img, float thr, float *cnt,
                                  hipStream_t s) {
    const int64_t groups = rows * L;
    if (groups <= 0) return hipSuccess;
    hipLaunchKernelGGL(occupied_counts, dim3((unsigned)((groups + 3) / 4)), dim3(256), 0, s, rows, L, g, img, thr,
                       cnt);
    return hipGetLastError();
}

}  // namespace supa
