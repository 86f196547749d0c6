// supa_order.hip -- the order in which the propagation kernel takes showers.
//
// A shower's expected cost grows linearly with its energy (about 4 E0 / e_cut
// particle-steps when nothing escapes: each split halves the energy on
// average and the cascade stops at the threshold).  Handing out the most
// expensive showers first leaves the cheap ones to fill the end of the
// launch, so no wave starts a long shower when the others are done (longest
// processing time first).  The order is a counting sort of the showers by
// a bucket of the exponent and leading bits of their fixed-point energy, descending: three kernels
// (histogram, scan of the buckets, scatter), or, up to ORDER_ONE showers, one
// block of the kernel that starts the call anyway.  The order within a bucket
// is arbitrary; results do not depend on the order at all.
#include <algorithm>

#include "supa_device.hpp"

namespace supa {

constexpr int ORDER_BUCKETS = 1024;           // 32 per octave of E_int
constexpr int ORDER_THREADS = 256;

// bucket 0 = most expensive
__device__ __forceinline__ int cost_bucket(float e0, float e_scale) {
    const float v = e0 * e_scale;
    if (!(v >= 1.0f)) return ORDER_BUCKETS - 1;           // tiny, zero, negative or NaN
    // 32 per octave, evenly in the mantissa: exponent and its five leading bits
    const int b = (int)(__float_as_uint(v) >> 18) - (127 << 5);
    return ORDER_BUCKETS - 1 - min(b, ORDER_BUCKETS - 1);
}

__global__ void __launch_bounds__(ORDER_THREADS) order_hist(const float *e0, int n, float e_scale,
                                                             uint32_t *hist) {
    __shared__ uint32_t h[ORDER_BUCKETS];
    for (int q = threadIdx.x; q < ORDER_BUCKETS; q += ORDER_THREADS) h[q] = 0u;
    __syncthreads();
    for (int i = blockIdx.x * ORDER_THREADS + threadIdx.x; i < n; i += gridDim.x * ORDER_THREADS)
        atomicAdd(&h[cost_bucket(e0[i], e_scale)], 1u);
    __syncthreads();
    for (int q = threadIdx.x; q < ORDER_BUCKETS; q += ORDER_THREADS)
        if (h[q]) atomicAdd(&hist[q], h[q]);
}

// one block: hist -> exclusive starts, in place
__global__ void __launch_bounds__(ORDER_BUCKETS) order_scan(uint32_t *hist) {
    __shared__ uint32_t s[ORDER_BUCKETS];
    const int t = threadIdx.x;
    s[t] = hist[t];
    __syncthreads();
    for (int off = 1; off < ORDER_BUCKETS; off <<= 1) {
        const uint32_t v = t >= off ? s[t - off] : 0u;
        __syncthreads();
        s[t] += v;
        __syncthreads();
    }
    hist[t] = s[t] - hist[t];
}

// Each block takes a contiguous run of ORDER_RUN showers: counts per bucket
// in LDS, one global reservation per bucket it holds (instead of one atomic
// per shower on a few hot counters), then LDS ranks within its reservation.
constexpr int ORDER_RUN = ORDER_THREADS * 16;

__global__ void __launch_bounds__(ORDER_THREADS) order_scatter(const float *e0, int n, float e_scale,
                                                                uint32_t *cursor, int32_t *order) {
    __shared__ uint32_t cnt[ORDER_BUCKETS], base[ORDER_BUCKETS];
    const int i0 = blockIdx.x * ORDER_RUN, i1 = min(n, i0 + ORDER_RUN);
    for (int q = threadIdx.x; q < ORDER_BUCKETS; q += ORDER_THREADS) cnt[q] = 0u;
    __syncthreads();
    for (int i = i0 + threadIdx.x; i < i1; i += ORDER_THREADS) atomicAdd(&cnt[cost_bucket(e0[i], e_scale)], 1u);
    __syncthreads();
    for (int q = threadIdx.x; q < ORDER_BUCKETS; q += ORDER_THREADS) {
        base[q] = cnt[q] ? atomicAdd(&cursor[q], cnt[q]) : 0u;
        cnt[q] = 0u;
    }
    __syncthreads();
    for (int i = i0 + threadIdx.x; i < i1; i += ORDER_THREADS) {
        const int b = cost_bucket(e0[i], e_scale);
        const uint32_t pos = base[b] + atomicAdd(&cnt[b], 1u);
        if (pos < (uint32_t)n) order[pos] = i;
    }
}

__global__ void order_clear(uint32_t *hist, unsigned long long *clk) {
    if (clk && blockIdx.x == 0 && threadIdx.x == 0) stamp(clk, CLK_CALL);
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < ORDER_BUCKETS) hist[q] = 0u;
}

// Rank in bucket b among the showers counted so far (h: the counts), with the
// bucket in the low ten bits.  One atomic for the lanes that share the first
// lane's bucket (all of them in a batch of one energy: 64 in turn on one
// counter).
__device__ __forceinline__ uint32_t order_rank(uint32_t *h, int b) {
    const int b0 = __builtin_amdgcn_readfirstlane(b);
    const uint64_t same = __ballot(b == b0);
    uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0));
    uint32_t base = 0u;
    if (b != b0 || rank == 0u) base = atomicAdd(&h[b], b != b0 ? 1u : (uint32_t)__builtin_popcountll(same));
    // (lane of rank 0: the first active one)
    rank = b == b0 ? rank + __builtin_amdgcn_readfirstlane(base) : base;
    return rank << 10 | (uint32_t)b;
}

// Start of a call: counters cleared, and the sub-batches' input / output
// blocks written from the launch's arguments (a copy from the host would be
// one more step of the call's chain).  With ORDER also the work order of its
// n <= ORDER_ONE showers, by the same block: their buckets and ranks in LDS.
template <bool ORDER>
__global__ void __launch_bounds__(ORDER ? 1024 : 256)
    supa_begin(unsigned long long *ctr, Cold *cold, ColdBlocks blocks, int n_cold, unsigned long long *clk,
               const float *e0, int n, float e_scale, int32_t *order) {
    __shared__ uint32_t h[ORDER ? ORDER_BUCKETS : 1], sums[16], place[ORDER ? ORDER_ONE : 1];
    const int t = (int)threadIdx.x;
    if (clk) {
        for (int q = t; q < CLK_WORDS; q += blockDim.x)
            if (q != CLK_CALL) clk[q] = 0ull;
        // (a work order by kernels of its own has stamped the start)
        if (t == 0 && (ORDER || !order)) stamp(clk, CLK_CALL);
    }
    for (int q = t; q < CTR_WORDS; q += blockDim.x) ctr[q] = 0ull;
    if (t < n_cold) cold[t] = blocks.c[t];
    if constexpr (ORDER) {
        static_assert(ORDER_BUCKETS == 1024 && ORDER_ONE <= 1 << 22, "one bucket per thread; rank and bucket in a word");
        h[t] = 0u;
        __syncthreads();
        // (loops, not straight code run once: its fetch took longer than the
        // work; the next round's eight loads in flight during a round)
        float e[8], en[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = t + 1024 * u < n ? e0[t + 1024 * u] : 0.0f;
        for (int i0 = t; i0 - t < n; i0 += 8 * 1024) {
#pragma unroll
            for (int u = 0; u < 8; ++u) en[u] = i0 + 1024 * (u + 8) < n ? e0[i0 + 1024 * (u + 8)] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 1024 * u;
                if (i >= n) continue;
                place[i] = order_rank(h, cost_bucket(e[u], e_scale));
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = en[u];
        }
        __syncthreads();
        // bucket counts -> starts
        const uint32_t v = h[t];
        uint32_t incl = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(incl, off, 64);
            if ((t & 63) >= off) incl += o;
        }
        if ((t & 63) == 63) sums[t >> 6] = incl;
        __syncthreads();
        uint32_t before = 0u;
#pragma unroll
        for (int w = 0; w < 16; ++w) before += w < (t >> 6) ? sums[w] : 0u;
        h[t] = before + incl - v;
        __syncthreads();
#pragma unroll 2
        for (int i = t; i < n; i += 1024) order[h[place[i] & 1023u] + (place[i] >> 10)] = i;
    }
    if (!clk) return;
    __syncthreads();
    if (t == 0) stamp(clk, CLK_BEGIN);
}

// order: null, or the array for the work order of n showers; written here when
// n <= ORDER_ONE, else already there.
hipError_t launch_begin(unsigned long long *ctr, Cold *cold, const Cold *h_cold, int n_cold, unsigned long long *clk,
                        const float *e0, int n, float e_scale, int32_t *order, hipStream_t s) {
    ColdBlocks blocks{};
    for (int j = 0; j < n_cold; ++j) blocks.c[j] = h_cold[j];
    if (order && n <= ORDER_ONE)
        hipLaunchKernelGGL(supa_begin<true>, dim3(1), dim3(1024), 0, s, ctr, cold, blocks, n_cold, clk, e0, n,
                           e_scale, order);
    else
        hipLaunchKernelGGL(supa_begin<false>, dim3(1), dim3(256), 0, s, ctr, cold, blocks, n_cold, clk, e0, n,
                           e_scale, order);
    return hipGetLastError();
}

int64_t order_scratch_words() { return ORDER_BUCKETS; }

// order[0..n) = a permutation of 0..n-1, most expensive first; hist: ORDER_BUCKETS words
hipError_t launch_cost_order(const float *e0, int n, float e_scale, uint32_t *hist, int32_t *order,
                             int n_cu, unsigned long long *clk, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int blocks = std::max(1, std::min((n + ORDER_THREADS - 1) / ORDER_THREADS, n_cu * 4));
    hipLaunchKernelGGL(order_clear, dim3(ORDER_BUCKETS / 256), dim3(256), 0, s, hist, clk);
    hipLaunchKernelGGL(order_hist, dim3(blocks), dim3(ORDER_THREADS), 0, s, e0, n, e_scale, hist);
    hipLaunchKernelGGL(order_scan, dim3(1), dim3(ORDER_BUCKETS), 0, s, hist);
    hipLaunchKernelGGL(order_scatter, dim3((n + ORDER_RUN - 1) / ORDER_RUN), dim3(ORDER_THREADS), 0, s, e0, n,
                       e_scale, hist, order);
    return hipGetLastError();
}

}  // namespace supa
