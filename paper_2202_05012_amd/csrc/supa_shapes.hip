// supa_shapes.hip -- evaluation kernels of include/supa_shapes.h: shower
// shape variables of hit point clouds (paper, section "Shower Shape
// Variables" and appendix "More shower shape variables") and the normalised
// Wasserstein-1 distance between histograms of two samples (section
// "Performance Analysis of Generative Models").
//
// Shape variables: one wave per shower (below), or, for large batches of few
// hits per shower, one lane per shower.  Such a lane streams its shower's segment
// of the hit arrays in aligned blocks of four hits (one 16-byte load per
// array), keeps the double-precision sums of the layer run it is in, and
// writes that layer's record when the run ends; lanes take showers from a
// queue (one atomic counter), so a lane that finishes a short shower goes on
// with the next one.  HBM traffic is one read of the hits and one write of
// the records.
//
// W1: per column, (1) count, shifted sums and min/max of both samples (per
// block partials, reduced in a fixed order), (2) one histogram per sample
// over the shared range (LDS histograms of a tile of columns, added into the
// global ones with integer atomics: exact), (3) one wave per column walks the
// cumulative counts.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>

#include "../../include/supa_shapes.h"

namespace {

constexpr int WAVE = 64;
constexpr int LV = SUPA_LAYER_VARS;
constexpr int SV = SUPA_SHOWER_VARS;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

struct ShapeArgs {
    int64_t n;
    int L;
    const int64_t *off;
    const int32_t *cnt;
    int cstride;
    int64_t len;  // entries of each hit array
    const float *x, *y, *e;
    const int32_t *layer;
    float *lv, *sv;
    int32_t *work;         // [0] showers in error, [1] next shower (queue)
    const int32_t *order;  // [n] showers in the order they are taken
};

// Sums of one layer run, in double precision.
struct Run {
    double sx, sxx, sy, syy, sr, se, see, sex, sexx, sey, seyy, ser;
    int n;
    float e1, e2;  // the two largest point energies
};

// sqrt of s >= 0: hardware reciprocal square root, then one Newton step on
// the residual (relative error about 1e-15), 0 for s = 0.
__device__ inline double sqrt_pos(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    const double r0 = s * y;
    const double e = __builtin_fma(-r0, r0, s);
    const double r = __builtin_fma(0.5 * y, e, r0);
    return s > 0.0 ? r : 0.0;
}

// 1 / v for v > 0: hardware reciprocal and two Newton steps (about 1 ulp).
__device__ inline double recip(double v) {
    double y = __builtin_amdgcn_rcp(v);
    y = __builtin_fma(__builtin_fma(-v, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-v, y, 1.0), y, y);
    return y;
}

__device__ inline void run_clear(Run &a) {
    a.sx = a.sxx = a.sy = a.syy = a.sr = a.se = a.see = 0.0;
    a.sex = a.sexx = a.sey = a.seyy = a.ser = 0.0;
    a.n = 0;
    a.e1 = a.e2 = -__builtin_inff();
}

// Adds one point when `take` (otherwise adds zeros: no branch).
__device__ inline void run_add(Run &a, float xf, float yf, float ef, bool take) {
    const double x = take ? xf : 0.0f, y = take ? yf : 0.0f, e = take ? ef : 0.0f;
    const double xx = x * x, yy = y * y;
    const double r = sqrt_pos(xx + yy);
    const double ex = e * x, ey = e * y;
    a.sx += x;
    a.sxx += xx;
    a.sy += y;
    a.syy += yy;
    a.sr += r;
    a.se += e;
    a.see = __builtin_fma(e, e, a.see);
    a.sex += ex;
    a.sexx = __builtin_fma(ex, x, a.sexx);
    a.sey += ey;
    a.seyy = __builtin_fma(ey, y, a.seyy);
    a.ser = __builtin_fma(e, r, a.ser);
    a.n += take ? 1 : 0;
    const float et = take ? ef : -__builtin_inff();  // running two largest
    a.e2 = __builtin_fmaxf(a.e2, __builtin_fminf(a.e1, et));
    a.e1 = __builtin_fmaxf(a.e1, et);
}

__device__ inline float dev_of(double m1, double m2) {
    const double v = __builtin_fma(-m1, m1, m2);
    return __builtin_amdgcn_sqrtf((float)(v > 0.0 ? v : 0.0));
}

// Writes every field of a layer record except FRACTION.  Sum of E r^2 is
// sum E x^2 + sum E y^2; sum r^2 is sum x^2 + sum y^2.
__device__ inline void write_layer(float *rec, const Run &a) {
    const float nan = __builtin_nanf("");
    const double in = recip((double)a.n);
    const double mx = a.sx * in, my = a.sy * in, mr = a.sr * in, me = a.se * in;
    f32x2 *r2 = (f32x2 *)rec;
    r2[0] = f32x2{(float)a.n, (float)mx};
    r2[1] = f32x2{(float)my, (float)mr};
    r2[2] = f32x2{(float)me, dev_of(mx, a.sxx * in)};
    r2[3] = f32x2{dev_of(my, a.syy * in), dev_of(mr, (a.sxx + a.syy) * in)};
    r2[4] = f32x2{dev_of(me, a.see * in), (float)a.se};
    if (a.se > 0.0) {
        const double ie = recip(a.se);
        const double cx = a.sex * ie, cy = a.sey * ie, cr = a.ser * ie;
        r2[5] = f32x2{(float)cx, (float)cy};
        r2[6] = f32x2{(float)cr, dev_of(cx, a.sexx * ie)};
        r2[7] = f32x2{dev_of(cy, a.seyy * ie), dev_of(cr, (a.sexx + a.seyy) * ie)};
    } else {
        r2[5] = f32x2{nan, nan};
        r2[6] = f32x2{nan, nan};
        r2[7] = f32x2{nan, nan};
    }
    const double e1 = a.e1, e2 = a.n > 1 ? (double)a.e2 : 0.0;  // E[2] = 0 for one point
    rec[SUPA_LV_ENERGY_RATIO] = (e1 + e2 > 0.0) ? (float)((e1 - e2) / (e1 + e2)) : nan;
}

__device__ inline void write_empty_layer(float *rec) {
    const float nan = __builtin_nanf("");
    f32x2 *r2 = (f32x2 *)rec;
    r2[0] = f32x2{0.0f, nan};
    r2[1] = f32x2{nan, nan};
    r2[2] = f32x2{nan, nan};
    r2[3] = f32x2{nan, nan};
    r2[4] = f32x2{nan, 0.0f};
    r2[5] = f32x2{nan, nan};
    r2[6] = f32x2{nan, nan};
    r2[7] = f32x2{nan, nan};
    rec[SUPA_LV_ENERGY_RATIO] = nan;
}

// work: [0] showers in error, [1] queue, [2] whether one wave takes a shower
// (else one lane), [3] unused, then the global order's bucket sizes and cursors
// (ORDER_BUCKETS each), then the order [n].
constexpr int ORDER_BUCKETS = 1024;
constexpr int WORK_HEAD = 4 + 2 * ORDER_BUCKETS;

// Batches of more than WAVE_CALLS showers per CU are summed by one wave per
// shower when a shower has MIN_WAVE_HITS hits on average, by one lane per
// shower otherwise (20 layers, 100,000 showers, us by wave / by lane: 941 hits
// 545 / 800, 94 hits 184 / 220, 47 hits 162 / 141; a million showers of 3 hits
// 1130 / 285: a wave's fixed work per shower is then all there is).  Smaller
// batches always by wave: one lane per shower leaves the chip idle (3,000
// showers of 942 hits 34 / 549, of 47 hits 16 / 86; 10,000 of 9 hits 23 / 33).
// The average is taken from the ends of the first and last segment, on the
// device: the arrays may be longer than what is in use.  It decides nothing
// but the speed.
constexpr int WAVE_CALLS = 64;
constexpr int MIN_WAVE_HITS = 64;

__global__ void shapes_clear(int32_t *work, int64_t n, const int64_t *off, const int32_t *cnt, int cstride,
                             int always) {
    for (int i = threadIdx.x; i < WORK_HEAD; i += blockDim.x) {
        int v = 0;
        if (i == 2 && n > 0)
            v = always || off[n - 1] + cnt[(size_t)(n - 1) * cstride] - off[0] >= MIN_WAVE_HITS * n ? 1 : 0;
        work[i] = v;
    }
}

// Order in which the lanes take showers: longest first, within windows of
// consecutive showers.  A wave's lanes then carry showers of similar length,
// so fewer lanes idle while the longest one finishes.  When every shower is
// in flight at once (one per lane) the window is the whole batch, sorted by
// two kernels (global bucket sizes, then each block reserves its range of
// every bucket with one atomic); otherwise windows of ORDER_WIN keep the
// showers in flight close together in memory, each sorted by one workgroup,
// and hold 63 waves' worth of showers so that the first (longest) wave of
// consecutive windows falls on different XCDs.  Both are counting sorts into
// 1024 buckets of the hit count on a log scale (32 per octave); the order
// within a bucket is whatever the atomics give, which changes no result (each
// shower is summed by one lane in its own hit order).
constexpr int ORDER_WIN = 63 * WAVE;
constexpr int ORDER_THREADS = 1024;

__device__ inline int count_bucket(int32_t c) {  // 0..1023, non-decreasing in c
    const uint32_t v = (c > 0 ? (uint32_t)c : 0u) + 1u;
    const int e = 31 - __builtin_clz(v);
    const uint32_t m = e >= 5 ? (v >> (e - 5)) & 31u : (v << (5 - e)) & 31u;
    return e * 32 + (int)m;
}

// dst[b] = sum of src[0 .. b) over the ORDER_BUCKETS buckets, by one wave
// (lane t < 64 of the caller); dst may be src.
__device__ inline void bucket_starts(const uint32_t *src, uint32_t *dst, int t) {
    constexpr int Q = ORDER_BUCKETS / WAVE;
    uint32_t v[Q], sum = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        v[q] = src[t * Q + q];
        sum += v[q];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d);
        if (t >= d) inc += o;
    }
    uint32_t run = inc - sum;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        dst[t * Q + q] = run;
        run += v[q];
    }
}

__global__ void __launch_bounds__(ORDER_THREADS)
    shapes_order(int64_t n, int64_t win, const int32_t *cnt, int cstride, const int32_t *by_wave,
                 int32_t *order) {
    __shared__ uint32_t hist[ORDER_BUCKETS];
    if (*by_wave) return;
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * win;
    const int64_t m = n - base < win ? n - base : win;
    for (int i = t; i < ORDER_BUCKETS; i += ORDER_THREADS) hist[i] = 0;
    __syncthreads();
    for (int64_t i = t; i < m; i += ORDER_THREADS)
        atomicAdd(&hist[ORDER_BUCKETS - 1 - count_bucket(cnt[(size_t)(base + i) * cstride])], 1u);
    __syncthreads();
    if (t < WAVE) bucket_starts(hist, hist, t);
    __syncthreads();
    // hist now holds each bucket's next free position
    for (int64_t i = t; i < m; i += ORDER_THREADS) {
        const int b = ORDER_BUCKETS - 1 - count_bucket(cnt[(size_t)(base + i) * cstride]);
        order[base + atomicAdd(&hist[b], 1u)] = (int32_t)(base + i);
    }
}

// Whole-batch order, pass 1: sizes of the buckets (gsize, zeroed before).
constexpr int ORDER_CHUNK = 4 * ORDER_THREADS;  // showers per block of the two passes

__global__ void __launch_bounds__(ORDER_THREADS)
    shapes_order_sizes(int64_t n, const int32_t *cnt, int cstride, const int32_t *by_wave, uint32_t *gsize) {
    __shared__ uint32_t hist[ORDER_BUCKETS];
    if (*by_wave) return;
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * ORDER_CHUNK;
    const int64_t m = n - base < ORDER_CHUNK ? n - base : ORDER_CHUNK;
    for (int i = t; i < ORDER_BUCKETS; i += ORDER_THREADS) hist[i] = 0;
    __syncthreads();
    for (int64_t i = t; i < m; i += ORDER_THREADS)
        atomicAdd(&hist[ORDER_BUCKETS - 1 - count_bucket(cnt[(size_t)(base + i) * cstride])], 1u);
    __syncthreads();
    for (int i = t; i < ORDER_BUCKETS; i += ORDER_THREADS)
        if (hist[i]) atomicAdd(&gsize[i], hist[i]);
}

// Pass 2: each block reserves its range of every bucket (gcur, zeroed
// before) and places its showers.
__global__ void __launch_bounds__(ORDER_THREADS)
    shapes_order_place(int64_t n, const int32_t *cnt, int cstride, const int32_t *by_wave,
                       const uint32_t *gsize, uint32_t *gcur, int32_t *order) {
    __shared__ uint32_t hist[ORDER_BUCKETS], start[ORDER_BUCKETS];
    if (*by_wave) return;
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * ORDER_CHUNK;
    const int64_t m = n - base < ORDER_CHUNK ? n - base : ORDER_CHUNK;
    for (int i = t; i < ORDER_BUCKETS; i += ORDER_THREADS) {
        hist[i] = 0;
        start[i] = gsize[i];
    }
    __syncthreads();
    if (t < WAVE) bucket_starts(start, start, t);
    int bk[4];
    uint32_t rank[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = t + (int64_t)u * ORDER_THREADS;
        bk[u] = i < m ? ORDER_BUCKETS - 1 - count_bucket(cnt[(size_t)(base + i) * cstride]) : -1;
        rank[u] = bk[u] >= 0 ? atomicAdd(&hist[bk[u]], 1u) : 0u;
    }
    __syncthreads();
    for (int i = t; i < ORDER_BUCKETS; i += ORDER_THREADS)
        if (hist[i]) start[i] += atomicAdd(&gcur[i], hist[i]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (bk[u] >= 0) order[start[bk[u]] + rank[u]] = (int32_t)(base + t + (int64_t)u * ORDER_THREADS);
}

// Records of finished layer runs wait in a per-wave LDS ring until 64 are
// ready, then the wave computes and writes 64 records at once (one per lane):
// the division and square roots of a record run with every lane busy instead
// of once per lane whose run happens to end.
constexpr int QCAP = 128;      // ring entries (a step adds at most 64)
constexpr int BLK = 32;        // hits per lane per step: one 128-byte line per array

struct Ring {
    double d[12][QCAP];
    int n[QCAP], s[QCAP], l[QCAP];
    float e1[QCAP], e2[QCAP];
};

// Adds the runs of the lanes with `cond` to the ring at t (wave-uniform).
__device__ inline void ring_put(Ring &q, int &t, bool cond, int s, int l, const Run &a) {
    const uint64_t m = __ballot(cond);
    if (cond) {
        const int slot = (t + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))) &
                         (QCAP - 1);
        q.d[0][slot] = a.sx;
        q.d[1][slot] = a.sxx;
        q.d[2][slot] = a.sy;
        q.d[3][slot] = a.syy;
        q.d[4][slot] = a.sr;
        q.d[5][slot] = a.se;
        q.d[6][slot] = a.see;
        q.d[7][slot] = a.sex;
        q.d[8][slot] = a.sexx;
        q.d[9][slot] = a.sey;
        q.d[10][slot] = a.seyy;
        q.d[11][slot] = a.ser;
        q.n[slot] = a.n;
        q.s[slot] = s;
        q.l[slot] = l;
        q.e1[slot] = a.e1;
        q.e2[slot] = a.e2;
    }
    t += __builtin_popcountll(m);
}

// Writes up to `most` (<= 64) records from the ring head h (wave-uniform call).
__device__ inline void ring_drain(Ring &q, int &h, int t, int most, float *lv, int L) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int k = (t - h) < most ? (t - h) : most;
    const int lane = threadIdx.x;
    if (lane < k) {
        const int slot = (h + lane) & (QCAP - 1);
        Run a;
        a.sx = q.d[0][slot];
        a.sxx = q.d[1][slot];
        a.sy = q.d[2][slot];
        a.syy = q.d[3][slot];
        a.sr = q.d[4][slot];
        a.se = q.d[5][slot];
        a.see = q.d[6][slot];
        a.sex = q.d[7][slot];
        a.sexx = q.d[8][slot];
        a.sey = q.d[9][slot];
        a.seyy = q.d[10][slot];
        a.ser = q.d[11][slot];
        a.n = q.n[slot];
        a.e1 = q.e1[slot];
        a.e2 = q.e2[slot];
        write_layer(lv + ((size_t)q.s[slot] * L + q.l[slot]) * LV, a);
    }
    h += k;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per workgroup; static LDS: the ring; dynamic LDS: float [L][64],
// the layer energies of each lane's current shower (for the fractions,
// written once E_tot is known).  Every cross-lane step (ring, drain, exit)
// runs in wave-uniform control flow.
__global__ void __launch_bounds__(WAVE) shapes_kernel(ShapeArgs A) {
    __shared__ Ring q;
    extern __shared__ float ef[];
    if (A.work[2]) return;                // a wave each
    const int lane = threadIdx.x;
    const int L = A.L;
    const float nan = __builtin_nanf("");
    uint32_t *queue = (uint32_t *)A.work + 1;

    int h = 0, t = 0;  // ring head and tail (wave-uniform)
    bool active = true;
    int64_t s = -1, pos = 0, end = 0;
    int cur = -1, depth = -1;
    bool bad = false;
    uint64_t seen = 0;
    double etot = 0.0, ld = 0.0, ld2 = 0.0;
    Run acc;
    run_clear(acc);

    for (;;) {
        // --- lanes whose shower is done: last run, empty layers, totals
        const bool closing = active && s >= 0 && pos >= end;
        ring_put(q, t, closing && !bad && cur >= 0, (int)s, cur, acc);
        if (closing && !bad) {
            float *base = A.lv + (size_t)s * L * LV;
            if (cur >= 0) {
                ef[cur * WAVE + lane] = (float)acc.se;
                etot += acc.se;
                ld += (double)cur * acc.se;
                ld2 += (double)cur * (double)cur * acc.se;
                if (acc.se > 0.0 && cur > depth) depth = cur;
            }
            const double it = etot > 0.0 ? recip(etot) : 0.0;
            for (int l = 0; l < L; ++l) {
                float *rec = base + (size_t)l * LV;
                if (!((seen >> l) & 1)) write_empty_layer(rec);
                rec[SUPA_LV_FRACTION] = etot > 0.0 ? (float)((double)ef[l * WAVE + lane] * it) : nan;
            }
            float *sv = A.sv + (size_t)s * SV;
            const double sd = ld * it;
            sv[SUPA_SV_E_TOT] = (float)etot;
            sv[SUPA_SV_DEPTH] = (float)depth;
            sv[SUPA_SV_L_D] = (float)ld;
            sv[SUPA_SV_S_D] = etot > 0.0 ? (float)sd : nan;
            sv[SUPA_SV_S_D_WIDTH] = etot > 0.0 ? dev_of(sd, ld2 * it) : nan;
        }
        // a shower in error: its earlier runs leave the ring first, then NaN
        if (__ballot(closing && bad)) {
            while (t - h > 0) ring_drain(q, h, t, WAVE, A.lv, L);
            if (closing && bad) {
                float *base = A.lv + (size_t)s * L * LV;
                for (int f = 0; f < L * LV; ++f) base[f] = nan;
                for (int f = 0; f < SV; ++f) A.sv[(size_t)s * SV + f] = nan;
                atomicAdd(A.work, 1);
            }
        }
        if (t - h >= WAVE) ring_drain(q, h, t, WAVE, A.lv, L);
        // --- next shower from the queue
        if (active && pos >= end) {
            const uint32_t next = atomicAdd(queue, 1u);
            if ((int64_t)next >= A.n) {
                active = false;
            } else {
                s = A.order[next];
                pos = A.off[s];
                end = pos + A.cnt[(size_t)s * A.cstride];
                // a segment reaching outside the arrays is the caller's error;
                // never read outside them
                pos = pos < 0 ? 0 : (pos > A.len ? A.len : pos);
                end = end < pos ? pos : (end > A.len ? A.len : end);
                cur = -1;
                depth = -1;
                bad = false;
                seen = 0;
                etot = ld = ld2 = 0.0;
                run_clear(acc);
                for (int l = 0; l < L; ++l) ef[l * WAVE + lane] = 0.0f;
            }
        }
        if (!__ballot(active)) break;

        // --- one aligned block of BLK hits per lane, clipped to [pos, end)
        const bool work = active && pos < end;
        const int64_t b0 = pos & ~(int64_t)(BLK - 1);
        float vx[BLK], vy[BLK], ve[BLK];
        int vl[BLK];
        // whole aligned blocks are read with 16-byte loads whenever they lie
        // inside the arrays (entries outside [pos, end) are then dropped);
        // only the arrays' last partial block is read entry by entry
        if (work && b0 + BLK <= A.len) {
#pragma unroll
            for (int k = 0; k < BLK; k += 4) {
                const f32x4 a = *(const f32x4 *)(A.x + b0 + k);
                const f32x4 b = *(const f32x4 *)(A.y + b0 + k);
                const f32x4 c = *(const f32x4 *)(A.e + b0 + k);
                const i32x4 d = *(const i32x4 *)(A.layer + b0 + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = b0 + k + j;
                    vx[k + j] = a[j];
                    vy[k + j] = b[j];
                    ve[k + j] = c[j];
                    vl[k + j] = (i >= pos && i < end) ? d[j] : -1;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < BLK; ++j) {
                const int64_t i = b0 + j;
                const bool in = work && i >= pos && i < end;
                vx[j] = in ? A.x[i] : 0.0f;
                vy[j] = in ? A.y[i] : 0.0f;
                ve[j] = in ? A.e[i] : 0.0f;
                vl[j] = in ? A.layer[i] : -1;
            }
        }
        // bit j: a new run starts at hit j of this lane's block; their OR
        // over the wave decides (uniformly) which steps need the switch code
        uint32_t msk = 0;
        {
            int p = cur;
#pragma unroll
            for (int j = 0; j < BLK; ++j) {
                const int l = vl[j];
                msk |= (uint32_t)(l >= 0 && l != p) << j;
                p = l >= 0 ? l : p;
            }
            if (bad) msk = 0;
        }
        uint32_t any = msk;
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1) any |= (uint32_t)__shfl_xor((int)any, d);
        any = __builtin_amdgcn_readfirstlane(any);
#pragma unroll
        for (int j = 0; j < BLK; ++j) {
            const int l = vl[j];
            if ((any >> j) & 1) {
                const bool sw = ((msk >> j) & 1) && !bad;  // a new run starts here
                ring_put(q, t, sw && cur >= 0, (int)s, cur, acc);
                if (sw) {
                    if (cur >= 0) {
                        ef[cur * WAVE + lane] = (float)acc.se;
                        etot += acc.se;
                        ld += (double)cur * acc.se;
                        ld2 += (double)cur * (double)cur * acc.se;
                        if (acc.se > 0.0 && cur > depth) depth = cur;
                    }
                    run_clear(acc);
                    if (l >= L || ((seen >> l) & 1)) {
                        bad = true;
                        cur = -1;
                    } else {
                        seen |= 1ull << l;
                        cur = l;
                    }
                }
                if (t - h >= WAVE) ring_drain(q, h, t, WAVE, A.lv, L);
            }
            run_add(acc, vx[j], vy[j], ve[j], l >= 0 && !bad);
        }
        if (work) pos = bad ? end : (b0 + BLK < end ? b0 + BLK : end);
    }
    while (t - h > 0) ring_drain(q, h, t, WAVE, A.lv, L);
}

// ---------------------------------------------------------------------------
// One wave per shower.  The segment is read once, coalesced, 256 hits per step
// (16 bytes per lane and array), hits of layer -1 left out, into an LDS tile
// of up to SHW_TILE hits.  The tile's layer runs are cut into fragments of
// about equal length, at most one per lane and never across a run, so that
// every lane sums hits of one layer only (no test for a change of layer in the
// loop) and lanes are evenly loaded.  The fragments' sums are then added run
// by run in order: sixteen lanes walk sixteen fragments, one lane per kind of
// sum, and the lane that owns the run (run r of the shower: lane r; more than
// 64 runs repeat a layer) takes at most four partial sums.  Every sum has a
// fixed order: results do not depend on the batch or on timing.
//
// Bound by vector instructions (2,000 per shower of 941 hits in 20 layers,
// half of them the sums; 80% of the issue slots), next to 1.5 GB of hits:
// 100,000 such showers 545 us (one lane per shower: 800 us, until the lane
// with the longest shower was done), 3,000 34 us (549).  768 hits per tile:
// 10 KB of LDS, four waves per SIMD (1,024: three waves, 570 us; 512: more
// tiles per shower, 690 us).  Reading the next tile's or shower's first step
// ahead cost more registers than it hid (605 us).  At most 128 workgroups per
// CU, striding over the showers: one shower each would be 15 us
// faster there, but leaving again 100,000 workgroups for nothing when the lanes
// do the work costs more.
// ---------------------------------------------------------------------------
constexpr int SHW_TILE = 768;
constexpr int SHW_STEP = 4 * WAVE;        // hits read per step
constexpr int SHW_SUMS = 12;
constexpr int SHW_LD = WAVE + 2;          // row of 16-byte aligned fragment sums, rows on different banks

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

struct WaveTile {
    union {
        float hit[3][SHW_TILE + 4];       // x, y, e; entry SHW_TILE is a point of zeros
        struct {                          // the fragments' sums (once the hits are read)
            double d[SHW_SUMS][SHW_LD];
            f32x2 top[WAVE];              // two largest energies
        } f;
    };
    int pos[WAVE + 1], lay[WAVE], flag[WAVE];
};

// orders LDS accesses of a wave's lanes among each other
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Data of another lane by DPP, 0 where there is none: shifts by 1, 2, 4, 8
// within rows of sixteen lanes, then row ends broadcast to the rows above.
template <int K>
__device__ inline int scan_src(int v) {
    if constexpr (K < 4) return __builtin_amdgcn_update_dpp(0, v, 0x110 + (1 << K), 0xf, 0xf, true);
    if constexpr (K == 4) return __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    return __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
}

template <int K>
__device__ inline double scan_src(double v) {
    return __hiloint2double(scan_src<K>(__double2hiint(v)), scan_src<K>(__double2loint(v)));
}

// sum over lanes 0 .. lane (lane 63: the wave's)
template <typename T>
__device__ inline T scan_sum(T v) {
    v += scan_src<0>(v);
    v += scan_src<1>(v);
    v += scan_src<2>(v);
    v += scan_src<3>(v);
    v += scan_src<4>(v);
    v += scan_src<5>(v);
    return v;
}

// maximum over the wave of v >= 0
__device__ inline int wave_max(int v) {
    v = max(v, scan_src<0>(v));
    v = max(v, scan_src<1>(v));
    v = max(v, scan_src<2>(v));
    v = max(v, scan_src<3>(v));
    v = max(v, scan_src<4>(v));
    v = max(v, scan_src<5>(v));
    return __builtin_amdgcn_readlane(v, WAVE - 1);
}

__device__ inline double wave_sum(double v) {
    v = scan_sum(v);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), WAVE - 1),
                            __builtin_amdgcn_readlane(__double2loint(v), WAVE - 1));
}

struct Four {
    f32x4 x, y, e;
    i32x4 l;
};

// This lane's four hits of the step at base: hits 4 lane .. 4 lane + 3 of the
// `here` hits there (others: any values).  Whole steps inside the arrays are
// read 16 bytes at a time (hits of the next segment included), only the
// arrays' end hit by hit.
__device__ inline Four read_four(const ShapeArgs &A, int64_t base, int here, int lane) {
    Four h;
    const float *x = A.x + base, *y = A.y + base, *e = A.e + base;
    const int32_t *layer = A.layer + base;
    const unsigned i = 4u * (unsigned)lane;
    if (base + SHW_STEP <= A.len) {
        h.x = *(const f32x4u *)(x + i);
        h.y = *(const f32x4u *)(y + i);
        h.e = *(const f32x4u *)(e + i);
        h.l = *(const i32x4u *)(layer + i);
    } else {
#pragma unroll
        for (unsigned u = 0; u < 4; ++u) {
            const unsigned j = (int)(i + u) < here ? i + u : 0u;
            h.x[u] = x[j];
            h.y[u] = y[j];
            h.e[u] = e[j];
            h.l[u] = layer[j];
        }
    }
    return h;
}

// Lanes whose hit u of a step is one of its `here` hits.
__device__ inline uint64_t lanes_with(int here, int u) {
    const int k = (here - u + 3) >> 2;
    return k <= 0 ? 0ull : k >= WAVE ? ~0ull : (1ull << k) - 1ull;
}

// The two largest of an earlier and a later part's.  As when the hits are taken
// one by one (run_add): at an energy that is not a number the largest so far
// becomes the second largest, too.
__device__ inline void add_top(float &e1, float &e2, float o1, float o2, bool later_nan) {
    e2 = __builtin_fmaxf(__builtin_fmaxf(e2, o2), __builtin_fminf(e1, o1));
    e2 = later_nan ? __builtin_fmaxf(e2, e1) : e2;
    e1 = __builtin_fmaxf(e1, o1);
}

// Adds lane - D's pair when it lies in the same row of sixteen and belongs to
// the same run; nan: whether an energy of this lane's part is not a number.
template <int D>
__device__ inline void seg_top(float &e1, float &e2, int &nan, int run) {
    const int r = __builtin_amdgcn_update_dpp(-1, run, 0x110 + D, 0xf, 0xf, false);
    const float o1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e1), 0x110 + D, 0xf, 0xf, false));
    const float o2 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e2), 0x110 + D, 0xf, 0xf, false));
    const int on = __builtin_amdgcn_update_dpp(0, nan, 0x110 + D, 0xf, 0xf, false);
    float s1 = o1, s2 = o2;
    add_top(s1, s2, e1, e2, nan != 0);
    e1 = r == run ? s1 : e1;
    e2 = r == run ? s2 : e2;
    nan |= r == run ? on : 0;
}

// Shape variables of shower s.
__device__ void wave_shower(const ShapeArgs &A, WaveTile &T, int64_t s, int lane) {
    const int L = A.L;
    const float nan = __builtin_nanf("");
    // a segment reaching outside the arrays is the caller's error; never read
    // outside them
    int64_t base = A.off[s];
    int64_t end = base + A.cnt[(size_t)s * A.cstride];
    base = base < 0 ? 0 : (base > A.len ? A.len : base);
    end = end < base ? base : (end > A.len ? A.len : end);

    Run own;                              // run `lane` of the shower
    run_clear(own);
    int R = 0, prev = -1;                 // runs so far, the layer of the last hit
    while (base < end && R <= WAVE) {
        const int raw = (int)(end - base < SHW_TILE ? end - base : SHW_TILE);
        const int rb = R > 0 ? R - 1 : 0; // the run that may go on in this tile
        const bool goes_on = R > 0;
        int m = 0;                        // hits in the tile
        if (lane < 3) T.hit[lane][SHW_TILE] = 0.0f;
        for (int b = 0; b < raw; b += SHW_STEP) {
            const int here = raw - b < SHW_STEP ? raw - b : SHW_STEP;
            Four h = read_four(A, base + b, here, lane);
            uint64_t in[4], out = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                in[u] = lanes_with(here, u);
                out |= __ballot(h.l[u] < 0) & in[u];
            }
            int p[4], at = m + 4 * lane;  // the layer before each hit, the first hit's place
            uint64_t st[4];               // lanes whose hit u starts a run
            if (!out && !(m & 3)) {       // every hit is taken
                p[0] = __builtin_amdgcn_update_dpp(prev, h.l[3], 0x138, 0xf, 0xf, false);   // lane - 1's last
#pragma unroll
                for (int u = 1; u < 4; ++u) p[u] = h.l[u - 1];
                *(f32x4 *)&T.hit[0][at] = h.x;
                *(f32x4 *)&T.hit[1][at] = h.y;
                *(f32x4 *)&T.hit[2][at] = h.e;
                m += here;
                // (a partial step is the segment's last)
                prev = __builtin_amdgcn_readlane(h.l[3], WAVE - 1);
#pragma unroll
                for (int u = 0; u < 4; ++u) st[u] = __ballot(h.l[u] != p[u]) & in[u];
            } else {
                int last = -1;            // the lane's last layer
                at = m;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    h.l[u] = 4 * lane + u < here ? h.l[u] : -1;
                    last = h.l[u] >= 0 ? h.l[u] : last;
                    const uint64_t vm = __ballot(h.l[u] >= 0);
                    at += lanes_below(vm);
                    m += (int)__builtin_popcountll(vm);
                }
                const uint64_t hm = __ballot(last >= 0);
                const uint64_t below = hm & ((1ull << lane) - 1ull);
                const int before = __shfl(last, below ? 63 - __builtin_clzll(below) : lane);
                int q = below ? before : prev, a = at;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    p[u] = q;
                    if (h.l[u] >= 0) {
                        q = h.l[u];
                        T.hit[0][a] = h.x[u];
                        T.hit[1][a] = h.y[u];
                        T.hit[2][a] = h.e[u];
                        ++a;
                    }
                    st[u] = __ballot(h.l[u] >= 0 && h.l[u] != p[u]);
                }
                if (hm) prev = __builtin_amdgcn_readlane(last, 63 - __builtin_clzll(hm));
            }
            if (st[0] | st[1] | st[2] | st[3]) {
                int r = R;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    r += lanes_below(st[u]);
                    R += (int)__builtin_popcountll(st[u]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool start = (st[u] >> lane) & 1;
                    if (start && r < WAVE) {
                        T.pos[r] = at;
                        T.lay[r] = h.l[u];
                    }
                    r += start ? 1 : 0;
                    at += h.l[u] >= 0 ? 1 : 0;
                }
            }
        }
        base += raw;
        if (R > WAVE) break;              // a layer comes twice
        if (m == 0) continue;
        wave_sync();
        // this lane's run in the tile: [p0, p1)
        const bool here = lane >= rb && lane < R;
        const int p0 = !here ? 0 : (goes_on && lane == rb) ? 0 : T.pos[lane];
        const int p1 = !here ? 0 : lane + 1 < R ? T.pos[lane + 1] : m;
        const int nr = p1 - p0;
        // fragment length F: the runs' last fragments are half full on average
        // (try that first); m / (64 - runs) always fits, and so does the
        // longest run.  nr + F <= 2 SHW_TILE: the quotients are exact.
        const int runs = R - rb, longest = wave_max(nr);
        const int free_ = WAVE - (runs >> 1);
        int F = min(longest, 1 + (int)((float)(m - 1) * __builtin_amdgcn_rcpf((float)free_)));
        int cnt = (int)(((float)(nr + F) - 0.5f) * __builtin_amdgcn_rcpf((float)F));
        int off = scan_sum(cnt);
        int total = __builtin_amdgcn_readlane(off, WAVE - 1);
        if (total > WAVE) {
            F = runs < WAVE ? min(longest, 1 + (int)((float)m * __builtin_amdgcn_rcpf((float)(WAVE - runs))))
                            : longest;
            cnt = (int)(((float)(nr + F) - 0.5f) * __builtin_amdgcn_rcpf((float)F));
            off = scan_sum(cnt);
            total = __builtin_amdgcn_readlane(off, WAVE - 1);
        }
        off -= cnt;
        // lane j takes fragment j: of the run whose first fragment is the last at or before j
        T.flag[lane] = -1;
        wave_sync();
        if (cnt > 0) T.flag[off] = lane;
        wave_sync();
        const int fl = T.flag[lane];
        const uint64_t firsts = __ballot(fl >= 0);
        const int f0 = 63 - __builtin_clzll(firsts & ((2ull << lane) - 1ull));   // (fragment 0 is a first one)
        const int run = __shfl(fl, f0);
        const int a0 = __shfl(p0, run) + (lane - f0) * F;
        const int left = __shfl(p1, run) - a0;
        const int len = lane < total ? min(F, left) : 0;
        Run acc;
        run_clear(acc);
        for (int k = 0; k < F; ++k) {
            const int i = k < len ? a0 + k : SHW_TILE;
            run_add(acc, T.hit[0][i], T.hit[1][i], T.hit[2][i], k < len);
        }
        wave_sync();
        T.f.d[0][lane] = acc.sx;
        T.f.d[1][lane] = acc.sxx;
        T.f.d[2][lane] = acc.sy;
        T.f.d[3][lane] = acc.syy;
        T.f.d[4][lane] = acc.sr;
        T.f.d[5][lane] = acc.se;
        T.f.d[6][lane] = acc.see;
        T.f.d[7][lane] = acc.sex;
        T.f.d[8][lane] = acc.sexx;
        T.f.d[9][lane] = acc.sey;
        T.f.d[10][lane] = acc.seyy;
        T.f.d[11][lane] = acc.ser;
        // the two largest energies of the run's fragments up to this one, in
        // the row of sixteen
        int nan_e = acc.se != acc.se ? 1 : 0;
        seg_top<1>(acc.e1, acc.e2, nan_e, run);
        seg_top<2>(acc.e1, acc.e2, nan_e, run);
        seg_top<4>(acc.e1, acc.e2, nan_e, run);
        seg_top<8>(acc.e1, acc.e2, nan_e, run);
        T.f.top[lane] = f32x2{acc.e1, acc.e2};
        wave_sync();
        // running sums over sixteen fragments, starting anew at each run
        if ((lane & 15) < SHW_SUMS) {
            f64x2 *row = (f64x2 *)&T.f.d[lane & 15][lane & 48];
            const int bits = (int)(uint32_t)(firsts >> (lane & 48));
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                f64x2 w = row[k];
                sum = ((bits >> (2 * k)) & 1) ? w.x : sum + w.x;
                w.x = sum;
                sum = ((bits >> (2 * k + 1)) & 1) ? w.y : sum + w.y;
                w.y = sum;
                row[k] = w;
            }
        }
        wave_sync();
        // the run's partial sums, one per sixteen fragments it has a part in
        const int lastf = off + cnt - 1;
        int f = cnt > 0 ? min(off | 15, lastf) : WAVE;
        while (__ballot(f <= lastf)) {
            if (f <= lastf) {
                own.sx += T.f.d[0][f];
                own.sxx += T.f.d[1][f];
                own.sy += T.f.d[2][f];
                own.syy += T.f.d[3][f];
                own.sr += T.f.d[4][f];
                const double se = T.f.d[5][f];
                own.se += se;
                own.see += T.f.d[6][f];
                own.sex += T.f.d[7][f];
                own.sexx += T.f.d[8][f];
                own.sey += T.f.d[9][f];
                own.seyy += T.f.d[10][f];
                own.ser += T.f.d[11][f];
                add_top(own.e1, own.e2, T.f.top[f].x, T.f.top[f].y, se != se);
                f = f == lastf ? WAVE : min(f + 16, lastf);
            }
        }
        own.n += nr;
        wave_sync();
    }

    // layers seen; a layer seen twice or out of range spoils the shower
    const bool mine = lane < R && R <= WAVE;
    const int l = mine ? T.lay[lane] : -1;
    uint64_t seen = 0;
    for (int r = 0; r < R && r < WAVE; ++r) {
        const int lr = __builtin_amdgcn_readlane(l, r);
        seen |= lr >= 0 && lr < 64 ? 1ull << lr : 0ull;
    }
    const bool bad = R > WAVE || __ballot(mine && l >= L) || (int)__builtin_popcountll(seen) != R;
    float *out = A.lv + (size_t)s * L * LV, *sv = A.sv + (size_t)s * SV;
    if (bad) {
        for (int f = lane; f < L * LV; f += WAVE) out[f] = nan;
        if (lane < SV) sv[lane] = nan;
        if (lane == 0) atomicAdd(A.work, 1);
        return;
    }
    const double se = mine ? own.se : 0.0;
    const double etot = wave_sum(se);
    const double ld = wave_sum((double)l * se), ld2 = wave_sum((double)l * (double)l * se);
    const int depth = wave_max(mine && own.se > 0.0 ? l + 1 : 0) - 1;
    const double it = etot > 0.0 ? recip(etot) : 0.0;
    if (mine) {
        write_layer(out + (size_t)l * LV, own);
        out[(size_t)l * LV + SUPA_LV_FRACTION] = etot > 0.0 ? (float)((double)(float)own.se * it) : nan;
    }
    if (lane < L && !((seen >> lane) & 1)) {
        write_empty_layer(out + (size_t)lane * LV);
        out[(size_t)lane * LV + SUPA_LV_FRACTION] = etot > 0.0 ? 0.0f : nan;
    }
    if (lane == 0) {
        const double sd = ld * it;
        sv[SUPA_SV_E_TOT] = (float)etot;
        sv[SUPA_SV_DEPTH] = (float)depth;
        sv[SUPA_SV_L_D] = (float)ld;
        sv[SUPA_SV_S_D] = etot > 0.0 ? (float)sd : nan;
        sv[SUPA_SV_S_D_WIDTH] = etot > 0.0 ? dev_of(sd, ld2 * it) : nan;
    }
}

__global__ void __launch_bounds__(WAVE) shapes_wave_kernel(ShapeArgs A) {
    __shared__ __attribute__((aligned(16))) WaveTile T;
    if (!A.work[2]) return;               // a lane each
    const int lane = threadIdx.x;
    for (int64_t s = blockIdx.x; s < A.n; s += gridDim.x) {
        wave_shower(A, T, s, lane);
        wave_sync();                      // (the tile is used again)
    }
}

__global__ void radius_kernel(int64_t n, const float *x, const float *y, float *r) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double a = x[i], b = y[i];
        r[i] = (float)__builtin_sqrt(a * a + b * b);
    }
}

// ---------------------------------------------------------------------------
// W1 between histograms
// ---------------------------------------------------------------------------

constexpr int W1_THREADS = 256;
constexpr int W1_HIST_WORDS = 8192;  // LDS histogram words per block (32 KB)
// Workgroups per sample at most: six per CU, as many as hold their histograms
// at once; both samples in one launch are two full rounds.  (2,048 per sample
// and a launch each: the histograms of 100,000 rows of 365 columns 2 x 63 us,
// a round of two thirds and one of a third; the sums 2 x 40 us.)
constexpr int W1_BLOCKS = 6 * 256;
constexpr int W1_ROWS = 8;           // rows per thread and round, all requested before any is used

struct Sample {
    const float *m;
    int64_t rows, ld;
    int rb;                          // row blocks
};

struct Partial {  // per (row block, column); sums shifted by the column's pivot
    double cnt, s1, s2, mn, mx;
};

struct ColInfo {
    double lo, scale, width, sigma, n_ref, n_smp;
    int32_t skip, pad;
};

__host__ __device__ inline int w1_cols_per_tile(int n_cols, int n_bins) {
    int ct = 1;
    while (ct < 64 && ct < n_cols && (ct * 2) * n_bins <= W1_HIST_WORDS) ct *= 2;
    return ct;
}

__host__ __device__ inline int w1_row_blocks(int64_t rows, int n_cols, int ct) {
    const int64_t tiles = (n_cols + ct - 1) / ct;
    int64_t rb = (rows + 255) / 256;
    const int64_t cap = W1_BLOCKS / tiles > 1 ? W1_BLOCKS / tiles : 1;
    if (rb > cap) rb = cap;
    if (rb < 1) rb = 1;
    return (int)rb;
}

__device__ inline bool finite(float v) { return __builtin_isfinite(v); }

// grid (tiles, row blocks of ref, then of smp)
__global__ void __launch_bounds__(W1_THREADS)
    w1_stats(Sample ref, Sample smp, int n_cols, int ct, Partial *part_ref, Partial *part_smp) {
    __shared__ double sh[5][W1_THREADS];
    const bool first = (int)blockIdx.y < ref.rb;
    const Sample S = first ? ref : smp;
    const int block = (int)blockIdx.y - (first ? 0 : ref.rb);
    Partial *part = first ? part_ref : part_smp;
    const float *m = S.m;
    const int64_t rows = S.rows, ld = S.ld;
    const int t = threadIdx.x;
    const int cl = t % ct, ph = t / ct, rpt = W1_THREADS / ct;
    const int c = blockIdx.x * ct + cl;
    const int64_t per = (rows + S.rb - 1) / S.rb;
    const int64_t r0 = (int64_t)block * per;
    const int64_t r1 = r0 + per < rows ? r0 + per : rows;
    double cnt = 0.0, s1 = 0.0, s2 = 0.0;
    float mn = __builtin_inff(), mx = -__builtin_inff();
    if (c < n_cols) {
        const float p0 = m[c];
        const double piv = finite(p0) ? (double)p0 : 0.0;
        for (int64_t r = r0 + ph; r < r1; r += W1_ROWS * (int64_t)rpt) {
            float v[W1_ROWS];
#pragma unroll
            for (int u = 0; u < W1_ROWS; ++u) {
                const int64_t q = r + (int64_t)u * rpt;
                v[u] = q < r1 ? m[q * ld + c] : __builtin_nanf("");
            }
#pragma unroll
            for (int u = 0; u < W1_ROWS; ++u) {
                if (!finite(v[u])) continue;
                const double d = (double)v[u] - piv;
                cnt += 1.0;
                s1 += d;
                s2 = __builtin_fma(d, d, s2);
                mn = v[u] < mn ? v[u] : mn;
                mx = v[u] > mx ? v[u] : mx;
            }
        }
    }
    sh[0][t] = cnt;
    sh[1][t] = s1;
    sh[2][t] = s2;
    sh[3][t] = mn;
    sh[4][t] = mx;
    __syncthreads();
    if (ph == 0 && c < n_cols) {
        for (int k = 1; k < rpt; ++k) {
            const int u = k * ct + cl;
            cnt += sh[0][u];
            s1 += sh[1][u];
            s2 += sh[2][u];
            mn = (float)sh[3][u] < mn ? (float)sh[3][u] : mn;
            mx = (float)sh[4][u] > mx ? (float)sh[4][u] : mx;
        }
        part[(size_t)block * n_cols + c] = Partial{cnt, s1, s2, (double)mn, (double)mx};
    }
}

// One wave per column: lane k adds the partials of row blocks k, k + 64, ...
// in order, then the lanes' sums are combined by a fixed butterfly (the same
// order on every run).
__global__ void __launch_bounds__(WAVE) w1_colinfo(int n_cols, int n_bins, const Partial *pr, int rbr,
                                                   const Partial *ps, int rbs, ColInfo *info) {
    const int c = blockIdx.x;
    const int lane = threadIdx.x;
    if (c >= n_cols) return;
    double nr = 0.0, s1 = 0.0, s2 = 0.0, mnr = __builtin_inf(), mxr = -__builtin_inf();
    for (int b = lane; b < rbr; b += WAVE) {
        const Partial p = pr[(size_t)b * n_cols + c];
        nr += p.cnt;
        s1 += p.s1;
        s2 += p.s2;
        mnr = p.mn < mnr ? p.mn : mnr;
        mxr = p.mx > mxr ? p.mx : mxr;
    }
    double ns = 0.0, mns = __builtin_inf(), mxs = -__builtin_inf();
    for (int b = lane; b < rbs; b += WAVE) {
        const Partial p = ps[(size_t)b * n_cols + c];
        ns += p.cnt;
        mns = p.mn < mns ? p.mn : mns;
        mxs = p.mx > mxs ? p.mx : mxs;
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        nr += __shfl_xor(nr, d);
        s1 += __shfl_xor(s1, d);
        s2 += __shfl_xor(s2, d);
        ns += __shfl_xor(ns, d);
        const double a = __shfl_xor(mnr, d), b = __shfl_xor(mxr, d);
        const double e = __shfl_xor(mns, d), f = __shfl_xor(mxs, d);
        mnr = a < mnr ? a : mnr;
        mxr = b > mxr ? b : mxr;
        mns = e < mns ? e : mns;
        mxs = f > mxs ? f : mxs;
    }
    if (lane != 0) return;
    ColInfo ci;
    ci.skip = (nr < 2.0 || ns < 1.0 || mnr == mxr) ? 1 : 0;
    ci.pad = 0;
    ci.n_ref = nr;
    ci.n_smp = ns;
    const double m1 = nr > 0.0 ? s1 / nr : 0.0;
    const double var = nr > 0.0 ? s2 / nr - m1 * m1 : 0.0;
    ci.sigma = __builtin_sqrt(var > 0.0 ? var : 0.0);
    ci.lo = mnr < mns ? mnr : mns;
    const double hi = mxr > mxs ? mxr : mxs;
    ci.width = ci.skip ? 0.0 : hi - ci.lo;
    ci.scale = ci.width > 0.0 ? (double)n_bins / ci.width : 0.0;
    info[c] = ci;
}

__global__ void w1_zero(uint32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// grid (tiles, row blocks of ref, then of smp); hist_*: [n_cols][n_bins].
__global__ void __launch_bounds__(W1_THREADS)
    w1_hist(Sample ref, Sample smp, int n_cols, int ct, int n_bins, const ColInfo *info, uint32_t *hist_ref,
            uint32_t *hist_smp) {
    extern __shared__ uint32_t hb[];  // [ct][n_bins]
    const bool first = (int)blockIdx.y < ref.rb;
    const Sample S = first ? ref : smp;
    const int block = (int)blockIdx.y - (first ? 0 : ref.rb);
    uint32_t *hist = first ? hist_ref : hist_smp;
    const float *m = S.m;
    const int64_t rows = S.rows, ld = S.ld;
    const int t = threadIdx.x;
    for (int i = t; i < ct * n_bins; i += W1_THREADS) hb[i] = 0;
    __syncthreads();
    const int cl = t % ct, ph = t / ct, rpt = W1_THREADS / ct;
    const int c = blockIdx.x * ct + cl;
    const int64_t per = (rows + S.rb - 1) / S.rb;
    const int64_t r0 = (int64_t)block * per;
    const int64_t r1 = r0 + per < rows ? r0 + per : rows;
    if (c < n_cols) {
        const ColInfo ci = info[c];
        if (!ci.skip) {
            uint32_t *h = hb + cl * n_bins;
            for (int64_t r = r0 + ph; r < r1; r += W1_ROWS * (int64_t)rpt) {
                float v[W1_ROWS];
#pragma unroll
                for (int u = 0; u < W1_ROWS; ++u) {
                    const int64_t q = r + (int64_t)u * rpt;
                    v[u] = q < r1 ? m[q * ld + c] : __builtin_nanf("");
                }
#pragma unroll
                for (int u = 0; u < W1_ROWS; ++u) {
                    if (!finite(v[u])) continue;
                    int k = (int)__builtin_floor(((double)v[u] - ci.lo) * ci.scale);
                    k = k < 0 ? 0 : (k >= n_bins ? n_bins - 1 : k);
                    atomicAdd(h + k, 1u);
                }
            }
        }
    }
    __syncthreads();
    for (int i = t; i < ct * n_bins; i += W1_THREADS) {
        const int cc = blockIdx.x * ct + i / n_bins;
        const uint32_t v = hb[i];
        if (cc < n_cols && v) atomicAdd(hist + (size_t)cc * n_bins + i % n_bins, v);
    }
}

// One wave per column: cumulative counts of both histograms, sum of the
// absolute differences of the cumulative fractions.
__global__ void __launch_bounds__(WAVE)
    w1_distance(int n_cols, int n_bins, const ColInfo *info, const uint32_t *hr, const uint32_t *hs,
                double *w1) {
    const int c = blockIdx.x;
    const int lane = threadIdx.x;
    const ColInfo ci = info[c];
    if (ci.skip) {
        if (lane == 0) w1[c] = __builtin_nan("");
        return;
    }
    const uint32_t *a = hr + (size_t)c * n_bins;
    const uint32_t *b = hs + (size_t)c * n_bins;
    uint64_t carry_a = 0, carry_b = 0;
    double acc = 0.0;
    for (int k0 = 0; k0 < n_bins; k0 += WAVE) {
        const int k = k0 + lane;
        uint64_t va = k < n_bins ? a[k] : 0, vb = k < n_bins ? b[k] : 0;
        // inclusive prefix sums across the wave
        for (int d = 1; d < WAVE; d <<= 1) {
            const uint64_t ua = __shfl_up(va, d), ub = __shfl_up(vb, d);
            if (lane >= d) {
                va += ua;
                vb += ub;
            }
        }
        va += carry_a;
        vb += carry_b;
        if (k < n_bins) {
            const double fa = (double)va / ci.n_ref, fb = (double)vb / ci.n_smp;
            acc += __builtin_fabs(fa - fb);
        }
        carry_a = __shfl(va, WAVE - 1);
        carry_b = __shfl(vb, WAVE - 1);
    }
    for (int d = WAVE / 2; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
    if (lane == 0) w1[c] = ci.width / (double)n_bins * acc / ci.sigma;
}

// One wave per group: lanes take columns c = lane, lane + 64, ...; the sums
// are combined by a fixed butterfly.
__global__ void __launch_bounds__(WAVE) w1_groups(int n_cols, const int32_t *group, int n_groups,
                                                  const double *w1, double *out) {
    const int g = blockIdx.x;
    const int lane = threadIdx.x;
    if (g >= n_groups) return;
    double s = 0.0;
    int k = 0;
    for (int c = lane; c < n_cols; c += WAVE) {
        const double v = w1[c];
        const bool in = group[c] == g && v == v;
        s += in ? v : 0.0;
        k += in ? 1 : 0;
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        s += __shfl_xor(s, d);
        k += __shfl_xor(k, d);
    }
    if (lane == 0) out[g] = k ? s / k : __builtin_nan("");
}

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct W1Layout {
    int ct, tiles, rbr, rbs;
    size_t off_pr, off_ps, off_info, off_hr, off_hs, total;
};

W1Layout w1_layout(int n_cols, int n_bins, int64_t n_ref, int64_t n_smp) {
    W1Layout w;
    w.ct = w1_cols_per_tile(n_cols, n_bins);
    w.tiles = (n_cols + w.ct - 1) / w.ct;
    w.rbr = w1_row_blocks(n_ref, n_cols, w.ct);
    w.rbs = w1_row_blocks(n_smp, n_cols, w.ct);
    size_t o = 0;
    w.off_pr = o;
    o += align256((size_t)w.rbr * n_cols * sizeof(Partial));
    w.off_ps = o;
    o += align256((size_t)w.rbs * n_cols * sizeof(Partial));
    w.off_info = o;
    o += align256((size_t)n_cols * sizeof(ColInfo));
    w.off_hr = o;
    o += align256((size_t)n_cols * n_bins * 4);
    w.off_hs = o;
    o += align256((size_t)n_cols * n_bins * 4);
    w.total = o;
    return w;
}

int g_cu_count = 0;

int cu_count() {
    if (g_cu_count == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            g_cu_count = n;
        else
            g_cu_count = 256;
    }
    return g_cu_count;
}

thread_local std::string t_err;

supa_status bad_arg(const char *msg) {
    t_err = msg;
    return SUPA_ERR_INVALID_ARG;
}

supa_status dev_err(hipError_t e, const char *what) {
    if (e == hipSuccess) return SUPA_OK;
    t_err = std::string(what) + ": " + hipGetErrorString(e);
    return SUPA_ERR_DEVICE;
}

}  // namespace

extern "C" const char *supa_shapes_last_error(void) { return t_err.c_str(); }

extern "C" int64_t supa_shapes_work_ints(int64_t n) { return n < 0 ? -1 : WORK_HEAD + n; }

extern "C" supa_status supa_shower_shapes(void *stream, int64_t n, int32_t n_layers,
                                          const int64_t *hit_offsets, const int32_t *hit_counts,
                                          int32_t counts_stride, int64_t hit_len, const float *hit_x,
                                          const float *hit_y, const float *hit_e,
                                          const int32_t *hit_layer, float *layer_vars,
                                          float *shower_vars, int32_t *work, int64_t work_ints) {
    if (n < 0 || n > INT32_MAX) return bad_arg("n out of range");
    if (n_layers < 1 || n_layers > 64) return bad_arg("n_layers must be 1..64");
    if (counts_stride < 1) return bad_arg("counts_stride must be >= 1");
    if (hit_len < 0) return bad_arg("hit_len < 0");
    if (!work) return bad_arg("work is NULL");
    if (work_ints < supa_shapes_work_ints(n)) return bad_arg("work holds fewer than supa_shapes_work_ints(n) int32");
    if (n > 0 && (!hit_offsets || !hit_counts || !hit_x || !hit_y || !hit_e || !hit_layer ||
                  !layer_vars || !shower_vars))
        return bad_arg("NULL array");
    // blocks of four hits are read with 16-byte loads
    if (n > 0 && (((uintptr_t)hit_x | (uintptr_t)hit_y | (uintptr_t)hit_e | (uintptr_t)hit_layer) & 15))
        return bad_arg("hit arrays must be 16-byte aligned");
    if (n > 0 && ((uintptr_t)layer_vars & 7)) return bad_arg("layer_vars must be 8-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    const int64_t few = (int64_t)cu_count() * WAVE_CALLS;
    hipLaunchKernelGGL(shapes_clear, dim3(1), dim3(1024), 0, s, work, n, hit_offsets, hit_counts, counts_stride,
                       n <= few ? 1 : 0);
    if (n == 0) return dev_err(hipGetLastError(), "shapes_clear");
    int32_t *order = work + WORK_HEAD;
    const int32_t *by_wave = work + 2;
    ShapeArgs A{n, n_layers, hit_offsets, hit_counts, counts_stride, hit_len, hit_x, hit_y, hit_e,
                hit_layer, layer_vars, shower_vars, work, order};
    hipLaunchKernelGGL(shapes_wave_kernel, dim3((unsigned)(n < 2 * few ? n : 2 * few)), dim3(WAVE), 0, s, A);
    if (n <= few) return dev_err(hipGetLastError(), "shapes_wave_kernel");
    const int64_t waves = (n + WAVE - 1) / WAVE;
    const int64_t cap = (int64_t)cu_count() * 16;
    const int grid = (int)(waves < cap ? waves : cap);
    if (waves <= cap) {  // every shower in flight at once (one per lane): one order
        uint32_t *gsize = (uint32_t *)work + 4, *gcur = gsize + ORDER_BUCKETS;
        const int blocks = (int)((n + ORDER_CHUNK - 1) / ORDER_CHUNK);
        hipLaunchKernelGGL(shapes_order_sizes, dim3(blocks), dim3(ORDER_THREADS), 0, s, n, hit_counts,
                           counts_stride, by_wave, gsize);
        hipLaunchKernelGGL(shapes_order_place, dim3(blocks), dim3(ORDER_THREADS), 0, s, n, hit_counts,
                           counts_stride, by_wave, gsize, gcur, order);
    } else {
        hipLaunchKernelGGL(shapes_order, dim3((int)((n + ORDER_WIN - 1) / ORDER_WIN)), dim3(ORDER_THREADS), 0,
                           s, n, (int64_t)ORDER_WIN, hit_counts, counts_stride, by_wave, order);
    }
    hipLaunchKernelGGL(shapes_kernel, dim3(grid), dim3(WAVE), (size_t)n_layers * WAVE * sizeof(float),
                       s, A);
    return dev_err(hipGetLastError(), "shapes_kernel");
}

extern "C" supa_status supa_hit_radius(void *stream, int64_t n, const float *x, const float *y,
                                       float *r) {
    if (n < 0) return bad_arg("n < 0");
    if (n == 0) return SUPA_OK;
    if (!x || !y || !r) return bad_arg("NULL array");
    int64_t blocks = (n + 255) / 256;
    const int64_t cap = (int64_t)cu_count() * 8;
    if (blocks > cap) blocks = cap;
    hipLaunchKernelGGL(radius_kernel, dim3((int)blocks), dim3(256), 0, (hipStream_t)stream, n, x, y, r);
    return dev_err(hipGetLastError(), "radius_kernel");
}

extern "C" size_t supa_w1_workspace_bytes(int32_t n_cols, int32_t n_bins, int64_t n_ref,
                                          int64_t n_smp) {
    if (n_cols < 1 || n_bins < 1 || n_ref < 1 || n_smp < 1) return 0;
    return w1_layout(n_cols, n_bins, n_ref, n_smp).total;
}

extern "C" supa_status supa_w1_normalized(void *stream, int32_t n_cols, const float *ref,
                                          int64_t n_ref, int64_t ref_ld, const float *smp,
                                          int64_t n_smp, int64_t smp_ld, int32_t n_bins,
                                          const int32_t *group_of_col, int32_t n_groups,
                                          double *w1, double *group_mean, void *workspace,
                                          size_t workspace_bytes) {
    if (n_cols < 1 || n_cols > 65535) return bad_arg("n_cols must be 1..65535");
    if (n_bins < 1 || n_bins > 4096) return bad_arg("n_bins must be 1..4096");
    if (n_ref < 1 || n_ref > INT32_MAX || n_smp < 1 || n_smp > INT32_MAX)
        return bad_arg("row counts must be 1..2^31-1");
    if (ref_ld < n_cols || smp_ld < n_cols) return bad_arg("leading dimension < n_cols");
    if (!ref || !smp || !w1 || !workspace) return bad_arg("NULL pointer");
    if (group_of_col && (n_groups < 1 || !group_mean)) return bad_arg("groups need n_groups >= 1 and group_mean");
    const W1Layout w = w1_layout(n_cols, n_bins, n_ref, n_smp);
    if (workspace_bytes < w.total) return bad_arg("workspace too small");
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    Partial *pr = (Partial *)(ws + w.off_pr), *ps = (Partial *)(ws + w.off_ps);
    ColInfo *info = (ColInfo *)(ws + w.off_info);
    uint32_t *hr = (uint32_t *)(ws + w.off_hr), *hs = (uint32_t *)(ws + w.off_hs);

    const int64_t zero_words = (int64_t)(w.total - w.off_hr) / 4;
    hipLaunchKernelGGL(w1_zero, dim3(cu_count() * 4), dim3(256), 0, s, hr, zero_words);
    const Sample A{ref, n_ref, ref_ld, w.rbr}, B{smp, n_smp, smp_ld, w.rbs};
    hipLaunchKernelGGL(w1_stats, dim3(w.tiles, w.rbr + w.rbs), dim3(W1_THREADS), 0, s, A, B, n_cols, w.ct, pr, ps);
    hipLaunchKernelGGL(w1_colinfo, dim3(n_cols), dim3(WAVE), 0, s, n_cols, n_bins, pr,
                       w.rbr, ps, w.rbs, info);
    const size_t lds = (size_t)w.ct * n_bins * 4;
    hipLaunchKernelGGL(w1_hist, dim3(w.tiles, w.rbr + w.rbs), dim3(W1_THREADS), lds, s, A, B, n_cols, w.ct, n_bins,
                       info, hr, hs);
    hipLaunchKernelGGL(w1_distance, dim3(n_cols), dim3(WAVE), 0, s, n_cols, n_bins, info, hr, hs, w1);
    if (group_of_col)
        hipLaunchKernelGGL(w1_groups, dim3(n_groups), dim3(WAVE), 0, s, n_cols, group_of_col,
                           n_groups, w1, group_mean);
    return dev_err(hipGetLastError(), "w1 kernels");
}
