/*
 * pg_kernels.h -- gfx950 kernels of the policy-gradient step that follows the
 * reward in every PA-GRPO update: group-normalised advantages and the
 * token-level clipped surrogate with separate lower and upper clip ratios
 * (the paper trains with clip ratios 0.2 and 0.28 and 8 rollouts per prompt,
 * Sec. 4 "Training Framework"; the objective itself is the standard GRPO one
 * with DAPO-style clip-higher and a token-level mean, which the paper does not
 * restate).
 *
 *   pg_prepare     (more than SCAN_PLAN_ROWS rows, then plan_rows; with fewer
 *                  pg_surrogate's blocks do it) segments and tokens per tile of
 *                  rows, exact, and the advantages, one thread per group: A_i =
 *                  (R_i - mean) / std over the group's float rewards
 *                  (population std, IEEE double, index order; A = 0 when all
 *                  rewards of the group are equal).
 *   pg_surrogate   HBM-bound, one wave per segment of a row (the segment plan
 *                  of the accounting path, two segments in flight per wave,
 *                  the waves taking them in turn):
 *                  d = logp - logp_old in float,
 *                  rho = exp(d) from the hardware exp2 (exp_ratio), the clip
 *                  decision on d against float thresholds ln(1 - eps_low),
 *                  ln(1 + eps_high), the objective term summed in double, the
 *                  gradient of the loss -J with respect to logp written in
 *                  float.  The row's advantage is uniform over a segment, so
 *                  its sign, and whether the segment holds a row end, are
 *                  wave-uniform branches rather than per-token selects.
 *   pg_final       loss, token count and clip counts in fixed order.
 */
#pragma once
#include "device_common.h"

namespace pk {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 load_f4(const float4 *p)
{
    v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void store_f4(float4 *p, float a, float b, float c, float d)
{
    v4f v = {a, b, c, d};
    __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(p));
}

struct PgArgs {
    const float *logp_base;  /* 16-byte aligned bases: pointer - mis elements */
    const float *old_base;
    float *grad_base;
    int64_t mis;
    const int64_t *starts;
    const int32_t *lengths;
    int64_t n;
    const int64_t *seg_off;
    const float *reward;
    int32_t G;
    float *adv;              /* per row */
    float thr_low, thr_high; /* ln(1 - eps_low), ln(1 + eps_high) */
    float lo_val, hi_val;    /* 1 - eps_low, 1 + eps_high */
    int64_t *n_tokens;       /* computed on the device */
    double *wsum;            /* [blocks] sum of the objective terms */
    int64_t *wcnt;           /* [blocks][2] clipped high, clipped low */
};

/* The advantages of a group from its rewards R[0 .. G) (adv may be R). */
__device__ __forceinline__ void group_advantage(const float *R, int32_t G, float *adv)
{
    bool equal = true;
    for (int32_t i = 1; i < G; ++i) equal = equal && R[i] == R[0];
    if (equal) {
        for (int32_t i = 0; i < G; ++i) adv[i] = 0.0f;
        return;
    }
    double s = 0.0;
    for (int32_t i = 0; i < G; ++i) s = __dadd_rn(s, (double)R[i]);
    const double mu = __ddiv_rn(s, (double)G);
    double ss = 0.0;
    for (int32_t i = 0; i < G; ++i) {
        const double d = __dsub_rn((double)R[i], mu);
        ss = __dadd_rn(ss, __dmul_rn(d, d));
    }
    const double sigma = __dsqrt_rn(__ddiv_rn(ss, (double)G));
    for (int32_t i = 0; i < G; ++i) adv[i] = (float)__ddiv_rn(__dsub_rn((double)R[i], mu), sigma);
}

/* What a batch of more than SCAN_PLAN_ROWS rows needs before its plan: block
 * b's tile of PLAN_TILE rows (segments and tokens, exact), and the advantages
 * of groups [b PLAN_THREADS, (b + 1) PLAN_THREADS), one thread per group. */
__global__ void __launch_bounds__(PLAN_THREADS) pg_prepare(PgArgs a, int64_t n_tiles, int64_t n_groups,
                                                           int64_t *__restrict__ tile_sum,
                                                           int64_t *__restrict__ len_sum)
{
    __shared__ int64_t part[PLAN_THREADS / WAVE];
    const int64_t grp = (int64_t)blockIdx.x * PLAN_THREADS + threadIdx.x;
    if (blockIdx.x < n_tiles) {
        const int64_t r0 = (int64_t)blockIdx.x * PLAN_TILE;
        const int64_t segs = tile_segments(a.starts, a.lengths, a.n, a.mis, r0, part);
        int64_t len = 0;
#pragma unroll
        for (int j = 0; j < PLAN_RPT; ++j) {
            const int64_t r = r0 + threadIdx.x + j * PLAN_THREADS;
            const int32_t l = a.lengths[min(r, a.n - 1)];
            len += r < a.n && l > 0 ? l : 0;
        }
        len = block_sum(len, part);
        if (threadIdx.x == 0) {
            tile_sum[blockIdx.x] = segs;
            len_sum[blockIdx.x] = len;
        }
    }
    if (grp < n_groups) group_advantage(a.reward + grp * a.G, a.G, a.adv + grp * a.G);
}

/* Wave-wide sums in a fixed order (butterfly over the 64 lanes). */
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, WAVE);
    return v;
}

__device__ __forceinline__ int64_t wave_sum(int64_t v)
{
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, WAVE);
    return v;
}

/* Loads of one segment: logp and logp_old vectors v0 + i*WAVE + lane. */
__device__ __forceinline__ void pg_loads(const PgArgs &a, const SegView &w, int lane, float4 (&xn)[LOADS],
                                         float4 (&xo)[LOADS])
{
    const float4 *pn = reinterpret_cast<const float4 *>(a.logp_base);
    const float4 *po = reinterpret_cast<const float4 *>(a.old_base);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int64_t v = w.v0 + i * WAVE + lane;
        if (!w.edge || v < w.v1) {
            xn[i] = load_f4(pn + v);
            xo[i] = load_f4(po + v);
        } else {
            xn[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            xo[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

/* e^d for the policy ratio, from the hardware base-2 exponential with the
 * exponent split in the manner of Cody and Waite: d log2(e) = h + r with
 * h = fl(d * L2E_HI) and r = (d * L2E_HI - h) + d * L2E_LO, where the first
 * difference is exact by an fma and L2E_HI + L2E_LO equals log2(e) to 2^-51.
 * Then e^d = 2^h * 2^r, and 2^r = 1 + r ln 2 up to (r ln 2)^2 / 2 < 2^-35
 * because |r| < 2^-17 below the overflow threshold.  An exhaustive sweep of
 * every float d in [-87.33, 88.72) (normal results) on gfx950 measured at
 * most 2.2 ulp against e^d in double (the hardware exp2 itself: 0.79 ulp);
 * the result is +inf above 88.72, as expf's is, and below -87.33 it is
 * within 2^-126 of e^d.  Five float operations and one exp2, against about
 * a dozen for expf with its range checks. */
__device__ __forceinline__ float exp_ratio(float d)
{
    const float L2E_HI = 1.44269502162933349609375f;   /* log2(e) rounded to float */
    const float L2E_LO = 1.925963033500011079e-8f;      /* log2(e) - L2E_HI */
    const float LN2 = 0.693147182464599609375f;         /* ln 2 rounded to float */
    const float h = d * L2E_HI;
    float r = __builtin_fmaf(d, L2E_HI, -h);
    r = __builtin_fmaf(d, L2E_LO, r);
    return __builtin_amdgcn_exp2f(h) * __builtin_fmaf(r, LN2, 1.0f);
}

/* Objective terms, gradient stores and clipped-token count of one loaded
 * segment whose row has advantage A of sign SIGN (0 also stands for a NaN
 * advantage: nothing is clipped).  A token is kept (its unclipped term is the
 * minimum) when d <= ln(1 + eps_high) for A > 0 and d >= ln(1 - eps_low) for
 * A < 0; clipA is the clip bound times A.  EDGE segments hold the first or the
 * last vector of the row, where tokens outside the row are neither counted
 * nor stored. */
template <int SIGN, bool EDGE>
__device__ __forceinline__ void pg_tokens(const PgArgs &a, const SegView &w, int lane, const float4 (&xn)[LOADS],
                                          const float4 (&xo)[LOADS], float A, float thr, float clipA, float inv_n,
                                          double &acc, uint32_t &clipped)
{
    const uint32_t span = (uint32_t)(w.q_hi - w.q_lo);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int64_t v = w.v0 + i * WAVE + lane;
        const int32_t b = 4 * (i * WAVE + lane) - w.q_lo;
        const float nn[4] = {xn[i].x, xn[i].y, xn[i].z, xn[i].w};
        const float oo[4] = {xo[i].x, xo[i].y, xo[i].z, xo[i].w};
        float g[4];
        bool in[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            in[j] = !EDGE || (uint32_t)(b + j) < span;
            const float d = __fsub_rn(nn[j], oo[j]);
            const float p = A * exp_ratio(d);
            const bool keep = SIGN > 0 ? d <= thr : SIGN < 0 ? d >= thr : true;
            g[j] = keep ? -p * inv_n : 0.0f;
            const float L = keep ? p : clipA;
            if (EDGE) {
                acc += (double)(in[j] ? L : 0.0f);
                if (SIGN != 0) clipped += (!keep && in[j]) ? 1u : 0u;
            } else {
                acc += (double)L;
                if (SIGN != 0) clipped += keep ? 0u : 1u;
            }
        }
        float *dst = a.grad_base + 4 * v;
        if (!EDGE || (in[0] && in[3])) {
            store_f4(reinterpret_cast<float4 *>(dst), g[0], g[1], g[2], g[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (in[j]) dst[j] = g[j];
        }
    }
}

/* One loaded segment: the row's advantage decides the branch for the whole
 * wave. */
__device__ __forceinline__ void pg_segment(const PgArgs &a, const float *adv, const SegView &w, int lane,
                                           const float4 (&xn)[LOADS], const float4 (&xo)[LOADS], float inv_n,
                                           double &acc, uint32_t &clip_hi, uint32_t &clip_lo)
{
    const float A = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(adv[w.row])));
    if (A > 0.0f) {
        const float clipA = a.hi_val * A;
        if (w.edge) pg_tokens<1, true>(a, w, lane, xn, xo, A, a.thr_high, clipA, inv_n, acc, clip_hi);
        else pg_tokens<1, false>(a, w, lane, xn, xo, A, a.thr_high, clipA, inv_n, acc, clip_hi);
    } else if (A < 0.0f) {
        const float clipA = a.lo_val * A;
        if (w.edge) pg_tokens<-1, true>(a, w, lane, xn, xo, A, a.thr_low, clipA, inv_n, acc, clip_lo);
        else pg_tokens<-1, false>(a, w, lane, xn, xo, A, a.thr_low, clipA, inv_n, acc, clip_lo);
    } else {
        if (w.edge) pg_tokens<0, true>(a, w, lane, xn, xo, A, 0.0f, 0.0f, inv_n, acc, clip_hi);
        else pg_tokens<0, false>(a, w, lane, xn, xo, A, 0.0f, 0.0f, inv_n, acc, clip_hi);
    }
}

/* One wave per segment of the plan.  The waves take chunks of segments in turn,
 * so that all of them stream inside one window of the three arrays: with a
 * contiguous range per wave (4,096 windows) 20,000 rows of 20,000 tokens took
 * 976 us, in chunks of 2 segments 882-910, of 4 914, of 8 940 (4.8 GB; torch's
 * sub of the same bytes 800).  A chunk is found by a search; where the plan is
 * in LDS that is cheap enough for chunks of one segment, which leave the waves
 * within one segment of each other (1,024 rows of 26,800 tokens: 67.4 us, 70.6
 * as ranges).  Arrays of tens of GB are the exception: there a range per wave is
 * within 1 % of the chunks where the buffers' placement is bad for it and 9 %
 * ahead where it is good (17.9e9 tokens, 4,270 segments per wave: ranges 39.8 and
 * chunks 39.4 ms in three processes, 36.5 and 39.8 in a fourth).  The crossing, over
 * three more processes each: 1,200 segments per wave ranges 10.7-12.0 and chunks
 * 10.9-11.1 ms, 1,600 15.0-15.7 and 14.5-14.7, 2,000 17.5-19.4 and 17.9-18.4, 2,600
 * 22.3-22.9 and 23.7-24.1, 3,200 27.0-27.9 and 29.3-29.9.  So from PG_RANGE_SEGS
 * segments per wave each wave takes one chunk, its share of them.  Two register buffers alternate so that the next segment's loads
 * are in flight while the current one is evaluated.
 * PLAN (up to SCAN_PLAN_ROWS rows): every block makes the plan, the token count
 * and the advantages itself in LDS, in blocks of 8 waves so that half as many
 * blocks do; block 0 also writes the advantages and the count.  In place of
 * launches for the plan, the count (two) and the advantages, which took 16 of
 * the 27 us of 64 rows of 3,500 tokens (13.8 now) and 20 of the 89 us of 1,024
 * rows of 26,800 (67 now). */
constexpr int PG_WAVES = 4, PG_PLAN_WAVES = 8;
constexpr int PG_RANGE_SEGS = 2048; /* segments per wave from which a wave takes one range */
template <bool PLAN>
constexpr int pg_waves() { return PLAN ? PG_PLAN_WAVES : PG_WAVES; }

template <bool PLAN>
__global__ void __launch_bounds__(WAVE * pg_waves<PLAN>(), 4) pg_surrogate(PgArgs a)
{
    constexpr int NW = pg_waves<PLAN>();
    __shared__ int64_t plan_off[PLAN ? SCAN_PLAN_ROWS + 1 : 1];
    __shared__ int64_t plan_st[PLAN ? SCAN_PLAN_ROWS : 1];
    __shared__ int32_t plan_ln[PLAN ? SCAN_PLAN_ROWS : 1];
    __shared__ float plan_adv[PLAN ? SCAN_PLAN_ROWS : 1];
    __shared__ int64_t part[3][NW];
    __shared__ double part_d[NW];
    const int t = threadIdx.x, lane = t & (WAVE - 1);
    const int wib = __builtin_amdgcn_readfirstlane(t / WAVE);
    const int64_t wave = uniform64((int64_t)blockIdx.x * NW + wib);
    const int64_t n_waves = (int64_t)gridDim.x * NW;
    const int64_t *seg_off = a.seg_off, *starts = a.starts;
    const int32_t *lengths = a.lengths;
    const float *adv = a.adv;
    int64_t N;
    if (PLAN) {
        for (int64_t r = t; r < a.n; r += WAVE * NW) plan_adv[r] = a.reward[r]; /* before block_plan's barriers */
        block_plan<NW>(a.starts, a.lengths, a.n, a.mis, plan_off, part[0], plan_st, plan_ln);
        int64_t len = 0;
        for (int64_t r = t; r < a.n; r += WAVE * NW) len += plan_ln[r] > 0 ? plan_ln[r] : 0;
        len = wave_inclusive_scan(len);
        /* part[0], which block_plan is done with and nothing writes again: no
         * barrier lies between the reads of N below and the kernel's last sums */
        if (lane == WAVE - 1) part[0][wib] = len;
        for (int64_t g = t; g < a.n / a.G; g += WAVE * NW) group_advantage(plan_adv + g * a.G, a.G, plan_adv + g * a.G);
        __syncthreads();
        N = 0;
        for (int w = 0; w < NW; ++w) N += part[0][w];
        if (blockIdx.x == 0) {
            for (int64_t r = t; r < a.n; r += WAVE * NW) a.adv[r] = plan_adv[r];
            if (t == 0) a.n_tokens[0] = N;
        }
        seg_off = plan_off;
        starts = plan_st;
        lengths = plan_ln;
        adv = plan_adv;
    } else {
        N = a.n_tokens[0];
    }
    N = uniform64(N);
    const int64_t S = uniform64(seg_off[a.n]);
    const int32_t chunk =
        PLAN ? 1 : __builtin_amdgcn_readfirstlane(
                       S < n_waves * PG_RANGE_SEGS ? 2 : (int32_t)min((S + n_waves - 1) / n_waves, (int64_t)INT32_MAX));
    const int64_t hop = (n_waves - 1) * chunk + 1; /* from a chunk's last segment to the next chunk's first */
    double acc = 0.0;
    /* per-lane clip counts: a lane sees at most a 64th of the batch's tokens */
    uint32_t clip_hi = 0, clip_lo = 0;
    int64_t s = wave * chunk;
    if (s < S) {
        const float inv_n = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int((float)__ddiv_rn(1.0, (double)N))));
        SegCursor cur;
        cur.seg_off = seg_off;
        cur.starts = starts;
        cur.lengths = lengths;
        cur.mis = a.mis;
        cur.s_begin = 0;
        cur.s_end = S;
        cur.seek(s, a.n);
        float4 na[LOADS], oa[LOADS], nb[LOADS], ob[LOADS];
        SegView w = cur.view(s);
        pg_loads(a, w, lane, na, oa);
        int32_t left = chunk - 1; /* segments left of the chunk after s */
        while (true) {
            SegView wn;
            int64_t sn = left > 0 ? s + 1 : s + hop;
            bool more = sn < S;
            if (more) {
                if (left == 0) cur.seek(sn, a.n);
                wn = cur.view(sn);
                pg_loads(a, wn, lane, nb, ob);
            }
            left = left > 0 ? left - 1 : chunk - 1;
            pg_segment(a, adv, w, lane, na, oa, inv_n, acc, clip_hi, clip_lo);
            if (!more) break;
            s = sn;
            w = wn;
            sn = left > 0 ? s + 1 : s + hop;
            more = sn < S;
            if (more) {
                if (left == 0) cur.seek(sn, a.n);
                wn = cur.view(sn);
                pg_loads(a, wn, lane, na, oa);
            }
            left = left > 0 ? left - 1 : chunk - 1;
            pg_segment(a, adv, w, lane, nb, ob, inv_n, acc, clip_hi, clip_lo);
            if (!more) break;
            s = sn;
            w = wn;
        }
    }
    acc = wave_sum(acc);
    const int64_t hi_sum = wave_sum((int64_t)clip_hi);
    const int64_t lo_sum = wave_sum((int64_t)clip_lo);
    if (lane == 0) {
        part_d[wib] = acc;
        part[1][wib] = hi_sum;
        part[2][wib] = lo_sum;
    }
    __syncthreads();
    if (t == 0) { /* the block's waves in order */
        double s = 0.0;
        int64_t hi = 0, lo = 0;
        for (int w = 0; w < NW; ++w) {
            s += part_d[w];
            hi += part[1][w];
            lo += part[2][w];
        }
        a.wsum[blockIdx.x] = s;
        a.wcnt[2 * blockIdx.x] = hi;
        a.wcnt[2 * blockIdx.x + 1] = lo;
    }
}

/* stats = {loss, tokens, clipped high, clipped low}, sums over the blocks in a
 * fixed order. */
__global__ void __launch_bounds__(RED_THREADS) pg_final(const double *__restrict__ wsum,
                                                        const int64_t *__restrict__ wcnt, int64_t blocks,
                                                        const int64_t *__restrict__ n_tokens, double *__restrict__ stats)
{
    __shared__ double part_d[RED_THREADS / WAVE];
    __shared__ int64_t part[2][RED_THREADS / WAVE];
    const int t = threadIdx.x, lane = t & (WAVE - 1), wv = t / WAVE;
    const int64_t N = n_tokens[0];
    double s = 0.0;
    int64_t hi = 0, lo = 0;
    for (int64_t b = t; b < blocks; b += RED_THREADS) { /* coalesced */
        s += wsum[b];
        hi += wcnt[2 * b];
        lo += wcnt[2 * b + 1];
    }
    s = wave_sum(s);
    hi = wave_sum(hi);
    lo = wave_sum(lo);
    if (lane == 0) {
        part_d[wv] = s;
        part[0][wv] = hi;
        part[1][wv] = lo;
    }
    __syncthreads();
    if (t != 0) return;
    for (int w = 1; w < RED_THREADS / WAVE; ++w) {
        s += part_d[w];
        hi += part[0][w];
        lo += part[1][w];
    }
    stats[PARASON_PG_STAT_LOSS] = N > 0 ? -__ddiv_rn(s, (double)N) : 0.0;
    stats[PARASON_PG_STAT_TOKENS] = (double)N;
    stats[PARASON_PG_STAT_CLIP_HIGH] = (double)hi;
    stats[PARASON_PG_STAT_CLIP_LOW] = (double)lo;
}

} /* namespace pk */
