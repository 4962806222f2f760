/*
 * parason_kernels.h -- gfx950 kernels of the Parason accounting/reward path.
 *
 * Data flow of one parason_run (all on the caller's stream):
 *
 *   plan_direct, or plan_tiles / plan_rows  (more than PLAN_ONE tiles of rows;
 *        plan_top between them for more than PLAN_TWO)
 *        Each row is cut into segments of SEG_VEC 16-byte vectors, starting at
 *        the 128-byte line that holds its first token.  An exclusive scan over
 *        the rows gives seg_off[i] (first segment of row i) and the segment count
 *        seg_off[n]; mode[i] is cleared.  A batch of at most SCAN_PLAN_ROWS
 *        rows skips these launches: every scan block makes the plan in LDS
 *        itself (scan_plan).
 *   scan_rows  (HBM-bound; one wave per segment, persistent grid)
 *        Streams every token once with 16-byte loads, tests it against the
 *        twelve tag ids with a wave ballot and compacts the rare tags (about
 *        0.1-1% of tokens) in position order.  A row whose segments all fall in
 *        one wave's range collects its events in that wave's LDS buffer and is
 *        written out, coalesced, as one compact list (mode[i] = 1).  Other rows
 *        leave their events in per-segment lists (mode[i] = 0).  Every list the scan writes is in the wave's region of the
 *        slot pool; seg[s] holds its length and first slot.
 *   rows_par  (small batches: one wave per row, one to four events per lane)
 *        Validity from local checks and a depth prefix sum; latency and branch
 *        tokens level by level with segmented scans (DPP).  A segment whose
 *        events the scan could not store (marked DENSE) is read again by the
 *        wave.  A row it cannot hold runs through the grammar's pushdown
 *        automaton on one lane, with MID_DEPTH frames in LDS: Text runs are the
 *        gaps between event positions.
 *   rows_quad  (larger batches: four rows per wave, one to eight events per lane)
 *        The same, for rows of up to QUAD_EVENTS events; others by the whole
 *        wave as in rows_par.  A row that does not fit that either is listed.
 *   rows_listed  (after rows_quad: one thread per listed row)
 *        The automaton with frames of open blocks in LDS (FAST_DEPTH per row,
 *        64 outline entries per block; MID_DEPTH for the rows that need more);
 *        a row that needs more still is handed to the deep tier.
 *   group_reward  (one thread per row)
 *        Statistics and Definition 3.1 in IEEE double, fixed order.  The deep
 *        tier's rows, those rows_listed or rows_par handed over, are run first
 *        by a thread of its first block, by the same automaton with frames and
 *        entry types in global workspace, and then the rewards of their groups
 *        (mode[i] bit MODE_DEEP marks them, so every other block skips those
 *        groups).  With batch metrics each block also leaves its partial sums.
 *   batch_moments, batch_reward  (batch-wide statistics, in place of it)
 *        Mergeable moments per tile of rows (the deep tier's rows as one more
 *        record), then the rewards, every block merging the records itself.
 *   metrics_final  (batch metrics of more than one block)
 *   batch_single  (batch-wide statistics of up to 1,024 rows: one block)
 *
 * Paper references: grammar -- figure "Context-Free Grammar for Parason"
 * (Sec. 3.2); latency -- Sec. 4 "Evaluation"; ratios, eta and the reward --
 * Sec. 3.3, Definition 3.1.
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"

namespace pk {

/* mode[i], one byte per row: where its events are, and whether the deep tier
 * evaluates it. */
constexpr uint8_t MODE_COMPACT = 1; /* one compact list with row positions (else per-segment lists) */
constexpr uint8_t MODE_DEEP = 2;    /* listed for the single-thread tier with global frames */

/* ------------------------------------------------------------------ plan */

/* tile_sum[b] = number of segments of rows [b*PLAN_TILE, (b+1)*PLAN_TILE). */
__global__ void __launch_bounds__(PLAN_THREADS) plan_tiles(const int64_t *__restrict__ starts,
                                                           const int32_t *__restrict__ lengths, int64_t n,
                                                           int64_t mis, int64_t *__restrict__ tile_sum)
{
    __shared__ int64_t part[PLAN_THREADS / WAVE];
    const int64_t t = tile_segments(starts, lengths, n, mis, (int64_t)blockIdx.x * PLAN_TILE, part);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = t;
}

/* tile_off = exclusive scan of tile_sum; seg_off[n] = total; clears counters. */
__global__ void __launch_bounds__(1024) plan_top(const int64_t *__restrict__ tile_sum, int64_t n_tiles,
                                                 int64_t *__restrict__ tile_off, int64_t *__restrict__ seg_off,
                                                 int64_t n, int32_t *__restrict__ counters)
{
    __shared__ int64_t part[1024 / WAVE];
    __shared__ int64_t carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    if (threadIdx.x < 4) counters[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t base = 0; base < n_tiles; base += 1024) {
        int64_t i = base + threadIdx.x;
        int64_t v = i < n_tiles ? tile_sum[i] : 0;
        int64_t inc = wave_inclusive_scan(v);
        if ((threadIdx.x & (WAVE - 1)) == WAVE - 1) part[threadIdx.x / WAVE] = inc;
        __syncthreads();
        int64_t before = carry_s;
        for (int w = 0; w < (int)(threadIdx.x / WAVE); ++w) before += part[w];
        if (i < n_tiles) tile_off[i] = before + inc - v;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t t = 0;
            for (int w = 0; w < 1024 / WAVE; ++w) t += part[w];
            carry_s += t;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) seg_off[n] = carry_s;
}

/* seg_off[i] = first segment of row i; mode[i] = 0 (events in per-segment
 * lists).  The segments before a block's tile: tile_off (TOP, after plan_top), or
 * the sum over the tiles before it, which each block adds up itself, so that a
 * plan of up to PLAN_TWO tiles takes two launches (64,000 rows: 10.0 + 4.9 + 8.3
 * us with plan_top and tiles of 4,096 rows, sixteen to a thread, 4.7 + 4.7 now);
 * the last block then writes the total and clears the counters as plan_top
 * does.  The block's rows are loaded coalesced and scanned through LDS, as a
 * thread's rows are consecutive.  mode and the sum n_tokens of the tiles'
 * len_sum are optional. */
template <bool TOP>
__global__ void __launch_bounds__(PLAN_THREADS) plan_rows(const int64_t *__restrict__ starts,
                                                          const int32_t *__restrict__ lengths, int64_t n,
                                                          int64_t mis, const int64_t *__restrict__ tile_sum,
                                                          const int64_t *__restrict__ tile_off,
                                                          int64_t *__restrict__ seg_off, uint8_t *__restrict__ mode,
                                                          int32_t *__restrict__ counters,
                                                          const int64_t *__restrict__ len_sum,
                                                          int64_t *__restrict__ n_tokens)
{
    __shared__ int64_t part[PLAN_THREADS / WAVE];
    __shared__ int64_t cnt[PLAN_TILE];
    const int t = (int)threadIdx.x, wv = t / WAVE;
    const bool last = blockIdx.x == gridDim.x - 1;
    const int64_t r0 = (int64_t)blockIdx.x * PLAN_TILE;
    int64_t before = 0;
    if (TOP) {
        before = tile_off[blockIdx.x];
    } else {
        for (int64_t b = t; b < (int64_t)blockIdx.x; b += PLAN_THREADS) before += tile_sum[b];
        if (last && t < 4) counters[t] = 0;
    }
#pragma unroll
    for (int j = 0; j < PLAN_RPT; ++j) {
        const int64_t r = r0 + t + j * PLAN_THREADS, q = min(r, n - 1);
        const int64_t c = row_segments(starts[q], lengths[q], mis);
        cnt[t + j * PLAN_THREADS] = r < n ? c : 0;
        if (mode && r < n) mode[r] = 0;
    }
    if (!TOP) before = block_sum(before, part);
    __syncthreads();
    int64_t c[PLAN_RPT], s = 0;
#pragma unroll
    for (int k = 0; k < PLAN_RPT; ++k) {
        c[k] = cnt[t * PLAN_RPT + k];
        s += c[k];
    }
    const int64_t inc = wave_inclusive_scan(s);
    if ((t & (WAVE - 1)) == WAVE - 1) part[wv] = inc;
    __syncthreads();
    int64_t off = before + inc - s;
    for (int w = 0; w < wv; ++w) off += part[w];
#pragma unroll
    for (int k = 0; k < PLAN_RPT; ++k) {
        cnt[t * PLAN_RPT + k] = off;
        off += c[k];
    }
    if (!TOP && last && t == PLAN_THREADS - 1) seg_off[n] = off; /* the last thread ends at the total */
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PLAN_RPT; ++j) {
        const int64_t r = r0 + t + j * PLAN_THREADS;
        if (r < n) seg_off[r] = cnt[t + j * PLAN_THREADS];
    }
    if (last && len_sum) {
        int64_t s = 0;
        for (int64_t b = t; b < (int64_t)gridDim.x; b += PLAN_THREADS) s += len_sum[b];
        s = block_sum(s, part);
        if (t == 0) n_tokens[0] = s;
    }
}

/* The plan of up to PLAN_ONE tiles in one launch: each block, one row per
 * thread, adds up the rows before its tile itself, from the rows' records in
 * the caches (a call on 2,056 rows of 700 tokens 26.9 us with plan_tiles and
 * plan_rows, 24.1 so; 8,192 rows of 3,500 58.4 and 56.3, 16,384 of 500 56.4 and
 * 55.6). */
__global__ void __launch_bounds__(PLAN_TILE) plan_direct(const int64_t *__restrict__ starts,
                                                         const int32_t *__restrict__ lengths, int64_t n, int64_t mis,
                                                         int64_t *__restrict__ seg_off, uint8_t *__restrict__ mode,
                                                         int32_t *__restrict__ counters)
{
    constexpr int NW = PLAN_TILE / WAVE;
    __shared__ int64_t part[2][NW];
    const int t = (int)threadIdx.x, wv = t / WAVE;
    const int64_t r = (int64_t)blockIdx.x * PLAN_TILE + t, q = min(r, n - 1);
    const int64_t c_own = row_segments(starts[q], lengths[q], mis), c = r < n ? c_own : 0;
    int64_t before = 0;
#pragma unroll 4
    for (int64_t b = t; b < (int64_t)blockIdx.x * PLAN_TILE; b += PLAN_TILE) before += row_segments(starts[b], lengths[b], mis);
    const int64_t inc = wave_inclusive_scan(c);
    before = wave_inclusive_scan(before);
    if ((t & (WAVE - 1)) == WAVE - 1) {
        part[0][wv] = inc;
        part[1][wv] = before;
    }
    __syncthreads();
    int64_t off = inc - c;
    for (int w = 0; w < NW; ++w) off += part[1][w] + (w < wv ? part[0][w] : 0);
    if (r < n) {
        seg_off[r] = off;
        mode[r] = 0;
        if (r == n - 1) seg_off[n] = off + c;
    }
    if (blockIdx.x == 0 && t < 4) counters[t] = 0;
}

/* ------------------------------------------------------------------ automaton */

/* The open block on top of the stack (kept in registers). */
struct Top {
    int32_t saved_acc;  /* latency of the enclosing body when <Parallel> came */
    int32_t block_main; /* <Parallel> + outline tokens so far */
    int32_t max_w;      /* longest finished thread */
    int32_t n_e;        /* outline entries */
    int32_t k;          /* threads so far */
    uint32_t saved_ctx; /* branch type of the enclosing context */
    uint64_t ent;       /* fast store: entry-type bits; deep store: first bit index */
};

/* LDS store: depth frames for each of nt rows in LDS, entry types as a 64-bit
 * mask. */
struct LdsStore {
    int32_t *lds; /* [depth][FRAME_WORDS][nt] */
    int tid, nt, depth;
    __device__ int32_t &at(int d, int f) { return lds[(d * FRAME_WORDS + f) * nt + tid]; }
    __device__ bool push(const Top &t, int d)
    {
        if (d > depth) return false;
        at(d - 1, 0) = t.saved_acc;
        at(d - 1, 1) = t.block_main;
        at(d - 1, 2) = t.max_w;
        at(d - 1, 3) = t.n_e;
        at(d - 1, 4) = t.k;
        at(d - 1, 5) = (int32_t)t.saved_ctx;
        at(d - 1, 6) = (int32_t)(uint32_t)t.ent;
        at(d - 1, 7) = (int32_t)(uint32_t)(t.ent >> 32);
        return true;
    }
    __device__ void pop(Top &t, int d)
    {
        t.saved_acc = at(d - 1, 0);
        t.block_main = at(d - 1, 1);
        t.max_w = at(d - 1, 2);
        t.n_e = at(d - 1, 3);
        t.k = at(d - 1, 4);
        t.saved_ctx = (uint32_t)at(d - 1, 5);
        t.ent = (uint64_t)(uint32_t)at(d - 1, 6) | ((uint64_t)(uint32_t)at(d - 1, 7) << 32);
    }
    __device__ void begin_block(Top &t) { t.ent = 0; }
    __device__ void end_block(const Top &) {}
    __device__ bool add_entry(Top &t, bool trial)
    {
        if (t.n_e >= FAST_ENTRIES) return false;
        if (trial) t.ent |= (uint64_t)1 << t.n_e;
        return true;
    }
    __device__ uint32_t entry_type(const Top &t, int32_t k) { return ((t.ent >> k) & 1u) ? T_TRI : T_SUB; }
};

/* Deep store: frames and entry bits in global workspace (single thread). */
struct GlobalStore {
    int32_t *frames;    /* [max_frames][FRAME_WORDS] */
    uint32_t *bits;     /* max_bits bits */
    int64_t max_frames; /* at most DEEP_FRAMES */
    int64_t max_bits;   /* at most DEEP_ENTRY_BITS */
    int64_t esp;      /* next free entry bit */
    __device__ bool push(const Top &t, int d)
    {
        if ((int64_t)d > max_frames) return false;
        int32_t *f = frames + (int64_t)(d - 1) * FRAME_WORDS;
        f[0] = t.saved_acc;
        f[1] = t.block_main;
        f[2] = t.max_w;
        f[3] = t.n_e;
        f[4] = t.k;
        f[5] = (int32_t)t.saved_ctx;
        f[6] = (int32_t)(uint32_t)t.ent;
        f[7] = (int32_t)(uint32_t)(t.ent >> 32);
        return true;
    }
    __device__ void pop(Top &t, int d)
    {
        const int32_t *f = frames + (int64_t)(d - 1) * FRAME_WORDS;
        t.saved_acc = f[0];
        t.block_main = f[1];
        t.max_w = f[2];
        t.n_e = f[3];
        t.k = f[4];
        t.saved_ctx = (uint32_t)f[5];
        t.ent = (uint64_t)(uint32_t)f[6] | ((uint64_t)(uint32_t)f[7] << 32);
    }
    __device__ void begin_block(Top &t) { t.ent = (uint64_t)esp; }
    __device__ void end_block(const Top &t) { esp = (int64_t)t.ent; }
    __device__ bool add_entry(Top &t, bool trial)
    {
        int64_t b = (int64_t)t.ent + t.n_e;
        if (b >= max_bits) return false;
        uint32_t w = bits[b >> 5], m = 1u << (b & 31);
        bits[b >> 5] = trial ? (w | m) : (w & ~m);
        esp = b + 1;
        return true;
    }
    __device__ uint32_t entry_type(const Top &t, int32_t k)
    {
        int64_t b = (int64_t)t.ent + k;
        return ((bits[b >> 5] >> (b & 31)) & 1u) ? T_TRI : T_SUB;
    }
};

enum : uint32_t { S_START, S_BODY, S_P_OPEN, S_O_OPEN, S_ENTRY, S_E_DONE, S_O_DONE, S_W_DONE, S_TRAIL };

/* Pushdown automaton of the grammar, fed with tag events in position order.
 * Text runs are the gaps between consecutive event positions.  LENIENT:
 * PARASON_CFG_LENIENT_GAPS (a compile-time choice, so that the strict
 * automaton carries no code for it). */
template <class Store, bool LENIENT>
struct Automaton {
    Store st;
    int32_t prev;      /* position of the last token consumed */
    uint32_t state;
    int32_t acc;       /* latency of the current body (main or thread) */
    int32_t depth, n_blocks, max_depth;
    int32_t n_sub, n_tri;
    uint32_t ctx;      /* innermost enclosing thread's branch type */
    uint32_t open_tag; /* class of the open entry tag */
    int32_t entry_len; /* Text tokens of the open entry */
    int32_t err;       /* first error position, -1 while none */
    bool mismatch;
    bool overflow;     /* the store ran out: hand the row to the slow path */
    Top top;

    __device__ void init()
    {
        prev = -1;
        state = S_START;
        acc = 0;
        depth = n_blocks = max_depth = 0;
        n_sub = n_tri = 0;
        ctx = T_MAIN;
        open_tag = 0;
        entry_len = 0;
        err = -1;
        mismatch = false;
        overflow = false;
    }

    __device__ void attribute(int32_t n)
    {
        n_sub += ctx == T_SUB ? n : 0;
        n_tri += ctx == T_TRI ? n : 0;
    }

    /* n > 0 Text tokens at prev+1 .. prev+n.  Returns false on error. */
    __device__ bool text(int32_t n)
    {
        switch (state) {
        case S_BODY:
            acc += n;
            attribute(n);
            break;
        case S_ENTRY:
            top.block_main += n;
            entry_len += n;
            attribute(n);
            break;
        case S_TRAIL:
            acc += n;
            break;
        default:
            /* between structural tags of an open region (after <Parallel>,
             * <Outlines>, an entry, </Outlines> or a thread): when lenient a
             * gap, decoded by the enclosing path like the outline */
            if (!LENIENT || state == S_START) {
                err = prev + 1;
                return false;
            }
            top.block_main += n;
            attribute(n);
            break;
        }
        prev += n;
        return true;
    }

    __device__ bool fail(int32_t p)
    {
        err = p;
        return false;
    }

    __device__ void open_thread()
    {
        uint32_t t = top.k < top.n_e ? st.entry_type(top, top.k) : T_MAIN;
        ctx = t;
        acc = 1;
        attribute(1);
        state = S_BODY;
    }

    /* The tag of class c at position p (prev == p - 1).  False on error or
     * store overflow. */
    __device__ bool tag(int32_t p, uint32_t c)
    {
        switch (state) {
        case S_START:
            if (c != C_THINK) return fail(p);
            acc = 1;
            state = S_BODY;
            break;
        case S_BODY:
            if (c == C_PAR) {
                if (depth >= 1 && !st.push(top, depth)) {
                    overflow = true;
                    return false;
                }
                top.saved_acc = acc;
                top.block_main = 1;
                top.max_w = 0;
                top.n_e = 0;
                top.k = 0;
                top.saved_ctx = ctx;
                st.begin_block(top);
                depth += 1;
                n_blocks += 1;
                max_depth = max(max_depth, depth);
                attribute(1);
                state = S_P_OPEN;
            } else if (c == C_END_THINK && depth == 0) {
                acc += 1;
                state = S_TRAIL;
            } else if (c == C_END_THR && depth > 0) {
                acc += 1;
                attribute(1);
                top.max_w = max(top.max_w, acc);
                top.k += 1;
                ctx = top.saved_ctx;
                state = S_W_DONE;
            } else {
                return fail(p);
            }
            break;
        case S_P_OPEN:
            if (c != C_OUT) return fail(p);
            top.block_main += 1;
            attribute(1);
            state = S_O_OPEN;
            break;
        case S_O_OPEN:
        case S_E_DONE:
            if (c == C_SUB || c == C_TRI) {
                top.block_main += 1;
                attribute(1);
                open_tag = c;
                entry_len = 0;
                state = S_ENTRY;
            } else if (c == C_END_OUT && state == S_E_DONE) {
                top.block_main += 1;
                attribute(1);
                state = S_O_DONE;
            } else {
                return fail(p);
            }
            break;
        case S_ENTRY:
            if (entry_len == 0 || c != open_tag + 1) return fail(p);
            if (!st.add_entry(top, open_tag == C_TRI)) {
                overflow = true;
                return false;
            }
            top.n_e += 1;
            top.block_main += 1;
            attribute(1);
            state = S_E_DONE;
            break;
        case S_O_DONE:
        case S_W_DONE:
            if (c == C_THR) {
                open_thread();
            } else if (c == C_END_PAR && state == S_W_DONE) {
                if (top.k != top.n_e) mismatch = true;
                attribute(1);
                int32_t lat = top.block_main + top.max_w + 1;
                acc = top.saved_acc + lat;
                st.end_block(top);
                depth -= 1;
                if (depth >= 1) st.pop(top, depth);
                state = S_BODY;
            } else {
                return fail(p);
            }
            break;
        default: /* S_TRAIL: only Text may follow </think> */
            return fail(p);
        }
        prev = p;
        return true;
    }

    __device__ bool event(int32_t p, uint32_t c)
    {
        int32_t gap = p - prev - 1;
        if (gap > 0 && !text(gap)) return false;
        return tag(p, c);
    }

    /* End of the row (no error or overflow so far). */
    __device__ void finish(int32_t len)
    {
        int32_t gap = len - prev - 1;
        if (gap > 0 && !text(gap)) return;
        if (state != S_TRAIL) err = len;
    }
};

struct RowOut {
    int32_t *total, *latency, *n_subtask, *n_trial, *n_blocks, *max_depth, *first_error_pos;
    uint32_t *flags;
};

__device__ __forceinline__ void write_row(const RowOut &o, int64_t r, int32_t total, int32_t lat, int32_t ns,
                                          int32_t nt, int32_t nb, int32_t md, int32_t fe, uint32_t fl)
{
    o.total[r] = total;
    o.latency[r] = lat;
    o.n_subtask[r] = ns;
    o.n_trial[r] = nt;
    o.n_blocks[r] = nb;
    o.max_depth[r] = md;
    o.first_error_pos[r] = fe;
    o.flags[r] = fl;
}

template <class Store, bool LENIENT>
__device__ __forceinline__ void write_result(const RowOut &o, int64_t r, int32_t len, const Automaton<Store, LENIENT> &A)
{
    if (A.err < 0) {
        uint32_t fl = PARASON_FLAG_VALID;
        if (A.mismatch) fl |= PARASON_FLAG_COUNT_MISMATCH;
        if (A.n_blocks > 0) fl |= PARASON_FLAG_TRIGGERED;
        write_row(o, r, len, A.acc, A.n_sub, A.n_tri, A.n_blocks, A.max_depth, -1, fl);
    } else {
        write_row(o, r, len, len, 0, 0, 0, 0, A.err, A.err == len ? PARASON_FLAG_TRUNCATED : 0u);
    }
}

struct RowArgs {
    const int32_t *tok_base;
    int64_t mis;
    const int64_t *starts;
    const int32_t *lengths;
    int64_t n;
    const int64_t *seg_off;
    int64_t seg_cap;
    const SegRec *seg;
    const uint32_t *slots;
    int64_t deep_frames;    /* frames of the deep tier's store in workspace ... */
    int64_t deep_bits;      /* ... and its entry bits */
    TagMatch tm;
    RowOut out;
};

/* Feed row r's events to A.  Returns false when A stopped early.
 *
 * Three sources, all feeding the one call of A.event below: a compact list
 * (the whole row: seg[first], row positions), or per segment
 * its stored list (segment positions) or, for a segment marked DENSE, its
 * tokens classified again one by one.  Lists start at slots + seg[s].list.
 * With two inlined copies of the automaton (one per source) the
 * gfx950 build returned wrong results for dense segments although the same
 * source is correct when compiled for the CPU, so the sources are merged into
 * one fetch loop. */
template <class Store, bool LENIENT>
__device__ bool drive_row(const RowArgs &a, int64_t r, int64_t g, int32_t len, bool compact,
                          Automaton<Store, LENIENT> &A)
{
    const int64_t s0 = a.seg_off[r], s1 = a.seg_off[r + 1];
    const int64_t vrow0 = row_first_vec(g), vend = row_end_vec(g, len);
    int64_t s = s0;              /* next segment to open */
    const uint32_t *ev = nullptr;
    int32_t e = 0, cnt = 0;      /* stored-event cursor and list length */
    int64_t base = 0;            /* row position of stored position 0 */
    bool dense = false;
    int64_t q = 0, q_end = 0;    /* dense cursor (element index on the token grid) */
    uint4 quad = make_uint4(0u, 0u, 0u, 0u);
    if (compact) {
        const SegRec rec = a.seg[s0];
        ev = a.slots + rec.list;
        cnt = rec.count;
        s = s1;
    }
    for (;;) {
        int32_t p = 0;
        uint32_t c = 0;
        for (;;) {
            if (!dense && e < cnt) {
                /* lists start 16-byte aligned and take multiples of 4 slots:
                 * read them 16 bytes at a time */
                if ((e & 3) == 0) quad = *reinterpret_cast<const uint4 *>(ev + e);
                const uint32_t k = (uint32_t)e & 3u;
                const uint32_t w = k == 0 ? quad.x : k == 1 ? quad.y : k == 2 ? quad.z : quad.w;
                ++e;
                p = (int32_t)(base + (w >> 4));
                c = w & 15u;
                break;
            }
            if (dense) {
                while (q < q_end) {
                    const int32_t t = a.tok_base[q];
                    const int64_t pp = q - g;
                    ++q;
                    if (pp < 0 || pp >= len) continue;
                    c = classify(a.tm, t, a.tm.contiguous != 0);
                    if (c) {
                        p = (int32_t)pp;
                        break;
                    }
                }
                if (c) break;
                dense = false;
            }
            if (s >= s1) break;
            /* open segment s */
            const int64_t v0 = vrow0 + (s - s0) * SEG_VEC;
            const SegRec rec = a.seg[s];
            const int32_t n_s = rec.count;
            base = 4 * v0 - g;
            e = 0;
            if (n_s != DENSE) {
                cnt = n_s;
                ev = a.slots + rec.list; /* not read when n_s is 0 */
            } else {
                cnt = 0;
                dense = true;
                q = 4 * v0;
                q_end = 4 * min(v0 + (int64_t)SEG_VEC, vend);
            }
            ++s;
        }
        if (c == 0) break; /* no more events */
        if (!A.event(p, c)) return false;
    }
    return true;
}

/* Rows whose nesting or entry count exceeded the LDS stores, one after the
 * other, on the calling thread with frames in global workspace. */
template <bool LENIENT>
__device__ void run_deep_rows(const RowArgs &a, const uint8_t *__restrict__ mode, int32_t n_deep,
                              const int32_t *__restrict__ deep_rows, int32_t *__restrict__ frames,
                              uint32_t *__restrict__ bits)
{
    for (int32_t i = 0; i < n_deep; ++i) {
        const int64_t r = deep_rows[i];
        const int32_t len = a.lengths[r];
        Automaton<GlobalStore, LENIENT> A;
        A.st.frames = frames;
        A.st.bits = bits;
        A.st.max_frames = a.deep_frames;
        A.st.max_bits = a.deep_bits;
        A.st.esp = 0;
        A.init();
        if (drive_row(a, r, a.starts[r] + a.mis, len, (mode[r] & MODE_COMPACT) != 0, A)) A.finish(len);
        if (A.overflow)
            write_row(a.out, r, len, 0, 0, 0, 0, 0, 0, PARASON_FLAG_DEPTH_LIMIT);
        else
            write_result(a.out, r, len, A);
    }
}

/* ------------------------------------------------------------------ rows_par */

constexpr int PAR_EVENTS = 512; /* events of a row rows_par holds in LDS */
constexpr int PAR_LEVELS = 64;  /* nesting rows_par evaluates */
/* Levels up to which par_row takes no lists of a level's events.  A list costs a
 * pass over the row's events, the scans over them eight: 60,000 rows of 162 events
 * in one level 226 us a call without and 241 with lists, of 502 events 345 and 376;
 * 60,000 different rows of up to 10 levels 397 and 304, of up to 30 2,315 and 980,
 * 60,000 equal rows nested 30 deep 1,495 and 902. */
constexpr int PAR_DIRECT = 2;

/* The classes that may follow state st (one bit per class). */
constexpr uint32_t allowed_classes(uint32_t st)
{
    switch (st) {
    case S_START: return 1u << C_THINK;
    case S_BODY: return (1u << C_PAR) | (1u << C_END_THINK) | (1u << C_END_THR);
    case S_P_OPEN: return 1u << C_OUT;
    case S_O_OPEN: return (1u << C_SUB) | (1u << C_TRI);
    case S_ENTRY: return (1u << C_END_SUB) | (1u << C_END_TRI);
    case S_E_DONE: return (1u << C_SUB) | (1u << C_TRI) | (1u << C_END_OUT);
    case S_O_DONE: return 1u << C_THR;
    case S_W_DONE: return (1u << C_THR) | (1u << C_END_PAR);
    default: return 0u; /* S_TRAIL */
    }
}

/* The state after a tag of class c: the class alone decides it. */
constexpr uint32_t state_after(int32_t c)
{
    switch (c) {
    case C_THINK: return S_BODY;
    case C_END_THINK: return S_TRAIL;
    case C_PAR: return S_P_OPEN;
    case C_END_PAR: return S_BODY;
    case C_OUT: return S_O_OPEN;
    case C_END_OUT: return S_O_DONE;
    case C_SUB:
    case C_TRI: return S_ENTRY;
    case C_END_SUB:
    case C_END_TRI: return S_E_DONE;
    case C_THR: return S_BODY;
    default: return S_W_DONE; /* C_END_THR */
    }
}

/* The two functions above as bit tables, for lanes whose classes differ (a
 * switch there runs every case under an execution mask):
 *   state_at(pc)      the state after a tag of class pc, S_START for pc = -1
 *                     (the row's start): one nibble per pc + 1;
 *   class_allowed     bit 13 * st + c of a 128-bit table;
 *   text_allowed      Text may stand in state st (strict grammar). */
constexpr uint64_t state_table()
{
    uint64_t t = S_START;
    for (int32_t c = 0; c <= (int32_t)C_END_THR; ++c) t |= (uint64_t)state_after(c) << (4 * (c + 1));
    return t;
}
constexpr uint64_t allowed_table(int word)
{
    uint64_t t = 0;
    for (uint32_t st = S_START; st <= S_TRAIL; ++st)
        for (uint32_t c = 0; c <= C_END_THR; ++c) {
            const uint32_t bit = 13u * st + c;
            if ((allowed_classes(st) >> c) & 1u && bit / 64u == (uint32_t)word) t |= 1ull << (bit % 64u);
        }
    return t;
}
constexpr uint64_t STATE_TAB = state_table();
constexpr uint64_t ALLOWED_TAB0 = allowed_table(0), ALLOWED_TAB1 = allowed_table(1);
constexpr uint32_t TEXT_STATES = (1u << S_BODY) | (1u << S_TRAIL) | (1u << S_ENTRY);
static_assert(13u * S_TRAIL + C_END_THR < 128u, "the table holds every state and class");
static_assert(C_END_THR + 2 <= 16, "a nibble per class and the start");

__device__ __forceinline__ uint32_t state_at(int32_t pc) { return (uint32_t)(STATE_TAB >> (4 * (pc + 1))) & 15u; }
__device__ __forceinline__ bool class_allowed(uint32_t st, int32_t c)
{
    const uint32_t bit = 13u * st + (uint32_t)c;
    return ((bit < 64u ? ALLOWED_TAB0 : ALLOWED_TAB1) >> (bit & 63u)) & 1u;
}
__device__ __forceinline__ bool text_allowed(uint32_t st) { return (TEXT_STATES >> st) & 1u; }

/* Reductions over the wave, the result in every lane. */
__device__ __forceinline__ int32_t wave_sum32(int32_t v)
{
    return lane63(dpp_incl_scan<OpAdd>(v, (int)(threadIdx.x & (WAVE - 1))));
}
__device__ __forceinline__ int32_t wave_min32(int32_t v)
{
    return lane63(dpp_incl_scan<OpMin>(v, (int)(threadIdx.x & (WAVE - 1))));
}
__device__ __forceinline__ int32_t wave_max32(int32_t v)
{
    return lane63(dpp_incl_scan<OpMax>(v, (int)(threadIdx.x & (WAVE - 1))));
}

/* Events in passes of PAR_PASS: event i0 + PAR_K * lane + k is element k of
 * the lane, so a row of up to PAR_PASS events takes one wave scan per
 * quantity instead of one per 64 events (the scans are latency: a chain of
 * DPP steps and cross-row reads each). */
constexpr int PAR_K = 4;
constexpr int PAR_PASS = PAR_K * WAVE;
static_assert(PAR_EVENTS % PAR_PASS == 0, "passes end inside the LDS arrays");

template <int K>
__device__ __forceinline__ void par_load(const int32_t *s, int32_t ib, int32_t (&v)[K])
{
    if constexpr (K == 4) {
        const int4 x = *reinterpret_cast<const int4 *>(s + ib);
        v[0] = x.x;
        v[1] = x.y;
        v[2] = x.z;
        v[3] = x.w;
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = s[ib + k];
    }
}

template <int K>
__device__ __forceinline__ void par_store(int32_t *s, int32_t ib, const int32_t (&v)[K])
{
    if constexpr (K == 4) {
        *reinterpret_cast<int4 *>(s + ib) = make_int4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) s[ib + k] = v[k];
    }
}

template <int K>
__device__ __forceinline__ int32_t par_pick(const int32_t (&v)[K], int32_t k)
{
    int32_t x = v[0];
#pragma unroll
    for (int i = 1; i < K; ++i) x = k == i ? v[i] : x;
    return x;
}

/* Inclusive scan over the wave's events in order, continuing from carry. */
template <class Op, int K>
__device__ __forceinline__ void par_incl_scan(int32_t (&v)[K], int32_t carry, int lane)
{
#pragma unroll
    for (int k = 1; k < K; ++k) v[k] = Op::f(v[k - 1], v[k]);
    const int32_t before = Op::f(carry, lane_before(dpp_incl_scan<Op>(v[K - 1], lane), Op::ident));
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = Op::f(before, v[k]);
}

/* The heads of segmented scans over the wave's events: seen[k], a head among
 * the lane's events 0 .. k. */
template <int K>
struct ParHeads {
    bool head[K], seen[K];
    SegHeads lanes;
};

template <int K>
__device__ __forceinline__ ParHeads<K> par_heads(const bool (&head)[K])
{
    ParHeads<K> h;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        h.head[k] = head[k];
        h.seen[k] = k > 0 ? h.seen[k > 0 ? k - 1 : 0] | head[k] : head[k];
    }
    h.lanes = dpp_seg_heads(h.seen[K - 1]);
    return h;
}

/* Segmented form: restarts at events with head set; events before the first
 * head continue from carry. */
template <class Op, int K>
__device__ __forceinline__ void par_seg_scan(int32_t (&v)[K], const ParHeads<K> &h, int32_t carry, int lane)
{
#pragma unroll
    for (int k = 1; k < K; ++k)
        if (!h.head[k]) v[k] = Op::f(v[k - 1], v[k]);
    const int32_t in = lane_before(dpp_seg_scan<Op>(v[K - 1], h.lanes, carry, lane), carry);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool seen = h.seen[k];
        if (!seen) v[k] = Op::f(in, v[k]);
    }
}

/* In X and in rows_quad an event is its class and, for a structural tag of a
 * block (<Parallel>, </Outlines>, <Thread>, </Thread>, </Parallel>), that block's
 * level (1 = top level; 0 for other tags), so that one compare finds the tags of
 * a level.  depth: open blocks before the event. */
__device__ __forceinline__ int32_t par_word(uint32_t c, int32_t depth)
{
    constexpr uint32_t BLOCK_TAGS = 1u << C_PAR | 1u << C_END_OUT | 1u << C_THR | 1u << C_END_THR | 1u << C_END_PAR;
    const uint32_t own = (uint32_t)((int32_t)(BLOCK_TAGS << (31u - c)) >> 31); /* all ones for these, else 0 */
    const uint32_t lev = (uint32_t)depth + (c == C_PAR ? 1u : 0u);
    return (int32_t)(c | (lev & own & 0xfffu) << 4);
}
__device__ __forceinline__ int32_t par_tag(uint32_t c, int32_t lev) { return (int32_t)c + lev * 16; }

/* A level's list: the numbers of the events that are its tags, and, with
 * PAR_INNER, of the </Parallel> of the blocks directly inside it. */
constexpr uint32_t PAR_INNER = 1u << 15;
typedef uint16_t __attribute__((may_alias)) half_t;

/* The LDS of a wave that evaluates a row with its lanes over the row's events:
 * per event its position, its word (in the lower half of X; the upper halves
 * hold a level's list), and, while the levels are evaluated, at a </Parallel> its
 * block's saved tokens and the tokens of its threads.  Until phase A the last
 * two hold the map from event to segment of the split-row gather.  8 KB per wave,
 * so that 20 waves (rows) fit a compute unit; with a word per quantity (16 KB)
 * it was 10. */
struct ParLds {
    int32_t P[PAR_EVENTS];
    int32_t X[PAR_EVENTS];
    int32_t TOK[PAR_EVENTS];
    int32_t SAV[PAR_EVENTS];
    __device__ uint32_t entry(int32_t j) const { return reinterpret_cast<const half_t *>(X)[2 * j + 1]; }
    __device__ void set_entry(int32_t j, uint32_t v) { reinterpret_cast<half_t *>(X)[2 * j + 1] = (half_t)v; }
    __device__ int32_t pos(int32_t i) const { return P[i]; }
    __device__ uint32_t cls(int32_t i) const { return (uint32_t)X[i] & 15u; }
};
static_assert(PAR_EVENTS <= (int)PAR_INNER, "an event's number and the flag fit a half word");
static_assert(PAR_LEVELS + 1 < (1 << 12), "a level fits its field");
static_assert(PAR_EVENTS >= 2 * PAR_PASS, "the gather of a split row keeps two words per segment of a chunk in SAV");
static_assert(MID_DEPTH * FRAME_WORDS <= PAR_EVENTS, "the automaton's frames fit TOK");

/* What a lane has found of its row so far. */
struct ParSums {
    int32_t sub, tri, saved;
    bool mismatch;
};

/* The tags of one segment of the row at g, read again by the whole wave: the
 * vectors x (vector v0 + i * WAVE + lane), of which the positions inside the
 * row count, appended to sP and sX from event m on.  Returns the new count;
 * events past PAR_EVENTS are counted and not stored. */
__device__ __forceinline__ int32_t par_classify(const RowArgs &a, const int4 (&x)[LOADS], int32_t bias, int32_t len,
                                                ParLds &l, int32_t m, int lane)
{
    const bool contig = a.tm.contiguous != 0;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int32_t t[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
        const int32_t p0 = bias + 4 * (i * WAVE + lane); /* row position of the vector's first token */
        if (bias + 4 * i * WAVE >= len) break;           /* wave-uniform: a short row's other vectors */
        uint32_t c[4];
        uint64_t b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = (uint32_t)(p0 + j) < (uint32_t)len ? classify(a.tm, t[j], contig) : (uint32_t)C_TEXT;
            b[j] = __ballot(c[j] != C_TEXT);
        }
        if ((b[0] | b[1] | b[2] | b[3]) == 0) continue; /* wave-uniform */
        uint32_t at = (uint32_t)m;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[j], at));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (c[j] != C_TEXT) {
                if (at < (uint32_t)PAR_EVENTS) {
                    l.P[at] = p0 + j;
                    l.X[at] = (int32_t)c[j];
                }
                ++at;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) m += __popcll(b[j]);
    }
    return m;
}

/* The vectors of the row's k-th segment; lanes past the row's end get the
 * row's last vector (par_classify drops positions outside the row). */
__device__ __forceinline__ void par_load_segment(const RowArgs &a, int64_t vrow0, int64_t vend, int64_t k,
                                                 int4 (&x)[LOADS], int lane)
{
    const int4 *src = reinterpret_cast<const int4 *>(a.tok_base);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) x[i] = src[min(vrow0 + k * SEG_VEC + i * WAVE + lane, vend - 1)];
}

/* The widths of rows_quad (and of a small level in par_row): QUAD_W lanes (one DPP row) per row, QUAD_K
 * consecutive events per lane. */
constexpr int QUAD_W = 16;
constexpr int QUAD_K = 8;
constexpr int QUAD_ROWS = WAVE / QUAD_W;
constexpr int QUAD_EVENTS = QUAD_W * QUAD_K;

/* Scans over the QUAD_W lanes of a row stay inside a DPP row: four shifts and
 * no carries between rows of lanes. */
template <class Op>
__device__ __forceinline__ int32_t quad_lane_scan(int32_t v)
{
    v = Op::f(v, row_shr<1>(v, Op::ident));
    v = Op::f(v, row_shr<2>(v, Op::ident));
    v = Op::f(v, row_shr<4>(v, Op::ident));
    return Op::f(v, row_shr<8>(v, Op::ident));
}

/* Value of the row's last lane, in all of its lanes. */
__device__ __forceinline__ int32_t quad_last(int32_t v, int lane) { return __shfl(v, lane | (QUAD_W - 1), WAVE); }

/* Inclusive scan over a row's events in order, continuing from carry. */
template <class Op, int K>
__device__ __forceinline__ void quad_incl_scan(int32_t (&v)[K], int32_t carry = Op::ident)
{
#pragma unroll
    for (int k = 1; k < K; ++k) v[k] = Op::f(v[k - 1], v[k]);
    const int32_t before = Op::f(carry, row_shr<1>(quad_lane_scan<Op>(v[K - 1]), Op::ident));
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = Op::f(before, v[k]);
}

/* Segment heads of a row's events, shared by the segmented scans over the
 * same heads: seen[k], a head among the lane's events 0 .. k; at[i], a head in
 * the 2^i lanes up to this one; before, in any lane before it. */
template <int K>
struct QuadHeads {
    bool seen[K];
    bool at[4], before;
};

template <int K>
__device__ __forceinline__ QuadHeads<K> quad_heads(const bool (&head)[K])
{
    QuadHeads<K> h;
    h.seen[0] = head[0];
#pragma unroll
    for (int k = 1; k < K; ++k) h.seen[k] = h.seen[k - 1] | head[k];
    int32_t f = h.seen[K - 1] ? 1 : 0;
    h.at[0] = f != 0;
    f |= row_shr<1>(f, 0);
    h.at[1] = f != 0;
    f |= row_shr<2>(f, 0);
    h.at[2] = f != 0;
    f |= row_shr<4>(f, 0);
    h.at[3] = f != 0;
    f |= row_shr<8>(f, 0);
    h.before = row_shr<1>(f, 0) != 0;
    return h;
}

/* Segmented inclusive scan: restarts at heads; events before the first head
 * continue from carry.  Op::ident must be Op's identity on v. */
template <class Op, int K>
__device__ __forceinline__ void quad_seg_scan(int32_t (&v)[K], const bool (&head)[K], const QuadHeads<K> &h,
                                              int32_t carry = Op::ident)
{
#pragma unroll
    for (int k = 1; k < K; ++k) v[k] = head[k] ? v[k] : Op::f(v[k - 1], v[k]);
    int32_t t = v[K - 1];
    int32_t o = Op::f(row_shr<1>(t, Op::ident), t);
    t = h.at[0] ? t : o;
    o = Op::f(row_shr<2>(t, Op::ident), t);
    t = h.at[1] ? t : o;
    o = Op::f(row_shr<4>(t, Op::ident), t);
    t = h.at[2] ? t : o;
    o = Op::f(row_shr<8>(t, Op::ident), t);
    t = h.at[3] ? t : o;
    const int32_t prev = row_shr<1>(t, Op::ident), in = h.before ? prev : Op::f(carry, prev);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = h.seen[k] ? v[k] : Op::f(in, v[k]);
}

/* A row's LDS in rows_quad: its events (row position << 4 | class), a level's list
 * and, as in ParLds, what is kept at a </Parallel>. */
struct QuadLds {
    uint32_t ev[QUAD_EVENTS], list[QUAD_EVENTS];
    int32_t SAV[QUAD_EVENTS], TOK[QUAD_EVENTS];
    __device__ uint32_t entry(int32_t j) const { return list[j]; }
    __device__ void set_entry(int32_t j, uint32_t v) { list[j] = v; }
    __device__ int32_t pos(int32_t i) const { return (int32_t)(ev[i] >> 4); }
    __device__ uint32_t cls(int32_t i) const { return ev[i] & 15u; }
};
static_assert(QUAD_ROWS * sizeof(QuadLds) <= sizeof(ParLds), "rows_quad keeps its events in par_row's LDS");

/* One level of a row from its list of n entries, K consecutive ones per lane of a
 * DPP row, and with PASSES as many times that as a list of the wave needs: its threads (tokens, latency, own tokens), then, from
 * those values still in registers, its blocks (saved tokens, thread types, count
 * mismatch).  l16: the lane among the row's; LDS is QuadLds or ParLds. */
template <int K, bool PASSES, class Lds>
__device__ __forceinline__ void quad_level(Lds &l, int32_t n, bool top, int lane, int l16, ParSums &out)
{
    int32_t c_thr = -1, c_S = 0, c_CH = 0;
    int32_t c_sum = 0, c_max = 0, c_n = 0, c_par = -1, c_eout = -1;
    for (int32_t j0 = 0;; j0 += K * QUAD_W) {
        bool thr[K], ethr[K], par[K], epar[K];
        int32_t id[K], at[K], S[K], CH[K], pi[K], oi[K], pos[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t j = j0 + K * l16 + k;
            const uint32_t q = j < n ? l.entry(j) : 0u;
            const bool inner = (q & PAR_INNER) != 0;
            id[k] = (int32_t)(q & (PAR_INNER - 1u));
            const uint32_t c = j < n && !inner ? l.cls(id[k]) : 0u;
            pos[k] = l.pos(id[k]);
            thr[k] = c == C_THR;
            ethr[k] = c == C_END_THR;
            par[k] = c == C_PAR;
            epar[k] = c == C_END_PAR;
            at[k] = thr[k] ? pos[k] : -1;
            S[k] = inner ? l.SAV[id[k]] : 0;
            CH[k] = inner ? l.TOK[id[k]] : 0;
            pi[k] = par[k] ? id[k] : -1;
            oi[k] = c == C_END_OUT ? id[k] : -1;
        }
        quad_incl_scan<OpMax>(at, c_thr); /* where the thread each entry is in begins */
        const QuadHeads<K> ht = quad_heads(thr);
        quad_seg_scan<OpAdd>(S, thr, ht, c_S);
        quad_seg_scan<OpAdd>(CH, thr, ht, c_CH);
        quad_incl_scan<OpMax>(pi, c_par); /* the block each entry is in ... */
        quad_incl_scan<OpMax>(oi, c_eout); /* ... and its outline's end */
        int32_t sum[K], mx[K], nt[K], own[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t tok = ethr[k] ? pos[k] - at[k] + 1 : 0;
            sum[k] = tok;
            mx[k] = ethr[k] ? tok - S[k] : 0; /* the thread's latency */
            own[k] = tok - CH[k];             /* its own tokens */
            nt[k] = ethr[k] ? 1 : 0;
        }
        const QuadHeads<K> hp = quad_heads(par);
        quad_seg_scan<OpAdd>(sum, par, hp, c_sum);
        quad_seg_scan<OpMax>(mx, par, hp, c_max);
        quad_seg_scan<OpAdd>(nt, par, hp, c_n);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t n_e = (oi[k] - pi[k] - 2) / 2;
            if (ethr[k]) {
                const int32_t kk = nt[k] - 1; /* thread kk pairs with entry kk */
                if (kk < n_e) {
                    const uint32_t t = l.cls(pi[k] + 2 + 2 * kk);
                    out.sub += t == C_SUB ? own[k] : 0;
                    out.tri += t == C_TRI ? own[k] : 0;
                }
            }
            if (epar[k]) {
                const int32_t saved = sum[k] - mx[k];
                l.SAV[id[k]] = saved;
                l.TOK[id[k]] = sum[k];
                out.mismatch = out.mismatch || nt[k] != n_e;
                out.saved += top ? saved : 0;
            }
        }
        if (!PASSES || __ballot(n > j0 + K * QUAD_W) == 0) break;
        c_thr = quad_last(at[K - 1], lane);
        c_S = quad_last(S[K - 1], lane);
        c_CH = quad_last(CH[K - 1], lane);
        c_sum = quad_last(sum[K - 1], lane);
        c_max = quad_last(mx[K - 1], lane);
        c_n = quad_last(nt[K - 1], lane);
        c_par = quad_last(pi[K - 1], lane);
        c_eout = quad_last(oi[K - 1], lane);
    }
}

/* quad_level over the whole wave, in passes of K consecutive entries per lane. */
template <int K>
__device__ __forceinline__ void par_level(ParLds &l, int32_t n, bool top, int lane, ParSums &out)
{
    int32_t c_thr = -1, c_S = 0, c_CH = 0;
    int32_t c_sum = 0, c_max = 0, c_n = 0, c_par = -1, c_eout = -1;
    for (int32_t j0 = 0; j0 < n; j0 += K * WAVE) {
        bool thr[K], ethr[K], par[K], epar[K];
        int32_t id[K], at[K], S[K], CH[K], pi[K], oi[K], pos[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t j = j0 + K * lane + k;
            const uint32_t q = j < n ? l.entry(j) : 0u;
            const bool inner = (q & PAR_INNER) != 0;
            id[k] = (int32_t)(q & (PAR_INNER - 1u));
            const uint32_t c = j < n && !inner ? l.cls(id[k]) : 0u;
            pos[k] = l.pos(id[k]);
            thr[k] = c == C_THR;
            ethr[k] = c == C_END_THR;
            par[k] = c == C_PAR;
            epar[k] = c == C_END_PAR;
            at[k] = thr[k] ? pos[k] : -1;
            S[k] = inner ? l.SAV[id[k]] : 0;
            CH[k] = inner ? l.TOK[id[k]] : 0;
            pi[k] = par[k] ? id[k] : -1;
            oi[k] = c == C_END_OUT ? id[k] : -1;
        }
        par_incl_scan<OpMax>(at, c_thr, lane); /* where the thread each entry is in begins */
        const ParHeads<K> ht = par_heads(thr), hp = par_heads(par);
        par_seg_scan<OpAdd>(S, ht, c_S, lane);
        par_seg_scan<OpAdd>(CH, ht, c_CH, lane);
        par_incl_scan<OpMax>(pi, c_par, lane);  /* the block each entry is in ... */
        par_incl_scan<OpMax>(oi, c_eout, lane); /* ... and its outline's end */
        int32_t sum[K], mx[K], nt[K], own[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t tok = ethr[k] ? pos[k] - at[k] + 1 : 0;
            sum[k] = tok;
            mx[k] = ethr[k] ? tok - S[k] : 0; /* the thread's latency */
            own[k] = tok - CH[k];
            nt[k] = ethr[k] ? 1 : 0;
        }
        par_seg_scan<OpAdd>(sum, hp, c_sum, lane);
        par_seg_scan<OpMax>(mx, hp, c_max, lane);
        par_seg_scan<OpAdd>(nt, hp, c_n, lane);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t n_e = (oi[k] - pi[k] - 2) / 2;
            if (ethr[k]) {
                const int32_t kk = nt[k] - 1; /* thread kk pairs with entry kk */
                if (kk < n_e) {
                    const uint32_t t = l.cls(pi[k] + 2 + 2 * kk);
                    out.sub += t == C_SUB ? own[k] : 0;
                    out.tri += t == C_TRI ? own[k] : 0;
                }
            }
            if (epar[k]) {
                const int32_t saved = sum[k] - mx[k];
                l.SAV[id[k]] = saved;
                l.TOK[id[k]] = sum[k];
                out.mismatch = out.mismatch || nt[k] != n_e;
                out.saved += top ? saved : 0;
            }
        }
        if (n <= K * WAVE) break;
        c_thr = lane63(at[K - 1]);
        c_S = lane63(S[K - 1]);
        c_CH = lane63(CH[K - 1]);
        c_sum = lane63(sum[K - 1]);
        c_max = lane63(mx[K - 1]);
        c_n = lane63(nt[K - 1]);
        c_par = lane63(pi[K - 1]);
        c_eout = lane63(oi[K - 1]);
    }
}

/* The two phases of par_row on the row's m events in LDS, K consecutive events
 * per lane and pass; SINGLE: one pass holds them (the scans then carry nothing
 * in).  One event per lane for rows of up to 64 (four of five of the
 * generator's), two for up to 128 (99 of 100): a wave's steps per pass grow with
 * K (8,192 rows of 3,500 tokens: 22.4 us with K = 4 for every row, 17.7 with 2
 * and 4; 8 rows: 9.0 and 7.5). */
template <bool LENIENT, int K, bool SINGLE>
__device__ __forceinline__ bool par_eval(const RowArgs &a, ParLds &l, int64_t r, int32_t len, int32_t m, int lane)
{
    constexpr int PASS = K * WAVE;
    /* phase A: validity, first error, depth before each event */
    int32_t prev_c = -1, prev_p = -1, depth = 0, err = INT32_MAX, max_depth = 0, n_blocks = 0;
    for (int32_t i0 = 0; i0 < m && err == INT32_MAX; i0 += PASS) {
        const int32_t ib = i0 + K * lane;
        int32_t c[K], p[K], dd[K];
        par_load(l.X, ib, c);
        par_load(l.P, ib, p);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (ib + k >= m) c[k] = p[k] = 0;
            dd[k] = ib + k < m ? (c[k] == C_PAR) - (c[k] == C_END_PAR) : 0;
        }
        int32_t d_in[K]; /* depth after each event */
#pragma unroll
        for (int k = 0; k < K; ++k) d_in[k] = dd[k];
        par_incl_scan<OpAdd>(d_in, depth, lane);
        int32_t pc = lane_before(c[K - 1], prev_c), pp = lane_before(p[K - 1], prev_p);
        int32_t e = INT32_MAX, open_depth = 0, pars = 0;
        int32_t xv[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            /* the checks of one event, without branches (bitwise, not
             * short-circuit: lanes hold different classes) */
            const int32_t db = d_in[k] - dd[k];
            const int32_t ck = c[k];
            const bool act = ib + k < m;
            const uint32_t st = state_at(pc);
            const int32_t gap = p[k] - pp - 1;
            const bool text_ok = (gap == 0) | text_allowed(st) | (LENIENT & (st != S_START));
            const bool closes_entry = (ck == C_END_SUB) | (ck == C_END_TRI);
            const bool tag_ok = class_allowed(st, ck) & !((ck == C_END_THINK) & (db != 0)) &
                                !((ck == C_END_THR) & (db == 0)) & !(closes_entry & ((ck != pc + 1) | (gap == 0)));
            const int32_t ek = text_ok ? (tag_ok ? INT32_MAX : p[k]) : pp + 1;
            const bool opens = act & (ck == C_PAR);
            e = min(e, act ? ek : INT32_MAX);
            open_depth = max(open_depth, opens ? db + 1 : 0);
            pars += opens ? 1 : 0;
            xv[k] = par_word((uint32_t)ck, db);
            pc = c[k];
            pp = p[k];
        }
        par_store(l.X, ib, xv);
        err = wave_min32(e);
        max_depth = max(max_depth, wave_max32(open_depth));
        n_blocks += wave_sum32(pars);
        /* the pass's last event: the one before the next pass's first */
        const int32_t last = min(m - i0, PASS) - 1;
        prev_c = __builtin_amdgcn_readlane(par_pick(c, last % K), last / K);
        prev_p = __builtin_amdgcn_readlane(par_pick(p, last % K), last / K);
        if (SINGLE) break;
        depth = lane63(d_in[K - 1]);
    }
    if (err == INT32_MAX) {
        /* the end of the row: the text after the last tag, then </think> must have come */
        const uint32_t st = state_at(prev_c);
        const int32_t gap = len - prev_p - 1;
        const bool text_ok = gap == 0 || text_allowed(st) || (LENIENT && st != S_START);
        if (!text_ok) err = prev_p + 1;
        else if (st != S_TRAIL) err = len;
    }
    if (err != INT32_MAX) {
        if (lane == 0) write_row(a.out, r, len, len, 0, 0, 0, 0, err, err == len ? PARASON_FLAG_TRUNCATED : 0u);
        return true;
    }
    if (max_depth > PAR_LEVELS) return false;
    __syncthreads();

    /* phase B: level by level, deepest first */
    ParSums t{0, 0, 0, false};
    for (int32_t lev = max_depth; lev >= 1; --lev) {
        if (K == 1 || max_depth <= PAR_DIRECT) {
            /* all of the row's events, as in par_level */
            int32_t c_thr = -1, c_S = 0, c_CH = 0;
            int32_t c_sum = 0, c_max = 0, c_n = 0, c_par = -1, c_eout = -1;
            for (int32_t i0 = 0; i0 < m; i0 += PASS) {
                const int32_t ib = i0 + K * lane;
                int32_t x[K], sav[K], tk[K];
                par_load(l.X, ib, x);
                par_load(l.SAV, ib, sav);
                par_load(l.TOK, ib, tk);
                bool thr[K], ethr[K], par[K], epar[K];
                int32_t ti[K], S[K], CH[K], pi[K], oi[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    /* phase A left class 0 in the places of the last pass past m */
                    const int32_t w = x[k]; /* the upper halves are 0: no lists */
                    const bool inner = w == par_tag(C_END_PAR, lev + 1);
                    thr[k] = w == par_tag(C_THR, lev);
                    ethr[k] = w == par_tag(C_END_THR, lev);
                    par[k] = w == par_tag(C_PAR, lev);
                    epar[k] = w == par_tag(C_END_PAR, lev);
                    ti[k] = thr[k] ? ib + k : -1;
                    S[k] = inner ? sav[k] : 0;
                    CH[k] = inner ? tk[k] : 0;
                    pi[k] = par[k] ? ib + k : -1;
                    oi[k] = w == par_tag(C_END_OUT, lev) ? ib + k : -1;
                }
                par_incl_scan<OpMax>(ti, c_thr, lane); /* the thread each event is in */
                const ParHeads<K> ht = par_heads(thr), hp = par_heads(par);
                par_seg_scan<OpAdd>(S, ht, c_S, lane);
                par_seg_scan<OpAdd>(CH, ht, c_CH, lane);
                par_incl_scan<OpMax>(pi, c_par, lane); /* the block each event is in ... */
                par_incl_scan<OpMax>(oi, c_eout, lane); /* ... and its outline's end */
                int32_t sum[K], mx[K], nt[K], own[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int32_t tok = ethr[k] ? l.P[ib + k] - l.P[max(ti[k], 0)] + 1 : 0;
                    sum[k] = tok;
                    mx[k] = ethr[k] ? tok - S[k] : 0; /* the thread's latency */
                    own[k] = tok - CH[k];
                    nt[k] = ethr[k] ? 1 : 0;
                }
                par_seg_scan<OpAdd>(sum, hp, c_sum, lane);
                par_seg_scan<OpMax>(mx, hp, c_max, lane);
                par_seg_scan<OpAdd>(nt, hp, c_n, lane);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int32_t n_e = (oi[k] - pi[k] - 2) / 2;
                    if (ethr[k]) {
                        const int32_t kk = nt[k] - 1; /* thread kk pairs with entry kk */
                        if (kk < n_e) {
                            const int32_t ty = l.X[pi[k] + 2 + 2 * kk] & 15;
                            t.sub += ty == C_SUB ? own[k] : 0;
                            t.tri += ty == C_TRI ? own[k] : 0;
                        }
                    }
                    if (epar[k]) {
                        const int32_t saved = sum[k] - mx[k];
                        l.SAV[ib + k] = saved;
                        l.TOK[ib + k] = sum[k];
                        t.mismatch = t.mismatch || nt[k] != n_e;
                        t.saved += lev == 1 ? saved : 0;
                    }
                }
                if (SINGLE) break;
                c_thr = lane63(ti[K - 1]);
                c_S = lane63(S[K - 1]);
                c_CH = lane63(CH[K - 1]);
                c_sum = lane63(sum[K - 1]);
                c_max = lane63(mx[K - 1]);
                c_n = lane63(nt[K - 1]);
                c_par = lane63(pi[K - 1]);
                c_eout = lane63(oi[K - 1]);
            }
        } else {
            /* the level's events first, as a list, so that a level costs what it
             * holds and not what the row holds */
            int32_t n = 0;
            for (int32_t i0 = 0; i0 < m; i0 += PASS) {
                const int32_t ib = i0 + K * lane;
                int32_t x[K], cnt = 0;
                bool own[K], inner[K];
                par_load(l.X, ib, x);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    /* phase A left class 0 in the places of the last pass past m */
                    const int32_t w = x[k] & 0xffff;
                    own[k] = w >> 4 == lev;
                    inner[k] = w == par_tag(C_END_PAR, lev + 1);
                    cnt += (own[k] | inner[k]) ? 1 : 0;
                }
                const int32_t incl = dpp_incl_scan<OpAdd>(cnt, lane);
                int32_t j = n + incl - cnt;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (own[k] | inner[k]) l.set_entry(j++, (uint32_t)(ib + k) | (inner[k] ? PAR_INNER : 0u));
                n += lane63(incl);
            }
            __syncthreads();
            if (n <= QUAD_W) quad_level<1, false>(l, n, lev == 1, lane, lane, t); /* in the first DPP row */
            else if (n <= WAVE) par_level<1>(l, n, lev == 1, lane, t);
            else par_level<PAR_K>(l, n, lev == 1, lane, t);
        }
        __syncthreads();
    }
    const int32_t n_sub = wave_sum32(t.sub), n_tri = wave_sum32(t.tri), saved = wave_sum32(t.saved);
    const bool mismatch = __ballot(t.mismatch) != 0;
    if (lane == 0) {
        uint32_t fl = PARASON_FLAG_VALID;
        if (mismatch) fl |= PARASON_FLAG_COUNT_MISMATCH;
        if (n_blocks > 0) fl |= PARASON_FLAG_TRIGGERED;
        write_row(a.out, r, len, len - saved, n_sub, n_tri, n_blocks, max_depth, -1, fl);
    }
    return true;
}

/* One row by one wave, its lanes over the row's events, up to four consecutive
 * events per lane and pass.  The same results as the automaton, from the
 * structure of the grammar:
 *   - the state before a tag is fixed by the class of the tag before it, and
 *     the nesting depth before it is a prefix sum, so every check of the
 *     automaton is local to an event and its predecessor; the row's first
 *     error is the smallest error position over the events (phase A);
 *   - for a valid row, with saved(P) = sum_k tokens(W_k) - max_k lat(W_k)
 *     over the threads W_k of block P, and lat(W) = tokens(W) - the saved
 *     tokens of the blocks directly inside W, the latency is the row's
 *     length less the saved tokens of its top-level blocks; a thread's own
 *     tokens (its tokens less those of the threads nested in it) take the
 *     type of the outline entry it pairs with.  Evaluated level by level,
 *     deepest first, with segmented scans (phase B): over the row's events where
 *     it has few levels, else over a list of the level's own.
 * Returns false, with nothing written, for a row of more than PAR_EVENTS
 * events or nested deeper than PAR_LEVELS.  Split rows are read from their
 * segments' lists directly, and a segment whose list the scan could not store
 * is read again by the wave (par_classify): for one lane alone those rows'
 * tokens are a chain of loads that held up a whole batch (the row kernel of
 * 8,192 rows of 3,500 tokens, whose outlines overflow a few of the scan's pool
 * regions: 372 us, 24 us read by the wave). */
template <bool LENIENT>
__device__ bool par_row(const RowArgs &a, ParLds &l, int64_t r, int64_t start, int32_t len, int64_t s0, int64_t s1,
                        bool compact, int lane)
{
    /* the row's events into LDS, in position order: from its compact list (row
     * positions), or gathered from its segments' lists (segment positions) */
    const int64_t g = start + a.mis;
    int32_t m = 0;
    bool held = true;
    if (compact) {
        const SegRec rec = a.seg[s0];
        m = rec.count;
        held = m <= PAR_EVENTS;
        const uint32_t *list = a.slots + rec.list;
        for (int32_t i0 = 0; held && i0 < m; i0 += 4 * WAVE) { /* four loads per lane in flight */
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t i = i0 + u * WAVE + lane;
                w[u] = i < m ? list[i] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t i = i0 + u * WAVE + lane;
                if (i < m) {
                    l.P[i] = (int32_t)(w[u] >> 4);
                    l.X[i] = (int32_t)(w[u] & 15u);
                }
            }
        }
    } else {
        /* PAR_PASS segments at a time, four per lane: their records in one
         * round of loads and an exclusive scan of their counts; then an LDS
         * map from event to segment (each segment that holds events marks its
         * first event, a running maximum spreads the marks) and the events'
         * loads in one round per PAR_PASS events.  A chunk ends at the first
         * DENSE segment; a run of DENSE segments at its start is read again. */
        const int64_t vrow0 = row_first_vec(g), vend = row_end_vec(g, len);
        int32_t *map = l.TOK, *seg_list = l.SAV, *seg_first = l.SAV + PAR_PASS;
        for (int64_t c0 = s0; held && c0 < s1;) {
            const int32_t jb = PAR_K * lane; /* the chunk's segment of element 0 */
            const int32_t n_c = (int32_t)min((int64_t)PAR_PASS, s1 - c0);
            int32_t cnt[PAR_K], lst[PAR_K], incl[PAR_K];
            int32_t dense0 = n_c, stored0 = n_c; /* the lane's first DENSE segment, and its first other one */
#pragma unroll
            for (int k = 0; k < PAR_K; ++k) {
                const int64_t s = c0 + jb + k;
                const SegRec rec = s < s1 ? a.seg[s] : SegRec{0, 0u};
                cnt[k] = rec.count;
                lst[k] = (int32_t)rec.list; /* meaningless for a segment without events */
            }
#pragma unroll
            for (int k = PAR_K - 1; k >= 0; --k) {
                if (cnt[k] == DENSE) dense0 = min(dense0, jb + k);
                else stored0 = min(stored0, jb + k);
            }
            const int32_t n_stored = wave_min32(dense0);
            if (n_stored == 0) {
                const int32_t n_dense = wave_min32(stored0);
                for (int32_t k = 0; k < n_dense; ++k) {
                    int4 x[LOADS];
                    par_load_segment(a, vrow0, vend, c0 - s0 + k, x, lane);
                    m = par_classify(a, x, (int32_t)(4 * (vrow0 + (c0 - s0 + k) * SEG_VEC) - g), len, l, m, lane);
                }
                held = m <= PAR_EVENTS;
                c0 += n_dense;
                continue;
            }
#pragma unroll
            for (int k = 0; k < PAR_K; ++k) {
                if (jb + k >= n_stored) cnt[k] = 0;
                incl[k] = cnt[k];
            }
            par_incl_scan<OpAdd>(incl, 0, lane);
            const int32_t total = lane63(incl[PAR_K - 1]);
            const int64_t chunk = c0;
            c0 += n_stored;
            held = m + total <= PAR_EVENTS;
            if (!held || total == 0) continue;
            const int32_t none[PAR_K] = {-1, -1, -1, -1};
            for (int32_t f0 = 0; f0 < total; f0 += PAR_PASS) par_store(map, f0 + jb, none);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PAR_K; ++k) {
                if (cnt[k] > 0) {
                    const int32_t e0 = incl[k] - cnt[k];
                    map[e0] = jb + k;
                    seg_list[jb + k] = lst[k];
                    seg_first[jb + k] = e0;
                }
            }
            __syncthreads();
            int32_t carry = -1;
            for (int32_t f0 = 0; f0 < total; f0 += PAR_PASS) {
                int32_t j[PAR_K];
                uint32_t w[PAR_K];
                par_load(map, f0 + jb, j);
                par_incl_scan<OpMax>(j, carry, lane); /* every event's segment (position 0 is marked) */
#pragma unroll
                for (int k = 0; k < PAR_K; ++k) {
                    const int32_t f = f0 + jb + k, jj = max(j[k], 0);
                    w[k] = f < total ? a.slots[(int64_t)(uint32_t)seg_list[jj] + (f - seg_first[jj])] : 0u;
                }
#pragma unroll
                for (int k = 0; k < PAR_K; ++k) {
                    const int32_t f = f0 + jb + k;
                    if (f < total) {
                        const int64_t seg = chunk + j[k];
                        l.P[m + f] = (int32_t)(4 * (vrow0 + (seg - s0) * SEG_VEC) - g + (int64_t)(w[k] >> 4));
                        l.X[m + f] = (int32_t)(w[k] & 15u);
                    }
                }
                carry = lane63(j[PAR_K - 1]);
            }
            __syncthreads(); /* the next chunk rewrites the map */
            m += total;
        }
    }
    if (!held) return false;
    __syncthreads();
    if (m <= WAVE) return par_eval<LENIENT, 1, true>(a, l, r, len, m, lane);
    if (m <= 2 * WAVE) return par_eval<LENIENT, 2, true>(a, l, r, len, m, lane);
    return par_eval<LENIENT, PAR_K, false>(a, l, r, len, m, lane);
}

/* One wave per row (a small batch).  A row par_row does not hold runs through
 * the automaton on lane 0 (the single automaton call site of this kernel),
 * with MID_DEPTH frames in LDS; one that needs still more is listed for the deep
 * tier. */
template <bool LENIENT>
__global__ void __launch_bounds__(64) rows_par(RowArgs a, uint8_t *__restrict__ mode,
                                               int32_t *__restrict__ counters, int32_t *__restrict__ deep_rows)
{
    __shared__ __align__(16) ParLds l;
    const int lane = threadIdx.x;
    const int64_t r = blockIdx.x;
    if (r >= a.n) return;
    /* the row's records in one round of loads, before any branch */
    const int64_t start = a.starts[r];
    const int32_t len = a.lengths[r];
    const int64_t S = a.seg_off[a.n], s0 = a.seg_off[r], s1 = a.seg_off[r + 1];
    const uint8_t md = mode[r];
    if (start < 0 || len < 0) {
        if (lane == 0) write_row(a.out, r, 0, 0, 0, 0, 0, 0, 0, PARASON_FLAG_BAD_ROW);
        return;
    }
    if (S > a.seg_cap) {
        if (lane == 0) write_row(a.out, r, len, 0, 0, 0, 0, 0, 0, PARASON_FLAG_WS_OVERFLOW);
        return;
    }
    if (par_row<LENIENT>(a, l, r, start, len, s0, s1, (md & MODE_COMPACT) != 0, lane)) return;
    if (lane == 0) {
        Automaton<LdsStore, LENIENT> A;
        A.st.lds = l.TOK; /* unused on this path */
        A.st.tid = 0;
        A.st.nt = 1;
        A.st.depth = MID_DEPTH;
        A.init();
        if (drive_row(a, r, start + a.mis, len, (md & MODE_COMPACT) != 0, A)) A.finish(len);
        if (A.overflow) {
            mode[r] = md | MODE_DEEP;
            deep_rows[atomicAdd(&counters[1], 1)] = (int32_t)r;
        } else {
            write_result(a.out, r, len, A);
        }
    }
}

/* ------------------------------------------------------------------ rows_quad */

/* The two phases of rows_quad on the m events of each of the wave's four rows (0
 * where not held), K consecutive events per lane, and the outputs of held rows. */
template <bool LENIENT, int K>
__device__ __forceinline__ void quad_eval(const RowArgs &a, QuadLds &l, int64_t r, int32_t len, int32_t m, bool held,
                                          int lane)
{
    const int l16 = lane & (QUAD_W - 1);
    /* phase A: validity, first error, depth before each event */
    const int32_t ib = K * l16;
    uint32_t e[K];
    int32_t word[K], d_in[K], dd[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        e[k] = ib + k < m ? l.ev[ib + k] : 0u;
        const uint32_t c = e[k] & 15u;
        dd[k] = (c == C_PAR ? 1 : 0) - (c == C_END_PAR ? 1 : 0);
        d_in[k] = dd[k];
    }
    quad_incl_scan<OpAdd>(d_in);
    int32_t err = INT32_MAX, max_depth = 0, n_blocks = 0;
    {
        /* -1 before the first event: a class before </think> and a position */
        const uint32_t e_prev = (uint32_t)row_shr<1>((int32_t)e[K - 1], -1);
        int32_t pc = l16 == 0 ? -1 : (int32_t)(e_prev & 15u), pp = l16 == 0 ? -1 : (int32_t)(e_prev >> 4);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t db = d_in[k] - dd[k];
            const int32_t ck = (int32_t)(e[k] & 15u), p = (int32_t)(e[k] >> 4);
            const bool act = ib + k < m;
            const uint32_t st = state_at(pc);
            const int32_t gap = p - pp - 1;
            const bool text_ok = (gap == 0) | text_allowed(st) | (LENIENT & (st != S_START));
            const bool closes_entry = (ck == C_END_SUB) | (ck == C_END_TRI);
            const bool tag_ok = class_allowed(st, ck) & !((ck == C_END_THINK) & (db != 0)) &
                                !((ck == C_END_THR) & (db == 0)) & !(closes_entry & ((ck != pc + 1) | (gap == 0)));
            const int32_t ek = text_ok ? (tag_ok ? INT32_MAX : p) : pp + 1;
            const bool opens = act & (ck == C_PAR);
            err = min(err, act ? ek : INT32_MAX);
            max_depth = max(max_depth, opens ? db + 1 : 0);
            n_blocks += opens ? 1 : 0;
            word[k] = par_word((uint32_t)ck, db);
            pc = ck;
            pp = p;
        }
    }
    err = quad_last(quad_lane_scan<OpMin>(err), lane);
    max_depth = quad_last(quad_lane_scan<OpMax>(max_depth), lane);
    n_blocks = quad_last(quad_lane_scan<OpAdd>(n_blocks), lane);
    if (held && err == INT32_MAX) {
        /* the end of the row: the text after the last tag, then </think> must have come */
        const uint32_t e_last = m > 0 ? l.ev[m - 1] : 0u;
        const int32_t pc = m > 0 ? (int32_t)(e_last & 15u) : -1, pp = m > 0 ? (int32_t)(e_last >> 4) : -1;
        const uint32_t st = state_at(pc);
        const int32_t gap = len - pp - 1;
        const bool text_ok = gap == 0 || text_allowed(st) || (LENIENT && st != S_START);
        if (!text_ok) err = pp + 1;
        else if (st != S_TRAIL) err = len;
    }
    const bool valid = held && err == INT32_MAX;
    if (!valid) {
#pragma unroll
        for (int k = 0; k < K; ++k) word[k] = 0; /* no structural tag of any level */
        max_depth = 0;
    }

    /* phase B: level by level, deepest first, as many as the wave's deepest row
     * has; the level's events as a list first, so that a level costs what it holds
     * and not what the row holds */
    ParSums t{0, 0, 0, false};
    for (int32_t lev = wave_max32(max_depth); lev >= 1; --lev) {
        bool own[K], inner[K];
        int32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            own[k] = word[k] >> 4 == lev;
            inner[k] = word[k] == par_tag(C_END_PAR, lev + 1);
            cnt += (own[k] | inner[k]) ? 1 : 0;
        }
        const int32_t incl = quad_lane_scan<OpAdd>(cnt);
        int32_t j = incl - cnt;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (own[k] | inner[k]) l.set_entry(j++, (uint32_t)(ib + k) | (inner[k] ? PAR_INNER : 0u));
        const int32_t n = quad_last(incl, lane);
        __syncthreads();
        if (K == 1 || __ballot(n > QUAD_W) == 0) quad_level<1, false>(l, n, lev == 1, lane, l16, t);
        else if (K == 2 || __ballot(n > 2 * QUAD_W) == 0) quad_level<2, false>(l, n, lev == 1, lane, l16, t);
        else quad_level<4, (K > 4)>(l, n, lev == 1, lane, l16, t);
        __syncthreads();
    }
    const int32_t n_sub = quad_last(quad_lane_scan<OpAdd>(t.sub), lane);
    const int32_t n_tri = quad_last(quad_lane_scan<OpAdd>(t.tri), lane);
    const int32_t saved = quad_last(quad_lane_scan<OpAdd>(t.saved), lane);
    const bool mismatch = ((uint32_t)(__ballot(t.mismatch) >> (lane & ~(QUAD_W - 1))) & 0xffffu) != 0;
    if (held && l16 == 0) {
        if (valid) {
            uint32_t fl = PARASON_FLAG_VALID;
            if (mismatch) fl |= PARASON_FLAG_COUNT_MISMATCH;
            if (n_blocks > 0) fl |= PARASON_FLAG_TRIGGERED;
            write_row(a.out, r, len, len - saved, n_sub, n_tri, n_blocks, max_depth, -1, fl);
        } else {
            write_row(a.out, r, len, len, 0, 0, 0, 0, err, err == len ? PARASON_FLAG_TRUNCATED : 0u);
        }
    }
}

/* A larger batch: four rows per wave, sixteen lanes per row, as many consecutive
 * events per lane (1, 2, 4 or 8) as the fullest of the four rows needs, up to
 * QUAD_EVENTS a row (99 of 100 of the generator's; the median row holds 38).
 * The same two phases as par_row, without phase A's passes.  It is bound by
 * instructions and, at few events per lane, by the latency of a wave's chain of
 * loads: par_row spends a wave's instructions on one row, whose events fill a
 * sixth of its 256 places, and the per-lane automaton's lanes wait for each other
 * in most of its states.  64,000 rows of 20,000 tokens: 48-60 us, one wave per
 * row 124, one lane per row 219; 712,000 rows: 352 us, 1,266, 644.  With eight
 * events per lane for every row, and up to eight of a level's, it took 133 vector
 * registers (three waves per SIMD) and 65-73 and 589 us; levels of at most four
 * entries per lane and pass leave 96, so that the five waves the LDS has room for
 * fit (2,000,000 rows of two to four tokens 1,532 us a call, 1,274 so, 1,053 with
 * one lane per row).
 * Rows it does not hold (more events, a segment the scan could not store) are
 * evaluated one after the other by the whole wave (par_row); one that par_row
 * does not hold either is listed for rows_listed. */
template <bool LENIENT>
__global__ void __launch_bounds__(64, 5) rows_quad(RowArgs a, const uint8_t *__restrict__ mode,
                                                int32_t *__restrict__ counters, int32_t *__restrict__ listed)
{
    __shared__ __align__(16) ParLds l;
    const int lane = threadIdx.x, l16 = lane & (QUAD_W - 1);
    QuadLds &ql = reinterpret_cast<QuadLds *>(&l)[lane / QUAD_W];
    const int64_t r0 = (int64_t)blockIdx.x * QUAD_ROWS;
    const int64_t r = min(r0 + lane / QUAD_W, a.n - 1);
    /* the row's records in one round of loads, before any branch */
    const int64_t start = a.starts[r];
    const int32_t len = a.lengths[r];
    const int64_t S = a.seg_off[a.n], s0 = a.seg_off[r], s1 = a.seg_off[r + 1];
    const bool compact = (mode[r] & MODE_COMPACT) != 0;
    const bool bad = start < 0 || len < 0;
    const bool over = S > a.seg_cap;
    const bool mine = r0 + lane / QUAD_W < a.n; /* the last wave's lanes past the batch repeat its last row */
    const bool eval = mine && !bad && !over;
    if (mine && !eval && l16 == 0) {
        if (bad) write_row(a.out, r, 0, 0, 0, 0, 0, 0, 0, PARASON_FLAG_BAD_ROW);
        else write_row(a.out, r, len, 0, 0, 0, 0, 0, 0, PARASON_FLAG_WS_OVERFLOW);
    }
    /* the row's m events into its LDS */
    const int64_t g = start + a.mis;
    int32_t m = 0;
    bool held = eval;
    const bool has_list = eval && compact;
    uint32_t first_slot = 0;
    if (has_list) {
        const SegRec rec = a.seg[s0];
        m = rec.count;
        held = m <= QUAD_EVENTS;
        first_slot = held && m > 0 ? rec.list : 0u;
    }
    if (held && has_list && 4 * l16 < m) {
        /* whole quads of four slots, as they are stored, a quad of the list's
         * first half and one of its second per lane */
        const uint4 *list = reinterpret_cast<const uint4 *>(a.slots + first_slot);
        const int32_t q1 = l16 + QUAD_W;
        const uint4 x = list[l16], y = 4 * q1 < m ? list[q1] : make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4 *>(ql.ev)[l16] = x;
        if (4 * q1 < m) reinterpret_cast<uint4 *>(ql.ev)[q1] = y;
    }
    const bool split = eval && !compact;
    held = held && (!split || len < (1 << 27));
    if (__ballot(split && held) != 0) {
        /* sixteen segments at a time: their records, an exclusive scan of
         * their counts, then every lane copies its segment's list */
        const int64_t vrow0 = row_first_vec(g);
        for (int64_t c0 = s0; __ballot(split && held && c0 < s1) != 0; c0 += QUAD_W) {
            const int64_t s = c0 + l16;
            const bool in = split && held && s < s1;
            const SegRec rec = in ? a.seg[s] : SegRec{0, 0u};
            const uint32_t dense = (uint32_t)(__ballot(rec.count == DENSE) >> (lane & ~(QUAD_W - 1))) & 0xffffu;
            const int32_t cnt = dense != 0 ? 0 : rec.count;
            const int32_t incl = quad_lane_scan<OpAdd>(cnt);
            const int32_t total = quad_last(incl, lane);
            held = held && dense == 0 && m + total <= QUAD_EVENTS;
            if (held && cnt > 0) {
                const int32_t base = (int32_t)(4 * (vrow0 + (s - s0) * SEG_VEC) - g);
                const uint4 *list = reinterpret_cast<const uint4 *>(a.slots + rec.list);
                uint32_t *dst = ql.ev + m + incl - cnt;
                const int32_t last = (cnt - 1) / 4;
                for (int32_t q = 0; q <= last; q += 2) { /* two quads in flight */
                    const uint4 x = list[q], y = list[min(q + 1, last)];
                    const uint32_t w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (4 * q + u < cnt)
                            dst[4 * q + u] = (uint32_t)(base + (int32_t)(w[u] >> 4)) << 4 | (w[u] & 15u);
                }
            }
            m += held ? total : 0;
        }
    }
    if (!held) m = 0;
    __syncthreads();

    /* as many events per lane as the fullest of the four rows has */
    if (__ballot(m > QUAD_W) == 0) quad_eval<LENIENT, 1>(a, ql, r, len, m, held, lane);
    else if (__ballot(m > 2 * QUAD_W) == 0) quad_eval<LENIENT, 2>(a, ql, r, len, m, held, lane);
    else if (__ballot(m > 4 * QUAD_W) == 0) quad_eval<LENIENT, 4>(a, ql, r, len, m, held, lane);
    else quad_eval<LENIENT, QUAD_K>(a, ql, r, len, m, held, lane);
    uint64_t todo = __ballot(eval && !held && l16 == 0);
    while (todo != 0) {
        __syncthreads(); /* the LDS is rewritten */
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int64_t rd = r0 + src / QUAD_W;
        const int64_t st = uniform64(a.starts[rd]), f0 = uniform64(a.seg_off[rd]), f1 = uniform64(a.seg_off[rd + 1]);
        const int32_t ln = __builtin_amdgcn_readfirstlane(a.lengths[rd]);
        const bool cp = __builtin_amdgcn_readfirstlane(mode[rd] & MODE_COMPACT) != 0;
        if (!par_row<LENIENT>(a, l, rd, st, ln, f0, f1, cp, lane) && lane == 0)
            listed[atomicAdd(&counters[0], 1)] = (int32_t)rd;
    }
}

/* The rows rows_quad listed (more than PAR_EVENTS events, or nested deeper than
 * PAR_LEVELS), by the automaton, one thread each, 64 at a time per wave: with
 * FAST_DEPTH frames per row, so that the LDS leaves room for the waves that
 * hide the latency of the branchy automaton; then those that need more frames
 * (or more than 64 entries in an open block), MID_ROWS at a time with
 * MID_DEPTH frames in the same LDS.  A row that needs still more is listed for
 * the deep tier. */
constexpr int MID_ROWS = FAST_DEPTH * WAVE / MID_DEPTH;
static_assert(MID_ROWS >= 1, "a deeper row fits the frames of a wave's rows");

template <bool LENIENT>
__global__ void __launch_bounds__(64) rows_listed(RowArgs a, uint8_t *__restrict__ mode, int32_t *__restrict__ counters,
                                                  const int32_t *__restrict__ listed, int32_t *__restrict__ deep_rows)
{
    __shared__ int32_t lds[FAST_DEPTH * FRAME_WORDS * WAVE];
    const int lane = threadIdx.x;
    const int32_t n_listed = counters[0];
    for (int32_t i0 = (int32_t)blockIdx.x * WAVE; i0 < n_listed; i0 += (int32_t)gridDim.x * WAVE) {
        uint64_t todo = ~0ull; /* the rows of this turn's lanes still to evaluate */
        bool deeper = false;
        while (todo != 0) {
            __syncthreads(); /* the frames' layout changes */
            /* every lane's row, or the next MID_ROWS of those that need more frames, in lanes 0, 1, ... */
            int src = lane;
            bool mine = i0 + lane < n_listed;
            if (deeper) {
                uint64_t t = todo;
                for (int k = 0; k < lane && k < MID_ROWS; ++k) t &= t - 1;
                mine = lane < MID_ROWS && t != 0;
                src = mine ? __builtin_ctzll(t) : 0;
                for (int k = 0; k < MID_ROWS; ++k) todo &= todo - 1;
            }
            bool again = false;
            if (mine) {
                const int64_t r = listed[i0 + src];
                const int32_t len = a.lengths[r];
                Automaton<LdsStore, LENIENT> A;
                A.st.lds = lds;
                A.st.tid = lane;
                A.st.nt = deeper ? MID_ROWS : WAVE;
                A.st.depth = deeper ? MID_DEPTH : FAST_DEPTH;
                A.init();
                if (drive_row(a, r, a.starts[r] + a.mis, len, (mode[r] & MODE_COMPACT) != 0, A)) A.finish(len);
                if (!A.overflow) {
                    write_result(a.out, r, len, A);
                } else if (deeper) {
                    mode[r] |= MODE_DEEP;
                    deep_rows[atomicAdd(&counters[1], 1)] = (int32_t)r;
                } else {
                    again = true;
                }
            }
            if (!deeper) {
                todo = __ballot(again);
                deeper = true;
            }
        }
    }
}

/* ------------------------------------------------------------------ scan */

typedef int v4i __attribute__((ext_vector_type(4)));

/* 16-byte streaming load (each token is read exactly once). */
__device__ __forceinline__ int4 load_vec(const int4 *p)
{
    v4i v = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(p));
    return make_int4(v.x, v.y, v.z, v.w);
}

/* Tag tests of the token scan: contiguous ids (a range check), hashed ids (one
 * lookup in the slot table held across the wave's lanes, tab = slot_id[lane])
 * or, for tag sets no shift pair separates, twelve compares. */
enum : int { TM_CONTIG = 0, TM_HASH = 1, TM_LINEAR = 2 };

template <int MODE>
__device__ __forceinline__ bool is_tag(const TagMatch &tm, int32_t t, int32_t tab)
{
    if (MODE == TM_CONTIG) return (uint32_t)t - (uint32_t)tm.base < 12u;
    if (MODE == TM_HASH) return __builtin_amdgcn_ds_bpermute((int)(tag_slot(tm, t) << 2), tab) == t;
    bool h = false;
#pragma unroll
    for (int k = 0; k < 12; ++k) h = h || (t == tm.ids[k]);
    return h;
}

/* The class of a token known to be a tag: for contiguous ids one shift of
 * the 64-bit nibble table (the id is base + o with o < 12). */
template <int MODE>
__device__ __forceinline__ uint32_t tag_class(const TagMatch &tm, int32_t t)
{
    if (MODE == TM_CONTIG) {
        const uint64_t lut = (uint64_t)tm.lut_hi << 32 | tm.lut_lo;
        return (uint32_t)(lut >> (4u * ((uint32_t)t - (uint32_t)tm.base))) & 15u;
    }
    return classify(tm, t, false);
}

/* For hashed ids, the class the slot's lane holds (tab_class = the class of
 * slot_id[lane]); every lane must call it, and only a tag's lane gets its
 * class.  With twelve compares per token column instead, 8,192 rows of 3,500
 * tokens took 75 us a call, 65 so. */
__device__ __forceinline__ uint32_t slot_class(const TagMatch &tm, int32_t t, int32_t tab_class)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(tag_slot(tm, t) << 2), tab_class);
}

/* Tags of the LOADS vectors x[i] (vector v0 + i*WAVE + lane of this lane) are
 * appended to dst[0 .. cap) in position order as (q + bias) << 4 | class, where
 * q = 4*(i*WAVE + lane) + j is the position in the segment; cnt counts all of
 * them, stored or not.  EDGE: the segment holds the first or last vector of its
 * row, so only positions q_lo <= q < q_hi belong to the row. */
template <int MODE, bool EDGE>
__device__ __forceinline__ void scan_vectors(const int4 (&x)[LOADS], int32_t q_lo, int32_t q_hi,
                                             uint32_t *__restrict__ dst, uint32_t cap, int32_t bias, uint32_t &cnt,
                                             const TagMatch &tm, int32_t tab, int32_t tab_class, int lane)
{
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int32_t t[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
        if (MODE == TM_CONTIG) {
            /* Contiguous ids are base .. base + 11 with base >= 0: a vector
             * holds a tag only if its largest (signed) token reaches base.
             * Three VALU operations per lane instead of eight settle the
             * vectors without a tag (about four in five at 0.1 % tags). */
            const int32_t hi = max(max(t[0], t[1]), max(t[2], t[3]));
            if (__ballot(hi >= tm.base) == 0) continue; /* wave-uniform */
        }
        const int32_t q0 = 4 * (i * WAVE + lane);
        uint64_t b[4];
        bool hits[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bool hit = is_tag<MODE>(tm, t[j], tab);
            if (EDGE) hit = hit && q0 + j >= q_lo && q0 + j < q_hi;
            b[j] = __ballot(hit);
            hits[j] = hit;
        }
        if ((b[0] | b[1] | b[2] | b[3]) == 0) continue; /* wave-uniform: most vectors hold no tag */
        uint32_t idx = cnt;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            idx = __builtin_amdgcn_mbcnt_hi((uint32_t)(b[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[j], idx));
        /* one store per token column that holds a tag, in the lane's position
         * order: with a loop over each lane's own tags every turn ran the whole
         * wave through the selection of its token (outline-heavy rows, a tag in
         * a hundred tokens: the scan of 8,192 rows of 3,500 32.4 us, 30.0 so) */
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (b[j] == 0) continue; /* wave-uniform */
            uint32_t c = MODE == TM_HASH ? slot_class(tm, t[j], tab_class) : 0u;
            if (hits[j]) {
                if (MODE != TM_HASH) c = tag_class<MODE>(tm, t[j]);
                if (idx < cap) dst[idx] = ((uint32_t)(q0 + j + bias) << 4) | c;
                ++idx;
            }
        }
        cnt += (uint32_t)(__popcll(b[0]) + __popcll(b[1]) + __popcll(b[2]) + __popcll(b[3]));
    }
}

__device__ __forceinline__ void issue_loads(int4 (&x)[LOADS], const int4 *src, int64_t v0, int64_t v1, bool edge,
                                            int lane)
{
    const int4 *p = src + v0 + lane;
    if (!edge) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) x[i] = load_vec(p + i * WAVE);
    } else {
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            x[i] = (v0 + i * WAVE + lane < v1) ? load_vec(p + i * WAVE) : make_int4(-1, -1, -1, -1);
    }
}

/* seg[s].count = DENSE for s in [a, b): the row kernels classify those
 * segments' tokens again. */

__device__ __forceinline__ void mark_dense(SegRec *seg, int64_t a, int64_t b, int lane)
{
    for (int64_t s = a + lane; s < b; s += WAVE) seg[s].count = DENSE;
}

struct ScanArgs {
    const int32_t *tok_base;
    int64_t mis;
    const int64_t *starts;
    const int32_t *lengths;
    int64_t n;
    const int64_t *seg_off;
    int64_t seg_cap;
    SegRec *seg;
    uint32_t *slots;
    uint32_t pool_slots; /* the pool: slots [0, pool_slots); wave w's region starts at
                            POOL_PER_SEG * s_begin + x * w and ends at POOL_PER_SEG * s_end + x * (w + 1),
                            with x = (pool_slots - POOL_PER_SEG * S) / W rounded down to 4 */
    uint8_t *mode;
    TagMatch tm;
    int32_t *counters;    /* cleared by a scan that plans the batch itself */
};

/* Row being collected by a scan wave, in processing order. */
struct RowCollect {
    uint32_t lcnt; /* events in the wave's LDS buffer */
    bool global;   /* events go to per-segment lists; the row kernel evaluates the row */
    uint32_t pc;    /* next free slot of the wave's pool region (a multiple of 4) ... */
    uint32_t p_end; /* ... and its end */
};

constexpr int EVL = 1024;                 /* LDS events per wave */
constexpr int SCAN_WAVES = 4;             /* waves per scan block */
/* Waves per block of a scan that plans in LDS.  Every block plans the whole
 * batch before its first load, so half as many blocks of twice the size plan
 * it half as often and are all dispatched sooner (a 2,048-row step: 2.7 us
 * less); the same per-CU occupancy. */
constexpr int SCAN_PLAN_WAVES = 8;
template <bool PLAN>
constexpr int scan_waves() { return PLAN ? SCAN_PLAN_WAVES : SCAN_WAVES; }

/* The whole of row `row` is in the wave's LDS buffer lev[0 .. lcnt): copy it,
 * coalesced, to the wave's pool region as one compact list for the row kernel
 * (mode 1).  A list that does not fit makes the row kernel classify the row's
 * segments again. */
__device__ __forceinline__ void flush_row(const ScanArgs &a, int64_t row, int64_t first, int64_t last, uint32_t lcnt,
                                          const uint32_t *lev, RowCollect &rc, int lane)
{
    const uint32_t need = (lcnt + 3u) & ~3u;
    if (need > rc.p_end - rc.pc) {
        mark_dense(a.seg, first, last + 1, lane);
        return;
    }
    uint32_t *dst = a.slots + rc.pc;
    /* lane i copies events other lanes wrote: the wave's LDS stores above
     * come first (a wave's LDS accesses are performed in program order; this
     * keeps the compiler from moving them across) */
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i = lane; i < lcnt; i += WAVE) dst[i] = lev[i];
    if (lane == 0) {
        a.seg[first] = SegRec{(int32_t)lcnt, rc.pc};
        a.mode[row] = MODE_COMPACT;
    }
    rc.pc += need;
}

/* Scan one segment whose loads are in x.  A row owned by the wave collects
 * its events in the wave's LDS buffer; any other row leaves its events in the
 * per-segment lists for the row kernels.  Returns true when this segment
 * completes a row whose events are all in the LDS buffer (rc.lcnt of them). */
template <int MODE, bool PLAN>
__device__ __forceinline__ bool collect_segment(const ScanArgs &a, const int4 (&x)[LOADS], const SegView &w,
                                                RowCollect &rc, uint32_t *lev, int32_t tab, int32_t tab_class,
                                                int lane)
{
    if (w.s == w.first) {
        rc.lcnt = 0;
        rc.global = !w.owned;
        if (PLAN) {
            /* the scan planned the batch itself: the wave holding a row's first
             * segment clears its mode (flush_row may set it again below) */
            if (lane == 0) a.mode[w.row] = 0;
        }
    }
    uint32_t cnt = 0; /* wave-uniform */
    if (!rc.global) {
        const int32_t bias = (int32_t)(4 * w.v0 - w.g); /* row position of segment position 0 */
        const uint32_t cap = (uint32_t)EVL - rc.lcnt;
        if (!w.edge) scan_vectors<MODE, false>(x, 0, SEG_TOK, lev + rc.lcnt, cap, bias, cnt, a.tm, tab, tab_class, lane);
        else scan_vectors<MODE, true>(x, w.q_lo, w.q_hi, lev + rc.lcnt, cap, bias, cnt, a.tm, tab, tab_class, lane);
        if (cnt > cap) {
            /* the row's events overflow the LDS buffer: its segments so far are
             * classified again by the row kernel, the rest use per-segment lists */
            mark_dense(a.seg, w.first, w.s + 1, lane);
            rc.global = true;
        } else {
            rc.lcnt += cnt;
        }
    } else {
        /* the segment's own list, in the wave's pool region */
        const uint32_t room = min(rc.p_end - rc.pc, (uint32_t)SEG_TOK); /* a multiple of 4 */
        uint32_t *dst = a.slots + rc.pc;
        if (!w.edge) scan_vectors<MODE, false>(x, 0, SEG_TOK, dst, room, 0, cnt, a.tm, tab, tab_class, lane);
        else scan_vectors<MODE, true>(x, w.q_lo, w.q_hi, dst, room, 0, cnt, a.tm, tab, tab_class, lane);
        const bool stored = cnt <= room;
        if (lane == 0) a.seg[w.s] = SegRec{stored ? (int32_t)cnt : DENSE, rc.pc};
        if (stored) rc.pc += (cnt + 3u) & ~3u;
    }
    return w.s == w.last && !rc.global;
}

/* block_plan by every scan block.  Block 0 also writes the plan to seg_off for
 * the row kernels, clears the mode of rows without segments (no scan wave
 * sees them; all rows when the batch overflows the workspace) and the
 * counters; every other row's mode is cleared by the wave holding its first
 * segment. */
template <int NW>
__device__ __forceinline__ void scan_plan(const ScanArgs &a, int64_t *off, int64_t *part, int64_t *st, int32_t *ln)
{
    block_plan<NW>(a.starts, a.lengths, a.n, a.mis, off, part, st, ln);
    const int t = (int)threadIdx.x;
    if (blockIdx.x == 0) {
        /* when the batch overflows the workspace no scan wave runs, so every
         * mode byte is cleared here */
        const bool overflow = off[a.n] > a.seg_cap;
        int64_t *seg_off = const_cast<int64_t *>(a.seg_off);
        for (int64_t r = t; r <= a.n; r += WAVE * NW) {
            seg_off[r] = off[r];
            if (r < a.n && (overflow || off[r + 1] == off[r])) a.mode[r] = 0;
        }
        if (t < 4) a.counters[t] = 0;
    }
}

/* Work distribution of a large scan.  Compute units do not all stream at the
 * same rate (on MI355X, with equal shares, the waves of four of the eight dies
 * finished about 9 % later than the others), so equal static shares leave
 * part of the chip idle at the end.  A scan with at least DYN_MIN_PER_WAVE segments per
 * wave therefore gives each wave an equal contiguous share of the first
 * S1 = S - S * DYN_NUM / DYN_DEN segments, and hands out the rest in chunks,
 * in segment order, through one counter: rounds of one chunk per wave whose
 * size halves from c0 = (S - S1) / (2 W) down to DYN_KMIN, then chunks of
 * DYN_KMIN to the end.  A wave that finishes early takes more chunks.  Rows cut
 * by a chunk boundary are split rows, handled as those cut by a share's
 * boundary.  Every range (share or chunk) has its own region of the slot pool:
 * range q (shares 0 .. W-1, then chunk i as W + i) covering segments [b, e)
 * owns slots [POOL_PER_SEG * b + x * q, POOL_PER_SEG * e + x * (q + 1)) past
 * the pool's start, x = (pool_slots - POOL_PER_SEG * S) / (W + chunks) rounded down
 * to 4, so regions are disjoint and in segment order. */
constexpr int64_t DYN_MIN_PER_WAVE = 256;
constexpr int64_t DYN_NUM = 3, DYN_DEN = 16;
constexpr int64_t DYN_KMIN = 32;
constexpr int64_t BLK_CHUNK = 2; /* segments per chunk of a block's own pool ... */
constexpr int64_t BLK_MIN = 64;  /* ... which a block has from this many segments on */

struct ScanSched {
    int64_t S, S1, c0, base_final, n_chunks, W;
    int32_t rounds;
    bool dyn;
    int64_t kmin; /* every field is wave-uniform */

    /* S units (segments) over W waves; kmin: the smallest chunk; num / den of
     * the units handed out in chunks (all wave-uniform) */
    __device__ void init(int64_t S_, int64_t W_, bool allow, int64_t kmin_ = DYN_KMIN, int64_t num = DYN_NUM,
                         int64_t den = DYN_DEN)
    {
        S = S_;
        W = W_;
        kmin = kmin_;
        dyn = allow && S >= DYN_MIN_PER_WAVE * kmin / DYN_KMIN * W;
        S1 = dyn ? S - S / den * num - S % den * num / den : S;
        c0 = (S - S1) / (2 * W);
        rounds = 0;
        int64_t b = S1;
        while ((c0 >> rounds) >= kmin) {
            b += W * (c0 >> rounds);
            ++rounds;
        }
        base_final = b;
        n_chunks = dyn ? W * rounds + (S - b + kmin - 1) / kmin : 0;
    }
    /* units [b, e) of chunk i < n_chunks */
    __device__ void chunk(int64_t i, int64_t &b, int64_t &e) const
    {
        if (i >= W * rounds) {
            b = base_final + (i - W * rounds) * kmin;
            e = min(b + kmin, S);
            return;
        }
        int64_t base = S1;
        int32_t r = 0;
        while (i >= W) {
            base += W * (c0 >> r);
            i -= W;
            ++r;
        }
        b = base + i * (c0 >> r);
        e = b + (c0 >> r);
    }
};

/* Scan segments [s_begin, s_end) (a share or a chunk), filling the pool region
 * [pc, p_end).  Two register buffers: segment s + 1 is in flight while s is
 * compacted (and a finished row's events flushed), so the wave always has a
 * segment in flight. */
template <int MODE, bool PLAN>
__device__ __forceinline__ void scan_range(const ScanArgs &a, const int64_t *seg_off, const int64_t *starts,
                                           const int32_t *lengths, int64_t s_begin, int64_t s_end,
                                           uint32_t pc, uint32_t p_end, uint32_t *lev, int32_t tab,
                                           int32_t tab_class, int lane)
{
    const int4 *src = reinterpret_cast<const int4 *>(a.tok_base);
    SegCursor cur;
    cur.seg_off = seg_off;
    cur.starts = starts;
    cur.lengths = lengths;
    cur.mis = a.mis;
    cur.s_begin = s_begin;
    cur.s_end = s_end;
    cur.seek(s_begin, a.n);

    RowCollect rc;
    rc.lcnt = 0;
    rc.global = true; /* a row already begun in the previous range */
    rc.pc = pc;
    rc.p_end = p_end;
    SegView w = cur.view(s_begin);
    int4 xa[LOADS], xb[LOADS];
    issue_loads(xa, src, w.v0, w.v1, w.edge, lane);
    int64_t s = s_begin;
    while (true) {
        SegView wn;
        bool more = s + 1 < s_end;
        if (more) {
            wn = cur.view(s + 1);
            issue_loads(xb, src, wn.v0, wn.v1, wn.edge, lane);
        }
        if (collect_segment<MODE, PLAN>(a, xa, w, rc, lev, tab, tab_class, lane))
            flush_row(a, w.row, w.first, w.last, rc.lcnt, lev, rc, lane);
        if (!more) break;
        ++s;
        w = wn;
        more = s + 1 < s_end;
        if (more) {
            wn = cur.view(s + 1);
            issue_loads(xa, src, wn.v0, wn.v1, wn.edge, lane);
        }
        if (collect_segment<MODE, PLAN>(a, xb, w, rc, lev, tab, tab_class, lane))
            flush_row(a, w.row, w.first, w.last, rc.lcnt, lev, rc, lane);
        if (!more) break;
        ++s;
        w = wn;
    }
}

/* One wave per segment: each wave scans its share of the segments, then (a
 * large scan) takes chunks of the rest until none is left. */
template <int MODE, bool PLAN>
__global__ void __launch_bounds__(WAVE * scan_waves<PLAN>(), PARASON_SCAN_WAVES_PER_SIMD) scan_rows(ScanArgs a)
{
    constexpr int NW = scan_waves<PLAN>();
    __shared__ uint32_t lds_ev[NW][EVL];
    __shared__ int64_t plan_off[PLAN ? SCAN_PLAN_ROWS + 1 : 1];
    __shared__ int64_t plan_st[PLAN ? SCAN_PLAN_ROWS : 1];
    __shared__ int32_t plan_ln[PLAN ? SCAN_PLAN_ROWS : 1];
    __shared__ int64_t plan_part[NW];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int64_t wave = uniform64((int64_t)blockIdx.x * NW + wib);
    const int64_t n_waves = (int64_t)gridDim.x * NW;
    const int64_t *seg_off = a.seg_off;
    /* a batch the scan plans (a small one): block k scans segments
     * [S k / nb, S (k + 1) / nb), its waves an equal share each of the first
     * L1 = L - 3 L / 16 of them, then the rest in chunks of BLK_CHUNK handed
     * out by an LDS counter, so that the block's waves end together (a block
     * of fewer than BLK_MIN segments keeps equal shares of all of them: its
     * waves are done before a counter would pay); ranges are numbered
     * k Q + wave (shares), k Q + NW + j (chunks), Q above any block's share
     * and chunk count. */
    __shared__ uint32_t blk_next;
    if (PLAN) {
        if (threadIdx.x == 0) blk_next = 0; /* before scan_plan's barriers */
        scan_plan<NW>(a, plan_off, plan_part, plan_st, plan_ln);
        seg_off = plan_off;
    }
    const int64_t S = uniform64(seg_off[a.n]);
    if (S > a.seg_cap) return; /* the row kernel reports PARASON_FLAG_WS_OVERFLOW */
    uint32_t *lev = lds_ev[wib];
    const int32_t tab = MODE == TM_HASH ? a.tm.slot_id[lane] : 0;
    const int32_t tab_class = MODE == TM_HASH ? (int32_t)classify(a.tm, tab, false) : 0; /* of a slot in use */
    int64_t b, e, q, Bk = 0, Ek = 0, L1 = 0, Q = 0;
    bool blk_dyn = false;
    uint32_t extra;
    ScanSched sch;
    if (PLAN) {
        /* 64-bit divisions are long on the scalar unit: by shifts when the
         * block count is a power of two (two blocks per compute unit) */
        const uint32_t nb = gridDim.x;
        const bool pow2 = (nb & (nb - 1)) == 0;
        const int sh = __builtin_ctz(nb);
        const int64_t k = blockIdx.x;
        Bk = uniform64(pow2 ? (S * k) >> sh : S * k / nb);
        Ek = uniform64(pow2 ? (S * (k + 1)) >> sh : S * (k + 1) / nb);
        Q = uniform64(NW + ((pow2 ? S >> sh : S / nb) + 1) * DYN_NUM / DYN_DEN / BLK_CHUNK + 2);
        /* slot indices fit 32 bits, which the host checks */
        extra = ((a.pool_slots - POOL_PER_SEG * (uint32_t)S) / (uint32_t)(nb * Q)) & ~3u;
        blk_dyn = Ek - Bk >= BLK_MIN;
        L1 = blk_dyn ? (Ek - Bk) - (Ek - Bk) * DYN_NUM / DYN_DEN : Ek - Bk;
        b = uniform64(Bk + L1 * wib / NW);
        e = uniform64(Bk + L1 * (wib + 1) / NW);
        q = k * Q + wib;
    } else {
        sch.init(S, n_waves, true);
        /* S1 < 2^40 and n_waves < 2^20 (checked on the host), so S1 * wave fits */
        b = uniform64(sch.S1 * wave / n_waves);
        e = uniform64(sch.S1 * (wave + 1) / n_waves);
        q = wave;
        extra = ((a.pool_slots - POOL_PER_SEG * (uint32_t)S) / (uint32_t)(n_waves + sch.n_chunks)) & ~3u;
    }
    while (true) {
        if (b < e) {
            const uint32_t pc = __builtin_amdgcn_readfirstlane(POOL_PER_SEG * (uint32_t)b + extra * (uint32_t)q);
            const uint32_t p_end =
                __builtin_amdgcn_readfirstlane(POOL_PER_SEG * (uint32_t)e + extra * (uint32_t)(q + 1));
            scan_range<MODE, PLAN>(a, seg_off, PLAN ? plan_st : a.starts, PLAN ? plan_ln : a.lengths, b, e, pc, p_end,
                                   lev, tab, tab_class, lane);
        }
        if (PLAN) {
            if (!blk_dyn) break;
            uint32_t j = 0;
            if (lane == 0) j = atomicAdd(&blk_next, 1u);
            j = __builtin_amdgcn_readfirstlane(j);
            b = uniform64(Bk + L1 + (int64_t)j * BLK_CHUNK);
            if (b >= Ek) break;
            e = uniform64(min(b + BLK_CHUNK, Ek));
            q = blockIdx.x * Q + NW + j;
            continue;
        }
        if (!sch.dyn) break;
        int32_t i = 0;
        if (lane == 0) i = atomicAdd(&a.counters[3], 1);
        i = __builtin_amdgcn_readfirstlane(i);
        if ((int64_t)i >= sch.n_chunks) break;
        sch.chunk(i, b, e);
        b = uniform64(b);
        e = uniform64(e);
        q = n_waves + i;
    }
}

/* The ceiling the token scan is measured against: a plain streaming read of
 * the same buffer with the scan's 16-byte nontemporal loads and persistent
 * grid, every unit handed out in chunks through a counter as ScanSched does
 * (a chunk unit is one 8 KB step of eight loads per lane, all issued before
 * any is used), and no other work.  Each wave stores the XOR of what it read to
 * sink[wave % sink_len] (so the loads are kept).  *next must be zero at the
 * launch (probe_reset clears it). */
constexpr int PROBE_LOADS = 8;
constexpr int PROBE_CHUNK = PROBE_LOADS * WAVE; /* 16-byte vectors per chunk */
constexpr int64_t PROBE_KMIN = 16;              /* the smallest chunk: 16 steps of 8 KB */

__global__ void probe_reset(int32_t *next) { *next = 0; }

__global__ void __launch_bounds__(WAVE * SCAN_WAVES) read_probe(const int4 *__restrict__ src, int64_t n_vec,
                                                                const int32_t *__restrict__ tail, int32_t n_tail,
                                                                uint32_t *__restrict__ sink, int64_t sink_len,
                                                                int32_t *__restrict__ next)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t wave = uniform64((int64_t)blockIdx.x * SCAN_WAVES + threadIdx.x / WAVE);
    const int64_t n_waves = (int64_t)gridDim.x * SCAN_WAVES;
    const int64_t n_chunks = n_vec / PROBE_CHUNK;
    ScanSched sch;
    /* units of 8 KB, all of them in chunks: the waves of a pure read
     * stream at rates several times apart, more than the scan's equal
     * shares leave room for */
    sch.init(n_chunks, n_waves, true, PROBE_KMIN, 1, 1);
    int64_t c0 = uniform64(sch.S1 * wave / n_waves), c1 = uniform64(sch.S1 * (wave + 1) / n_waves);
    uint32_t acc = 0;
    while (true) {
        for (int64_t c = c0; c < c1; ++c) {
            int4 x[PROBE_LOADS];
            const int4 *p = src + c * PROBE_CHUNK + lane;
#pragma unroll
            for (int i = 0; i < PROBE_LOADS; ++i) x[i] = load_vec(p + i * WAVE);
#pragma unroll
            for (int i = 0; i < PROBE_LOADS; ++i) acc ^= (uint32_t)(x[i].x ^ x[i].y ^ x[i].z ^ x[i].w);
        }
        if (!sch.dyn) break;
        int32_t i = 0;
        if (lane == 0) i = atomicAdd(next, 1);
        i = __builtin_amdgcn_readfirstlane(i);
        if ((int64_t)i >= sch.n_chunks) break;
        sch.chunk(i, c0, c1);
        c0 = uniform64(c0);
        c1 = uniform64(c1);
    }
    if (wave == n_waves - 1) {
        /* the vectors after the last whole chunk, then the last 0-3 elements */
        for (int64_t v = n_chunks * PROBE_CHUNK + lane; v < n_vec; v += WAVE) {
            const int4 x = load_vec(src + v);
            acc ^= (uint32_t)(x.x ^ x.y ^ x.z ^ x.w);
        }
        if (lane < n_tail) acc ^= (uint32_t)tail[lane];
    }
    /* XOR over the wave by DPP (row_shr) and readlane, as the scans do */
    uint32_t v = acc;
    v ^= (uint32_t)row_shr<1>((int32_t)v, 0);
    v ^= (uint32_t)row_shr<2>((int32_t)v, 0);
    v ^= (uint32_t)row_shr<4>((int32_t)v, 0);
    v ^= (uint32_t)row_shr<8>((int32_t)v, 0);
    const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 15) ^
                       (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 31) ^
                       (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 47) ^ (uint32_t)lane63((int32_t)v);
    if (lane == 0) sink[wave % sink_len] = w;
}

/* ------------------------------------------------------------------ reward */

struct RewardArgs {
    const int32_t *total, *latency, *n_subtask, *n_trial;
    const uint32_t *flags;
    const uint8_t *correct;
    int64_t n_groups;
    int32_t G;
    int64_t n;
    double alpha, beta_s, beta_r, rho, rho_clip;
    uint32_t cfg_flags;
    float *reward, *r_subtask, *r_trial, *eta;
    float *accel;   /* optional: total / latency */
    int32_t *saved; /* optional: total - latency */
};

constexpr uint32_t NOT_EVALUATED = PARASON_FLAG_DEPTH_LIMIT | PARASON_FLAG_WS_OVERFLOW | PARASON_FLAG_BAD_ROW;

__device__ __forceinline__ double ratio(int32_t n, int32_t total)
{
    return total > 0 ? __ddiv_rn((double)n, (double)total) : 0.0;
}

/* Do all rows of the group have the same ratio n/total?  Exact (cross-multiplied). */
__device__ __forceinline__ bool same_ratio(const int32_t *nn, const int32_t *tt, int64_t r0, int32_t G)
{
    int64_t n0 = tt[r0] > 0 ? nn[r0] : 0, d0 = tt[r0] > 0 ? tt[r0] : 1;
    for (int32_t i = 1; i < G; ++i) {
        int64_t ni = tt[r0 + i] > 0 ? nn[r0 + i] : 0, di = tt[r0 + i] > 0 ? tt[r0 + i] : 1;
        if (ni * d0 != n0 * di) return false;
    }
    return true;
}

/* mean and population standard deviation of x over the group, by index order */
struct Moments {
    double mu, sigma;
};

template <class F>
__device__ __forceinline__ Moments moments(F x, int32_t G)
{
    double s = 0.0;
    for (int32_t i = 0; i < G; ++i) s = __dadd_rn(s, x(i));
    double mu = __ddiv_rn(s, (double)G);
    double ss = 0.0;
    for (int32_t i = 0; i < G; ++i) {
        double d = __dsub_rn(x(i), mu);
        ss = __dadd_rn(ss, __dmul_rn(d, d));
    }
    return Moments{mu, __dsqrt_rn(__ddiv_rn(ss, (double)G))};
}

__device__ __forceinline__ double zscore(double x, Moments m, bool all_equal)
{
    return (all_equal || m.sigma == 0.0) ? 0.0 : __ddiv_rn(__dsub_rn(x, m.mu), m.sigma);
}

/* A row's accounting outputs and correctness, loaded once. */
struct RowVals {
    uint32_t fl;
    int32_t lat, tot, ns, nt;
    uint8_t correct;
};

__device__ __forceinline__ RowVals row_vals(const RewardArgs &a, int64_t r)
{
    return RowVals{a.flags[r], a.latency[r], a.total[r], a.n_subtask[r], a.n_trial[r], a.correct[r]};
}

/* Stores row r's reward and ratios; returns the reward as stored. */
__device__ __forceinline__ float write_reward(const RewardArgs &a, int64_t r, const RowVals &v, double zT, double zs,
                                              double zr, double xs, double xr)
{
    const int32_t tot = v.tot;
    const double e = tot > 0 ? __dsub_rn(1.0, __ddiv_rn((double)v.lat, (double)tot)) : 0.0;
    const bool valid = (v.fl & PARASON_FLAG_VALID) != 0;
    const bool c = v.correct != 0 && (valid || (a.cfg_flags & PARASON_CFG_INVALID_KEEPS_CORRECTNESS));
    const double accel = __dmul_rn(a.rho, e);
    const double clipped = accel < a.rho_clip ? accel : a.rho_clip;
    double inner = __dsub_rn(1.0, __dmul_rn(a.alpha, zT));
    inner = __dadd_rn(inner, __dmul_rn(a.beta_s, zs));
    inner = __dadd_rn(inner, __dmul_rn(a.beta_r, zr));
    inner = __dadd_rn(inner, clipped);
    const double R = __dadd_rn(-1.0, __dmul_rn(__dmul_rn(2.0, c ? 1.0 : 0.0), inner));
    a.reward[r] = (float)R;
    if (a.r_subtask) a.r_subtask[r] = (float)xs;
    if (a.r_trial) a.r_trial[r] = (float)xr;
    if (a.eta) a.eta[r] = (float)e;
    /* a row with tokens has latency >= 1 (an invalid row's latency is its length) */
    if (a.accel) a.accel[r] = tot > 0 ? (float)__ddiv_rn((double)tot, (double)v.lat) : 1.0f;
    if (a.saved) a.saved[r] = tot - v.lat;
    return (float)R;
}

__device__ __forceinline__ float write_nan(const RewardArgs &a, int64_t r, const RowVals &v)
{
    const float nan = __int_as_float(0x7fc00000);
    a.reward[r] = nan;
    if (a.r_subtask) a.r_subtask[r] = nan;
    if (a.r_trial) a.r_trial[r] = nan;
    if (a.eta) a.eta[r] = nan;
    if (a.accel) a.accel[r] = nan;
    if (a.saved) a.saved[r] = (v.fl & NOT_EVALUATED) ? 0 : v.tot - v.lat;
    return nan;
}

/* A group of G rows (G a power of two up to 64) in G consecutive lanes of one
 * wave: each lane loads its own row once and reads the others' values with
 * shuffles, in the group's order.  GC > 0 fixes G at compile time (the
 * paper's G = 8), so that the group's shuffles are unrolled and issue
 * together instead of one sum step after another. */
template <int GC>
__device__ __forceinline__ float group_reward_lanes(const RewardArgs &a, int64_t r, int32_t G_run, const RowVals &v)
{
    const int32_t G = GC > 0 ? GC : G_run;
    const int lane = threadIdx.x & (WAVE - 1);
    const int gl = lane & ~(G - 1); /* the group's first lane */
    const uint64_t gmask = (G == WAVE ? ~0ull : ((1ull << G) - 1ull)) << gl;
    const uint32_t fl = v.fl;
    const int32_t lat = v.lat, tot = v.tot, ns = v.ns, nt = v.nt;
    if ((__ballot(!(fl & NOT_EVALUATED)) & gmask) != gmask) {
        return write_nan(a, r, v); /* the whole group returns here */
    }
    const bool lat_equal = (__ballot(lat == __shfl(lat, gl, WAVE)) & gmask) == gmask;
    /* exact equality of the ratios, cross-multiplied against the group's first row */
    const int64_t d = tot > 0 ? tot : 1;
    const int64_t d0 = __shfl(d, gl, WAVE);
    const int64_t s_n = tot > 0 ? ns : 0, t_n = tot > 0 ? nt : 0;
    const bool sub_equal = (__ballot(s_n * d0 == __shfl(s_n, gl, WAVE) * d) & gmask) == gmask;
    const bool tri_equal = (__ballot(t_n * d0 == __shfl(t_n, gl, WAVE) * d) & gmask) == gmask;
    const double xT = (double)lat, xs = ratio(ns, tot), xr = ratio(nt, tot);
    const Moments mT = moments([&](int32_t j) { return __shfl(xT, gl + j, WAVE); }, G);
    const Moments ms = moments([&](int32_t j) { return __shfl(xs, gl + j, WAVE); }, G);
    const Moments mr = moments([&](int32_t j) { return __shfl(xr, gl + j, WAVE); }, G);
    return write_reward(a, r, v, zscore(xT, mT, lat_equal), zscore(xs, ms, sub_equal), zscore(xr, mr, tri_equal), xs,
                        xr);
}

/* Row r's reward from its group's values in memory, in the group's row order
 * (any group size, any thread layout). */
__device__ __forceinline__ float group_reward_memory(const RewardArgs &a, int64_t r)
{
    const int32_t G = a.G;
    const int64_t r0 = r - r % G;
    bool evaluated = true;
    bool lat_equal = true;
    for (int32_t i = 0; i < G; ++i) {
        evaluated = evaluated && !(a.flags[r0 + i] & NOT_EVALUATED);
        lat_equal = lat_equal && a.latency[r0 + i] == a.latency[r0];
    }
    const RowVals v = row_vals(a, r);
    if (!evaluated) return write_nan(a, r, v);
    const bool sub_equal = same_ratio(a.n_subtask, a.total, r0, G);
    const bool tri_equal = same_ratio(a.n_trial, a.total, r0, G);
    auto xT = [&](int32_t i) { return (double)a.latency[r0 + i]; };
    auto xs = [&](int32_t i) { return ratio(a.n_subtask[r0 + i], a.total[r0 + i]); };
    auto xr = [&](int32_t i) { return ratio(a.n_trial[r0 + i], a.total[r0 + i]); };
    const Moments mT = moments(xT, G), ms = moments(xs, G), mr = moments(xr, G);
    const int32_t i = (int32_t)(r - r0);
    return write_reward(a, r, v, zscore(xT(i), mT, lat_equal), zscore(xs(i), ms, sub_equal),
                        zscore(xr(i), mr, tri_equal), xs(i), xr(i));
}

/* The deep tier's rows (listed by rows_par or rows_listed), run by the first
 * block of group_reward instead of a launch of their own. */
struct DeepArgs {
    RowArgs rows;
    const uint8_t *mode;
    const int32_t *counters; /* counters[1]: rows in deep_rows */
    int32_t *deep_rows;
    int32_t *frames;
    uint32_t *bits;
};

/* deep_rows in row order, by one block (part: a word per wave).  The list is
 * filled through an atomic counter, so its order is the scheduler's, and sums in
 * list order would differ in their last bits from call to call.  It is written
 * again from the rows' MODE_DEEP marks: sixteen rows per thread and step,
 * whatever the number of deep rows (a batch with two or more only). */
__device__ __forceinline__ void order_deep_rows(const DeepArgs &d, int64_t n, int32_t *part)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    int32_t found = 0;
    for (int64_t r0 = 0; r0 < n; r0 += 16 * (int64_t)blockDim.x) {
        const int64_t r = r0 + 16 * (int64_t)threadIdx.x;
        uint32_t hit = 0; /* bit j: row r + j */
        if (r < n) {      /* the section is padded to whole quads */
            const uint4 q = *reinterpret_cast<const uint4 *>(d.mode + r);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int j = 0; j < 16; ++j) hit |= ((w[j / 4] >> (8 * (j % 4))) & MODE_DEEP) != 0 ? 1u << j : 0u;
            if (n - r < 16) hit &= (1u << (n - r)) - 1u;
        }
        const int32_t cnt = __popcll(hit), incl = dpp_incl_scan<OpAdd>(cnt, lane);
        __syncthreads(); /* part's use before */
        if (lane == WAVE - 1) part[wv] = incl;
        __syncthreads();
        int32_t at = found + incl - cnt;
        for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) {
            at += w < wv ? part[w] : 0;
            found += part[w];
        }
        for (; hit != 0; hit &= hit - 1) d.deep_rows[at++] = (int32_t)(r + __builtin_ctz(hit));
    }
    __syncthreads();
}

/* ------------------------------------------------------------------ batch metrics */

constexpr int NMI = 9; /* valid, triggered, correct, truncated, mismatch, sum total, latency, Subtask, Trial */

/* Sums over some rows of the batch. */
struct MetricRec {
    int64_t c[NMI];
    double reward;
};

constexpr int RED_SINGLE = 1024;     /* rows whose reductions one block does */
constexpr int RED_ONE_ROW = 1 << 16; /* rows up to which a reduction's thread takes one row */
constexpr int64_t RED_TILES = 1024;  /* at most so many moment records: every block of the rewards merges them all */
constexpr int RED_WAVES = RED_SINGLE / WAVE;

/* Sum over the wave of values below 2^32, exact, in every lane. */
__device__ __forceinline__ int64_t wave_sum_u32(int32_t v)
{
    return (int64_t)wave_sum32((int32_t)((uint32_t)v & 0xffffu)) + ((int64_t)wave_sum32((int32_t)((uint32_t)v >> 16)) << 16);
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) v = __dadd_rn(v, __shfl(v, lane ^ d, WAVE));
    return v;
}

/* The block's rows (one per thread with `has`: its accounting v and its stored
 * reward R) added to rec, which thread 0 holds: counts by ballots, token sums
 * exactly, the rewards' sum in a fixed tree.  Every thread calls this. */
__device__ __forceinline__ void block_metrics(bool has, const RowVals &v, float R, MetricRec *lds /* [RED_WAVES] */,
                                              MetricRec &rec)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const uint32_t f = has ? v.fl : 0u;
    MetricRec w;
    w.c[0] = __popcll(__ballot((f & PARASON_FLAG_VALID) != 0));
    w.c[1] = __popcll(__ballot((f & PARASON_FLAG_TRIGGERED) != 0));
    w.c[2] = __popcll(__ballot(has && v.correct != 0));
    w.c[3] = __popcll(__ballot((f & PARASON_FLAG_TRUNCATED) != 0));
    w.c[4] = __popcll(__ballot((f & PARASON_FLAG_COUNT_MISMATCH) != 0));
    w.c[5] = wave_sum_u32(has ? v.tot : 0);
    w.c[6] = wave_sum_u32(has ? v.lat : 0);
    w.c[7] = wave_sum_u32(has ? v.ns : 0);
    w.c[8] = wave_sum_u32(has ? v.nt : 0);
    w.reward = wave_sum_f64(has ? (double)R : 0.0);
    __syncthreads(); /* the records of a call before */
    if (lane == 0) lds[wv] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < (int)(blockDim.x / WAVE); ++i) {
            for (int k = 0; k < NMI; ++k) rec.c[k] += lds[i].c[k];
            rec.reward = __dadd_rn(rec.reward, lds[i].reward);
        }
    }
}

__device__ __forceinline__ MetricRec no_metrics()
{
    MetricRec r;
    for (int k = 0; k < NMI; ++k) r.c[k] = 0;
    r.reward = 0.0;
    return r;
}

/* The PARASON_METRIC_COUNT metrics from the sums over the batch's n rows. */
__device__ __forceinline__ void write_metrics(const MetricRec &rec, int64_t n_rows, double *m)
{
    const int64_t *c = rec.c;
    const double n = (double)n_rows;
    const int64_t st = c[5], sl = c[6];
    for (int k = 0; k < PARASON_METRIC_COUNT; ++k) m[k] = 0.0;
    m[PARASON_METRIC_ROWS] = n;
    m[PARASON_METRIC_VALID] = (double)c[0];
    m[PARASON_METRIC_TRIGGERED] = (double)c[1];
    m[PARASON_METRIC_CORRECT] = (double)c[2];
    m[PARASON_METRIC_TRUNCATED] = (double)c[3];
    m[PARASON_METRIC_COUNT_MISMATCH] = (double)c[4];
    m[PARASON_METRIC_SUM_TOTAL] = (double)st;
    m[PARASON_METRIC_SUM_LATENCY] = (double)sl;
    m[PARASON_METRIC_SUM_SUBTASK] = (double)c[7];
    m[PARASON_METRIC_SUM_TRIAL] = (double)c[8];
    if (n_rows > 0) {
        m[PARASON_METRIC_TRIGGER_RATIO] = __ddiv_rn((double)c[1], n);
        m[PARASON_METRIC_MEAN_LATENCY] = __ddiv_rn((double)sl, n);
        m[PARASON_METRIC_MEAN_TOTAL] = __ddiv_rn((double)st, n);
        m[PARASON_METRIC_MEAN_SAVED] = __ddiv_rn((double)(st - sl), n);
        m[PARASON_METRIC_ACCURACY] = __ddiv_rn((double)c[2], n);
        m[PARASON_METRIC_MEAN_REWARD] = __ddiv_rn(rec.reward, n);
    }
    if (sl > 0) m[PARASON_METRIC_ACCELERATION] = __ddiv_rn((double)st, (double)sl);
    if (st > 0) {
        m[PARASON_METRIC_SUBTASK_SHARE] = __ddiv_rn((double)c[7], (double)st);
        m[PARASON_METRIC_TRIAL_SHARE] = __ddiv_rn((double)c[8], (double)st);
    }
}

/* A block's metrics: the metrics themselves when it is the only one, else its
 * record for metrics_final. */
__device__ __forceinline__ void put_metrics(const MetricRec &rec, int64_t n_rows, MetricRec *recs, double *metrics)
{
    if (threadIdx.x != 0) return;
    if (gridDim.x == 1) write_metrics(rec, n_rows, metrics);
    else recs[blockIdx.x] = rec;
}

/* The metrics of a batch from its blocks' records, in one block: every thread
 * adds a run of records in order, then the threads' sums in a fixed tree. */
__global__ void __launch_bounds__(RED_THREADS) metrics_final(const MetricRec *__restrict__ recs, int64_t n_recs,
                                                             int64_t n_rows, double *__restrict__ metrics)
{
    __shared__ int64_t il[NMI * RED_THREADS];
    __shared__ double dl[RED_THREADS];
    const int64_t per = (n_recs + RED_THREADS - 1) / RED_THREADS;
    MetricRec t = no_metrics();
    for (int64_t i = threadIdx.x * per; i < min(n_recs, (threadIdx.x + 1) * per); ++i) {
        const MetricRec x = recs[i];
        for (int k = 0; k < NMI; ++k) t.c[k] += x.c[k];
        t.reward = __dadd_rn(t.reward, x.reward);
    }
    double d[1] = {t.reward};
    block_tree_sum<int64_t, NMI>(t.c, il);
    block_tree_sum<double, 1>(d, dl);
    t.reward = d[0];
    if (threadIdx.x == 0) write_metrics(t, n_rows, metrics);
}

/* ------------------------------------------------------------------ per-group rewards */

/* One thread per row.  A group within one wave shares its values by shuffles
 * (group_reward_lanes); otherwise every thread of a group computes the group's
 * moments itself from memory.  Either way the sums run in the group's row
 * order, so every thread of a group holds the same values; a group takes G
 * threads instead of one, which keeps the GPU busy when a batch has few
 * groups (an RL step has 128).
 *
 * Rows listed for the deep tier (normally none) are evaluated here first, by
 * thread 0 of block 0; after a barrier that block computes the rewards of the
 * groups holding them (a group listed twice is written twice, with the same
 * values, and counted once).  Every block skips those groups: it tells them by
 * the MODE_DEEP mark, which nothing writes during this launch, so no block
 * reads a row another block is writing.
 *
 * With metrics the block sums them from the values it holds: a launch of its
 * own that read every row again took 7.8 us at 1,024 rows (15 us at 8,192),
 * and its combining launch 4 us more; up to RED_SINGLE rows one block does it
 * all (1,024 rows: 16.2 us in three launches, 8.9 us in one). */
template <bool LENIENT, bool METRICS>
__global__ void __launch_bounds__(METRICS ? RED_SINGLE : RED_THREADS)
group_reward(RewardArgs a, DeepArgs d, MetricRec *__restrict__ recs, double *__restrict__ metrics)
{
    __shared__ MetricRec lds[METRICS ? RED_WAVES : 1];
    __shared__ int32_t part[METRICS ? RED_WAVES : 1];
    const int32_t G = a.G;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    /* the row's values in the same round of loads as the deep count (rows of
     * groups the deep tier writes during this launch are not read from v) */
    const RowVals v = row_vals(a, min(r, a.n - 1));
    const int32_t n_deep = d.counters[1]; /* the same for every thread */
    MetricRec rec = no_metrics();
    if (n_deep > 0 && blockIdx.x == 0) {
        if (METRICS && n_deep > 1) order_deep_rows(d, a.n, part); /* their rewards' sum in row order */
        if (threadIdx.x == 0) run_deep_rows<LENIENT>(d.rows, d.mode, n_deep, d.deep_rows, d.frames, d.bits);
        __syncthreads();
        for (int64_t k0 = 0; k0 < (int64_t)n_deep * G; k0 += blockDim.x) {
            const int64_t k = k0 + threadIdx.x;
            bool count = k < (int64_t)n_deep * G;
            RowVals w = v;
            float R = 0.0f;
            if (count) {
                const int64_t rd = d.deep_rows[k / G], g0 = rd - rd % G, rk = g0 + k % G;
                R = group_reward_memory(a, rk);
                w = row_vals(a, rk);
                /* a group counts with its first deep row */
                for (int64_t i = g0; i < rd; ++i) count = count && (d.mode[i] & MODE_DEEP) == 0;
            }
            if (METRICS) block_metrics(count, w, R, lds, rec);
        }
    }
    bool mine = r < a.n; /* n is a multiple of G: whole groups only */
    if (n_deep > 0 && mine) {
        const int64_t r0 = r - r % G;
        for (int32_t i = 0; i < G; ++i) mine = mine && (d.mode[r0 + i] & MODE_DEEP) == 0; /* the same for a whole group */
    }
    float R = 0.0f;
    if (mine) {
        if (G == 8) R = group_reward_lanes<8>(a, r, G, v);
        else if (G <= WAVE && (G & (G - 1)) == 0) R = group_reward_lanes<0>(a, r, G, v);
        else R = group_reward_memory(a, r);
    }
    if (!METRICS) return;
    block_metrics(mine, v, R, lds, rec);
    put_metrics(rec, a.n, recs, metrics);
}

/* ------------------------------------------------------------------ batch-wide statistics */

/* Mean and sum of squared deviations of latency, Subtask ratio and Trial ratio
 * over some rows; two such sets merge by the pairwise update of Chan, Golub
 * and LeVeque ("Updating Formulae and a Pairwise Algorithm for Computing
 * Sample Variances", 1979), whose error is that of a two-pass sum. */
struct Moms {
    double n, mean[3], m2[3];
};

__device__ __forceinline__ Moms no_moms() { return Moms{0.0, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}}; }

__device__ __forceinline__ Moms merge_moms(const Moms &x, const Moms &y)
{
    if (y.n == 0.0) return x;
    if (x.n == 0.0) return y;
    Moms z;
    z.n = __dadd_rn(x.n, y.n);
    const double fy = __ddiv_rn(y.n, z.n), fxy = __dmul_rn(x.n, fy);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double d = __dsub_rn(y.mean[k], x.mean[k]);
        z.mean[k] = __dadd_rn(x.mean[k], __dmul_rn(d, fy));
        z.m2[k] = __dadd_rn(__dadd_rn(x.m2[k], y.m2[k]), __dmul_rn(__dmul_rn(d, d), fxy));
    }
    return z;
}

__device__ __forceinline__ Moms row_moms(const RowVals &v)
{
    return Moms{1.0, {(double)v.lat, ratio(v.ns, v.tot), ratio(v.nt, v.tot)}, {0.0, 0.0, 0.0}};
}

/* What of a row differs from another row: bit 0 latency, 1 Subtask ratio, 2
 * Trial ratio (exact, cross-multiplied). */
__device__ __forceinline__ uint32_t differs(const RowVals &v, const RowVals &w)
{
    const int64_t tv = v.tot > 0 ? v.tot : 1, tw = w.tot > 0 ? w.tot : 1;
    const int64_t sv = v.tot > 0 ? v.ns : 0, sw = w.tot > 0 ? w.ns : 0;
    const int64_t rv = v.tot > 0 ? v.nt : 0, rw = w.tot > 0 ? w.nt : 0;
    return (v.lat != w.lat ? 1u : 0u) | (sv * tw != sw * tv ? 2u : 0u) | (rv * tw != rw * tv ? 4u : 0u);
}

constexpr uint32_t NOT_EVAL_BIT = 8u; /* next to the three bits of differs() */

/* A tile of rows: its moments, one of its rows, and what differs between them. */
struct MomentRec {
    Moms m;
    RowVals first;
    uint32_t bits;
};
static_assert(2 * sizeof(MomentRec) <= 256, "a batch of one tile fits the smallest section");
static_assert(2 * sizeof(MomentRec) <= RED_THREADS * sizeof(int32_t), "a record per tile and one more");
static_assert(sizeof(MetricRec) <= 256, "a record per block of 256 rows");

/* Moments over the block and the OR of bits, in every thread: a butterfly over
 * the wave (lane 0's result counts), then the waves in order. */
__device__ __forceinline__ Moms block_moms(Moms m, uint32_t &bits, Moms *lds /* [RED_WAVES] */, uint32_t *lds_bits)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    for (int d = 1; d < WAVE; d <<= 1) {
        Moms o;
        o.n = __shfl(m.n, lane ^ d, WAVE);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            o.mean[k] = __shfl(m.mean[k], lane ^ d, WAVE);
            o.m2[k] = __shfl(m.m2[k], lane ^ d, WAVE);
        }
        m = merge_moms(m, o);
    }
    uint32_t b = 0;
#pragma unroll
    for (uint32_t k = 1; k <= NOT_EVAL_BIT; k <<= 1) b |= __ballot((bits & k) != 0) != 0 ? k : 0u;
    __syncthreads(); /* the values of a call before */
    if (lane == 0) {
        lds[wv] = m;
        lds_bits[wv] = b;
    }
    __syncthreads();
    m = lds[0];
    bits = lds_bits[0];
    for (int i = 1; i < (int)(blockDim.x / WAVE); ++i) {
        m = merge_moms(m, lds[i]);
        bits |= lds_bits[i];
    }
    return m;
}

/* Row r's reward under the batch's moments. */
__device__ __forceinline__ float batch_row(const RewardArgs &a, int64_t r, const RowVals &v, const Moms &m, uint32_t bits)
{
    if (bits & NOT_EVAL_BIT) return write_nan(a, r, v);
    const Moms x = row_moms(v);
    double z[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        z[k] = zscore(x.mean[k], Moments{m.mean[k], __dsqrt_rn(__ddiv_rn(m.m2[k], m.n))}, ((bits >> k) & 1u) == 0);
    return write_reward(a, r, v, z[0], z[1], z[2], x.mean[1], x.mean[2]);
}

__device__ __forceinline__ uint32_t row_bits(const RowVals &v, const RowVals &first)
{
    return differs(v, first) | ((v.fl & NOT_EVALUATED) ? NOT_EVAL_BIT : 0u);
}

/* The moments of each tile of RED_THREADS * rpt rows (rpt rows per thread).
 * The deep tier's rows (normally none) are left out of their tiles: block 0
 * evaluates them, on one thread, and leaves their moments as the record after
 * the last tile's (every other block skips them by their MODE_DEEP mark).  So
 * the statistics take one launch where four read the rows twice, a thread's
 * sixteen rows one after the other (8,192 rows: 40 us with the deep tier's own
 * launch, 5.4 us now). */
template <bool LENIENT>
__global__ void __launch_bounds__(RED_THREADS) batch_moments(RewardArgs a, DeepArgs d, MomentRec *__restrict__ recs,
                                                             int32_t rpt)
{
    __shared__ Moms lds[RED_WAVES];
    __shared__ uint32_t lds_bits[RED_WAVES];
    __shared__ int32_t part[RED_WAVES];
    __shared__ int64_t first_row;
    const int64_t t0 = (int64_t)blockIdx.x * RED_THREADS * rpt, t1 = min(a.n, t0 + (int64_t)RED_THREADS * rpt);
    const int32_t n_deep = d.counters[1];
    int64_t f = t0;
    if (n_deep > 0) {
        if (blockIdx.x == 0 && n_deep > 1) order_deep_rows(d, a.n, part); /* their moments merge in row order */
        if (threadIdx.x == 0) {
            if (blockIdx.x == 0) run_deep_rows<LENIENT>(d.rows, d.mode, n_deep, d.deep_rows, d.frames, d.bits);
            while (f < t1 && (d.mode[f] & MODE_DEEP)) ++f;
            first_row = f;
        }
        __syncthreads();
        f = first_row;
    }
    Moms m = no_moms();
    uint32_t bits = 0;
    RowVals first = row_vals(a, min(f, t1 - 1)); /* not used when every row of the tile is a deep one */
    for (int32_t j = 0; j < rpt; ++j) {
        const int64_t r = t0 + (int64_t)j * RED_THREADS + threadIdx.x; /* coalesced */
        if (r >= t1 || (n_deep > 0 && (d.mode[r] & MODE_DEEP))) continue;
        const RowVals v = row_vals(a, r);
        m = merge_moms(m, row_moms(v));
        bits |= row_bits(v, first);
    }
    m = block_moms(m, bits, lds, lds_bits);
    if (threadIdx.x == 0) recs[blockIdx.x] = MomentRec{m, first, bits};
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        MomentRec x{no_moms(), first, 0u};
        for (int32_t i = 0; i < n_deep; ++i) {
            const RowVals v = row_vals(a, d.deep_rows[i]);
            if (i == 0) x.first = v;
            x.m = merge_moms(x.m, row_moms(v));
            x.bits |= row_bits(v, x.first);
        }
        recs[gridDim.x] = x;
    }
}

/* One thread per row; every block merges the n_recs records of the batch itself. */
__global__ void __launch_bounds__(RED_THREADS) batch_reward(RewardArgs a, const MomentRec *__restrict__ moments,
                                                            int32_t n_recs, MetricRec *__restrict__ recs,
                                                            double *__restrict__ metrics)
{
    __shared__ Moms lds[RED_WAVES];
    __shared__ uint32_t lds_bits[RED_WAVES];
    __shared__ MetricRec lds_m[RED_WAVES];
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const RowVals v = row_vals(a, min(r, a.n - 1));
    int32_t f = 0; /* a record with rows */
    while (moments[f].m.n == 0.0) ++f;
    const RowVals first = moments[f].first;
    Moms m = no_moms();
    uint32_t bits = 0;
    for (int32_t i = threadIdx.x; i < n_recs; i += blockDim.x) {
        const MomentRec x = moments[i];
        if (x.m.n == 0.0) continue;
        m = merge_moms(m, x.m);
        bits |= x.bits | differs(x.first, first);
    }
    m = block_moms(m, bits, lds, lds_bits);
    float R = 0.0f;
    if (r < a.n) R = batch_row(a, r, v, m, bits);
    if (!metrics) return;
    MetricRec rec = no_metrics();
    block_metrics(r < a.n, v, R, lds_m, rec);
    put_metrics(rec, a.n, recs, metrics);
}

/* Up to RED_SINGLE rows in one block: the deep tier, the moments, the rewards
 * and the metrics. */
template <bool LENIENT>
__global__ void __launch_bounds__(RED_SINGLE) batch_single(RewardArgs a, DeepArgs d, double *__restrict__ metrics)
{
    __shared__ Moms lds[RED_WAVES];
    __shared__ uint32_t lds_bits[RED_WAVES];
    __shared__ MetricRec lds_m[RED_WAVES];
    const int64_t r = threadIdx.x;
    const int32_t n_deep = d.counters[1];
    if (n_deep > 0) {
        if (threadIdx.x == 0) run_deep_rows<LENIENT>(d.rows, d.mode, n_deep, d.deep_rows, d.frames, d.bits);
        __syncthreads();
    }
    const RowVals v = row_vals(a, min(r, a.n - 1)), first = row_vals(a, 0);
    const bool has = r < a.n;
    uint32_t bits = has ? row_bits(v, first) : 0u;
    const Moms m = block_moms(has ? row_moms(v) : no_moms(), bits, lds, lds_bits);
    float R = 0.0f;
    if (has) R = batch_row(a, r, v, m, bits);
    if (!metrics) return;
    MetricRec rec = no_metrics();
    block_metrics(has, v, R, lds_m, rec);
    put_metrics(rec, a.n, nullptr, metrics);
}

} /* namespace pk */
