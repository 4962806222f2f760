/*
 * pg.hip -- C-ABI of the policy-gradient step (kernels in pg_kernels.h).
 *
 * Launches use hipLaunchKernelGGL, as in parason.hip, so that the same source
 * also compiles against a host-side stand-in for the HIP runtime.
 */
#include "abi_common.h"
#include "pg_kernels.h"

using abi::ALIGN;
using abi::align_up;
using abi::cu_count;
using abi::is_finite;

namespace {

constexpr int PG_WAVES_PER_CU = 16;
constexpr int64_t PG_MAX_WAVES = 1 << 16;

struct PgLayout {
    size_t seg_off, counters, plan, n_tokens, wsum, wcnt, end;
};

PgLayout pg_layout_for(int64_t n)
{
    PgLayout L;
    const size_t rows = (size_t)(n > 0 ? n : 1);
    /* sizes that are no longer needed are kept, so that workspaces keep theirs */
    const size_t units = (rows + 4095) / 4096;
    size_t o = 0;
    L.seg_off = o;
    o = align_up(o + (size_t)(n + 1) * sizeof(int64_t));
    o = align_up(o + units * sizeof(int64_t));
    o = align_up(o + units * sizeof(int64_t));
    L.counters = o;
    o = align_up(o + 4 * sizeof(int32_t));
    /* a byte per row: 24 per PLAN_TILE rows, the plan's scratch and the tiles' token counts */
    L.plan = o;
    o = align_up(o + rows);
    o = align_up(o + units * sizeof(int64_t));
    L.n_tokens = o;
    o = align_up(o + sizeof(int64_t));
    L.wsum = o;
    o = align_up(o + (size_t)PG_MAX_WAVES * sizeof(double));
    L.wcnt = o;
    o = align_up(o + (size_t)PG_MAX_WAVES * 2 * sizeof(int64_t));
    L.end = o;
    return L;
}

}  // namespace

extern "C" {

int parason_pg_workspace_size(int64_t n_traj, size_t *bytes)
{
    if (!bytes) return PARASON_ERR_NULL;
    if (n_traj < 0 || n_traj > INT32_MAX) return PARASON_ERR_SIZE;
    *bytes = pg_layout_for(n_traj).end;
    return PARASON_OK;
}

int parason_pg_run(const parason_pg_config *cfg, const float *reward, const float *logp, const float *logp_old,
                   const int64_t *starts, const int32_t *lengths, int64_t n_traj, float *advantage, float *grad,
                   double *stats, void *workspace, size_t workspace_bytes, void *stream_ptr)
{
    if (!cfg) return PARASON_ERR_NULL;
    if (n_traj < 0 || n_traj > INT32_MAX) return PARASON_ERR_SIZE;
    if (cfg->group_size < 1 || n_traj % cfg->group_size != 0) return PARASON_ERR_GROUP;
    if (!is_finite(cfg->clip_low) || !is_finite(cfg->clip_high) || cfg->clip_low < 0.0 || cfg->clip_low >= 1.0 ||
        cfg->clip_high < 0.0)
        return PARASON_ERR_PARAM;
    if (n_traj == 0) return PARASON_OK;
    if (!reward || !logp || !logp_old || !starts || !lengths || !advantage || !grad || !stats || !workspace)
        return PARASON_ERR_NULL;
    const uintptr_t a0 = (uintptr_t)logp, a1 = (uintptr_t)logp_old, a2 = (uintptr_t)grad;
    if (((a0 | a1 | a2) & 3u) != 0 || (a0 & 15u) != (a1 & 15u) || (a0 & 15u) != (a2 & 15u) ||
        ((uintptr_t)workspace & (ALIGN - 1)) != 0)
        return PARASON_ERR_ALIGN;
    const PgLayout L = pg_layout_for(n_traj);
    if (workspace_bytes < L.end) return PARASON_ERR_WORKSPACE;
    const int cus = cu_count();
    if (cus <= 0) return PARASON_ERR_DEVICE;
    const int64_t waves = (int64_t)cus * PG_WAVES_PER_CU;
    if (waves > PG_MAX_WAVES) return PARASON_ERR_DEVICE;
    hipStream_t stream = (hipStream_t)stream_ptr;

    const int64_t mis = (int64_t)((a0 & 15u) >> 2);
    char *ws = (char *)workspace;
    int64_t *n_tokens = (int64_t *)(ws + L.n_tokens);
    double *wsum = (double *)(ws + L.wsum);
    int64_t *wcnt = (int64_t *)(ws + L.wcnt);

    pk::PgArgs pa;
    pa.logp_base = logp - mis;
    pa.old_base = logp_old - mis;
    pa.grad_base = grad - mis;
    pa.mis = mis;
    pa.starts = starts;
    pa.lengths = lengths;
    pa.n = n_traj;
    pa.seg_off = (int64_t *)(ws + L.seg_off);
    pa.reward = reward;
    pa.G = cfg->group_size;
    pa.adv = advantage;
    pa.thr_low = (float)std::log1p(-cfg->clip_low);
    pa.thr_high = (float)std::log1p(cfg->clip_high);
    pa.lo_val = (float)(1.0 - cfg->clip_low);
    pa.hi_val = (float)(1.0 + cfg->clip_high);
    pa.n_tokens = n_tokens;
    pa.wsum = wsum;
    pa.wcnt = wcnt;
    /* Blocks that plan the batch themselves all read the rewards while the
     * first of them writes the advantages: a caller's advantages over the
     * rewards take the launches, where each group's thread reads its rewards
     * before it writes. */
    const bool in_place = advantage < reward + n_traj && reward < advantage + n_traj;
    const bool plan = n_traj <= pk::SCAN_PLAN_ROWS && !in_place;
    const int64_t blocks = waves / (plan ? pk::PG_PLAN_WAVES : pk::PG_WAVES);
    if (plan) {
        hipLaunchKernelGGL(pk::pg_surrogate<true>, dim3((unsigned)blocks), dim3(pk::PG_PLAN_WAVES * pk::WAVE), 0,
                           stream, pa);
    } else {
        const int64_t tiles = abi::plan_tile_count(n_traj), n_groups = n_traj / cfg->group_size;
        const int64_t group_blocks = (n_groups + pk::PLAN_THREADS - 1) / pk::PLAN_THREADS;
        int64_t *scratch = (int64_t *)(ws + L.plan), *len_sum = scratch + 2 * tiles;
        hipLaunchKernelGGL(pk::pg_prepare, dim3((unsigned)(tiles > group_blocks ? tiles : group_blocks)),
                           dim3(pk::PLAN_THREADS), 0, stream, pa, tiles, n_groups, scratch, len_sum);
        abi::launch_plan(starts, lengths, n_traj, mis, scratch, (int64_t *)(ws + L.seg_off),
                         (int32_t *)(ws + L.counters), nullptr, len_sum, n_tokens, stream);
        hipLaunchKernelGGL(pk::pg_surrogate<false>, dim3((unsigned)blocks), dim3(pk::PG_WAVES * pk::WAVE), 0, stream,
                           pa);
    }
    hipLaunchKernelGGL(pk::pg_final, dim3(1), dim3(pk::RED_THREADS), 0, stream, wsum, wcnt, blocks, n_tokens, stats);
    return hipGetLastError() == hipSuccess ? PARASON_OK : PARASON_ERR_HIP;
}

}  // extern "C"
