"""The policy-gradient step where its plan changes hands: in LDS up to 2,048
rows, in launches beyond, one plan tile and several, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import pg_oracle as PO
from paper_2608_24658_amd import parason as PX
from paper_2608_24658_amd.synth import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,G", [(1, 1), (8, 8), (1024, 8), (2048, 8), (2048, 2048), (2049, 3), (2056, 8), (3000, 1), (9000, 8)])
def test_plan_boundaries(n, G):
    P = S.make_params(dict(seed=n, len_kind=1, len_lo=1, len_hi=2500))
    lengths, _ = S.host_rows(P, n)
    if n > 1:
        lengths[n // 2] = 0
    check(P, lengths, n, G)


@pytest.mark.parametrize("more", [-8, 0, 4008])
def test_range_per_wave(more):
    # one segment per row of at most 3 tokens: 2,048 segments per wave (16 waves
    # per CU) and beyond, where a wave takes one range in place of chunks
    n = torch.cuda.get_device_properties(0).multi_processor_count * 16 * 2048 + more
    lengths = np.random.default_rng(n).integers(1, 4, n).astype(np.int32)
    check(S.make_params(dict(seed=7, len_kind=1, len_lo=1, len_hi=3)), lengths, n, 8)


def check(P, lengths, n, G):
    N = int(lengths.astype(np.int64).sum())
    starts = np.concatenate([[0], np.cumsum(lengths[:-1].astype(np.int64))])
    old, new = S.host_logp(P, 0, N)
    reward = np.random.default_rng(n).choice(np.array([-1.0, 1.0, 1.25, 0.8], np.float32), n)
    dev = [torch.as_tensor(x).cuda() for x in (reward, new, old, starts, lengths)]
    got = PX.pg_run(*dev, group_size=G)
    some = min(n, 16384 // G * G)
    adv = PO.advantages(reward[:some], G)
    a32 = got["advantage"].cpu().numpy()
    # the same double expression in the same order, stored as float
    assert np.all(np.abs(a32[:some] - adv) <= 2.0 ** -24 * np.abs(adv))
    A = np.repeat(a32.astype(np.float64), lengths)
    d = new.astype(np.float64) - old.astype(np.float64)
    d32 = new - old
    hi, lo = np.float32(np.log1p(0.28)), np.float32(np.log1p(-0.2))
    clip_hi, clip_lo = (A > 0) & (d32 > hi), (A < 0) & (d32 < lo)  # the kernel's own decisions
    clipped = clip_hi | clip_lo
    grad = np.where(clipped, 0.0, -A * np.exp(d) / max(N, 1))
    g = got["grad"].cpu().numpy()
    # the kernel's exponential (2.2 ulp) and three float products
    assert np.all(np.abs(g - grad) <= 2.0 ** -20 * np.abs(grad))
    st = got["stats"].cpu().numpy()
    terms = np.where(clipped, np.where(clip_hi, 1.28, 0.8) * A, A * np.exp(d))
    assert st[1] == N and st[2] == clip_hi.sum() and st[3] == clip_lo.sum()
    assert abs(st[0] + terms.sum() / max(N, 1)) <= 2.0 ** -20 * np.abs(terms).sum() / max(N, 1)


@pytest.mark.parametrize("n", [64, 2048, 2056])
def test_advantages_over_the_rewards(n):
    """The advantages written over the rewards: the same advantages and gradients."""
    P = S.make_params(dict(seed=n, len_kind=1, len_lo=1, len_hi=2500))
    lengths, _ = S.host_rows(P, n)
    starts = np.concatenate([[0], np.cumsum(lengths[:-1].astype(np.int64))])
    old, new = S.host_logp(P, 0, int(lengths.astype(np.int64).sum()))
    reward = np.random.default_rng(n).choice(np.array([-1.0, 1.0, 1.25, 0.8], np.float32), n)
    r, lp, lo, st, ln = (torch.as_tensor(x).cuda() for x in (reward, new, old, starts, lengths))
    want = PX.pg_run(r, lp, lo, st, ln, group_size=8)
    grad, stats = torch.empty_like(lp), torch.empty(4, dtype=torch.float64, device="cuda")
    ws = torch.empty(PX.pg_workspace_size(n), dtype=torch.uint8, device="cuda")
    rc = PX.pg_run_raw(PX.PgConfig(8, 0.2, 0.28), r.data_ptr(), lp.data_ptr(), lo.data_ptr(), st.data_ptr(), ln.data_ptr(),
                       n, r.data_ptr(), grad.data_ptr(), stats.data_ptr(), ws.data_ptr(), ws.numel(),
                       torch.cuda.current_stream().cuda_stream)
    assert rc == PX.OK
    assert torch.equal(r, want["advantage"]) and torch.equal(grad, want["grad"])
    assert torch.equal(stats[1:], want["stats"][1:])
