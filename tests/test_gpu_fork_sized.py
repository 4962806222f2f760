"""Fork and join sized by the call itself (a sizing call, then the contexts
from what it left in the workspace) against calls with known capacities, on
both sides of the batch sizes where the launches change, and nothing to copy."""
import numpy as np
import pytest
import torch

from oracle import fork_oracle as F
from paper_2608_24658_amd import parason as PX
from paper_2608_24658_amd.synth import synth as S

pytestmark = pytest.mark.gpu
TAGS = S.CONTIGUOUS_TAGS


@pytest.mark.parametrize("n,forks", [(1, True), (48, True), (1024, True), (1025, True), (2048, True), (2049, True), (4104, True), (64, False)])
def test_sized_by_the_call(n, forks):
    P = S.make_params(dict(seed=n, len_kind=0, len_lo=300, len_hi=900))
    tok, st, ln, _ = S.host_batch(P, n)
    rng = np.random.default_rng(n)
    if forks:  # cut each row after one of its outlines
        for i in range(n):
            ends = np.nonzero(tok[st[i]: st[i] + ln[i]] == TAGS[5])[0]
            if ends.size:
                ln[i] = int(rng.choice(ends)) + 1
    dev = [torch.as_tensor(x).cuda() for x in (tok, st, ln)]
    for seed in (True, False):
        px = PX.Parason(TAGS)
        a = px.fork(*dev, seed=seed)
        W, T, over = a["totals"].tolist()
        assert over == 0 and (W > 0 or not forks or n == 1)
        b = px.fork(*dev, seed=seed, max_workers=W, ctx_capacity=T)
        for k in b:
            assert torch.equal(a[k], b[k]), k
    wtok, wst, wln = a["ctx_tokens"], a["ctx_starts"], a["ctx_lengths"]
    c = px.join(*dev, a["worker_off"], wtok, wst, wln)
    d = px.join(*dev, a["worker_off"], wtok, wst, wln, capacity=int(c["totals"][0]))
    for k in d:
        assert torch.equal(c[k], d[k]), k


@pytest.mark.parametrize("n", [120, 1024, 1025])
@pytest.mark.parametrize("lenient", [False, True])
def test_outlines_around_the_window(n, lenient):
    """Outlines that begin inside, right at and before the last 2,048 tokens a
    block looks at, and rows with more tags there than its list holds, in a
    batch of one block per row and in one of one wave per row: the same."""
    think, _, par, _, out, end_out, sub, end_sub, tri, end_tri = (int(x) for x in TAGS[:10])

    def row(before, entries, gap=0):
        r = [think] + [7] * before + [par] + [9] * gap + [out]
        for k, text in enumerate(entries):
            r += [sub, *[11] * text, end_sub] if k % 2 else [tri, *[11] * text, end_tri]
        return r + [end_out]

    kinds = []
    for total in range(2038, 2056):  # tokens from <Outlines> to the row's end around the window
        kinds.append(row(5, [total - 8, 1]))
        kinds.append(row(3000, [total - 8, 1]))
    kinds += [row(10, [1] * k) for k in (1, 8, 9, 250, 254, 255, 256, 300)]  # 2 tags an entry
    kinds += [row(0, [3, 0]), row(2, [5, 5], gap=2), [think, 7, end_out], [end_out], row(4, [2])[:-1], [out, end_out],
              [par, out, end_out], [7] * 2500 + [end_out], row(2, []), []]
    rows = [kinds[i % len(kinds)] for i in range(n)]
    lengths = np.array([len(r) for r in rows], np.int32)
    starts = np.concatenate([[0], np.cumsum(lengths[:-1])]).astype(np.int64)
    dev = [torch.as_tensor(x).cuda() for x in (np.concatenate([np.asarray(r, np.int32) for r in rows]), starts, lengths)]
    px = PX.Parason(TAGS, flags=PX.CFG_LENIENT_GAPS if lenient else 0)
    got = px.fork(*dev)
    m = len(kinds)
    ref = F.fork(kinds, TAGS, F.FORK_SEED_ENTRY, lenient)
    st, off = got["row_status"].cpu().numpy(), got["worker_off"].cpu().numpy()
    cs, cl = got["ctx_starts"].cpu().numpy(), got["ctx_lengths"].cpu().numpy()
    ct, kind = got["ctx_tokens"].cpu().numpy(), got["ctx_kind"].cpu().numpy()
    for i in range(n):
        a, b = ref["worker_off"][i % m], ref["worker_off"][i % m + 1]
        assert st[i] == ref["status"][i % m], (i, st[i])
        assert off[i + 1] - off[i] == b - a, i
        if i < m or n - i <= m:
            for k in range(b - a):
                j = off[i] + k
                assert (kind[j] == 2) == (ref["kind"][a + k] == F.TRI) and np.array_equal(ct[cs[j]: cs[j] + cl[j]], ref["ctx"][a + k]), (i, k)
