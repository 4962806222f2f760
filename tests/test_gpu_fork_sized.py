"""Fork and join sized by the call itself (a sizing call, then the contexts
from what it left in the workspace) against calls with known capacities, on
both sides of the batch sizes where the launches change, and nothing to copy."""
import numpy as np
import pytest
import torch

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
