"""The row kernels where the scan cannot store a segment's events: outlines so
dense that a scan wave's pool region runs out (rows are then read again by the
wave that evaluates them), at the batch sizes where the kernels change, against
the oracle.  On the CPU the emulated build gets a small pool, on the GPU the
batches are large enough to use the real one up."""
import os
import subprocess

import numpy as np
import pytest

import grammar_pins as GP
from adversarial import adversarial_streams, deep_stream, pack
from gpu_util import DEFAULT_COEF, compare, insert_gaps, oracle_expect
from oracle import oracle as O
from paper_2608_24658_amd import parason as PX
from paper_2608_24658_amd.synth import synth as S
from test_gpu_metrics import check_metrics
from test_simt_emulation import CLANG, CSRC, FEW, MANY, ROOT, SIMT, TAGS, check, run_emu

G = 8


def short_rows(n, lo, hi, seed, tags=TAGS, len_kind=0, **kw):
    P = S.make_params(dict(seed=seed, len_kind=len_kind, len_lo=lo, len_hi=hi, **kw), tag_ids=tags)
    return S.host_batch(P, n)


@pytest.fixture(scope="module")
def emu_small_pool(tmp_path_factory):
    """Four slots per segment and 512 in all: most ranges run out."""
    if not os.path.exists(CLANG):
        pytest.skip("no host clang++ with the sanitizers")
    out = str(tmp_path_factory.mktemp("rows") / "emu")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined", "-ffp-contract=off", "-DPARASON_POOL_MIN=512", "-I", SIMT,
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                           os.path.join(CSRC, "parason.hip"), os.path.join(SIMT, "emu_main.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("cus", [MANY, FEW])
@pytest.mark.parametrize("tags", ["contiguous", "scattered"])
def test_unstored_segments(emu_small_pool, cus, tags):
    """Rows of 1 to 3,000 tokens (one to four segments each, some cut off),
    on every kind of batch: the scan's own plan and the larger ones."""
    ids = TAGS if tags == "contiguous" else S.SCATTERED_TAGS
    tok, st, ln, co = short_rows(320, 1, 3000, 11, ids, len_kind=1, p_trunc=0.1, p_trigger=1.0)
    for shift in (0, 3):
        check(emu_small_pool, tok, st, ln, co, ids, cus=cus, shift=shift, what="unstored cus %d shift %d" % (cus, shift))
    P = S.make_params("small", tag_ids=ids)
    t2, s2, l2, c2 = S.host_batch(P, 64)
    rng = np.random.default_rng(5)
    rows = [insert_gaps(t2[s2[i]: s2[i] + l2[i]], ids, rng) for i in range(64)]
    lengths = np.array([r.size for r in rows], np.int32)
    starts = np.concatenate([[0], np.cumsum(lengths[:-1])]).astype(np.int64)
    check(emu_small_pool, np.concatenate(rows), starts, lengths, c2, ids, flags=PX.CFG_LENIENT_GAPS, cus=cus,
          what="unstored, lenient")


@pytest.mark.parametrize("cus", [16, FEW])
def test_unstored_segments_adversarial(emu_small_pool, cus):
    """Strings the row kernels hand on (too many events, too deep) next to
    ones they hold, with most lists unstored."""
    tokens, starts, lengths = pack(adversarial_streams(), TAGS)
    correct = (np.arange(lengths.size) % 3 != 0).astype(np.uint8)
    check(emu_small_pool, tokens, starts, lengths, correct, cus=cus, what="unstored adversarial")


@pytest.mark.parametrize("n", [1024, 1032])
def test_emulated_batch_statistics(emu_small_pool, n):
    """One block and several, with rows of the deep tier among them."""
    tokens, starts, lengths = pack(with_deep_rows(n, n), S.CONTIGUOUS_TAGS)
    correct = (np.arange(n) % 3 != 0).astype(np.uint8)
    check(emu_small_pool, tokens, starts, lengths, correct, flags=PX.CFG_BATCH_STATS, cus=MANY, what="batch stats")


@pytest.mark.parametrize("flags", [0, PX.CFG_BATCH_STATS])
@pytest.mark.parametrize("n,cus", [(1024, MANY), (1032, MANY), (2056, FEW)])
def test_emulated_deep_rows_in_any_order(emu_small_pool, n, cus, flags):
    """The deep tier's list is filled by atomics, so its order is the
    scheduler's.  The rewards, the batch statistics and the metrics of blocks run
    in index order and from the last to the first: bit for bit the same.  So that
    an order shows, the mean latency is a whole number that one row has, and a
    weight of 1e18 makes that row's reward under batch statistics the rounding
    error of the mean; without them a weight of 1e15 next to the -1 of wrong
    answers makes the sum of the rewards inexact."""
    streams = with_deep_rows(n, n, [int(x) for x in np.random.default_rng(n).integers(66, 130, 200)])
    rest = int(oracle_latency(streams[2:]).sum())
    mean = rest // (n - 2) + 2
    streams[1:3] = [[GP.THINK] + [GP.TEXT] * (k - 2) + [GP.END_THINK] for k in (mean, 2)]
    fill = n * mean - int(oracle_latency(streams).sum()) + 2
    assert fill >= 2
    streams[2] = [GP.THINK] + [GP.TEXT] * (fill - 2) + [GP.END_THINK]
    tokens, starts, lengths = pack(streams, TAGS)
    correct = (np.arange(n) % 3 != 0).astype(np.uint8)
    coef = dict(alpha=1e18 if flags else 1e15, beta_subtask=0.0, beta_trial=0.0, rho=0.5, rho_clip=0.25)
    got, back = (run_emu(emu_small_pool, tokens, starts, lengths, correct, flags=flags, cus=cus, coef=coef, metrics=True,
                         blocks=x, divergent=True)[0] for x in ("forward", "reverse"))
    for k in got:
        assert np.array_equal(got[k], back[k], equal_nan=True), k
    rows, R, rs, rt, eta = oracle_expect(tokens, starts, lengths, correct, TAGS, G, coef, flags)
    if not flags:
        compare(got, rows, R, rs, rt, eta, what="deep rows")
        check_metrics(got["metrics"], rows, correct, R)


def nested_stream(rng, k, depth, per_level=1):
    """depth levels of blocks with k entries (and k threads, or one more or less
    now and then), per_level of a block's threads holding a block of the next
    level, so that a level's list holds 2 k + 3 tags per block and one more per
    block directly inside."""
    def block(d):
        s = [GP.PAR, GP.OUT]
        for _ in range(k):
            o, c = (GP.SUB, GP.END_SUB) if rng.random() < 0.5 else (GP.TRI, GP.END_TRI)
            s += [o] + [GP.TEXT] * int(rng.integers(1, 3)) + [c]
        s += [GP.END_OUT]
        n = max(1, k + int(rng.choice([0, 0, 0, 0, 1, -1])))
        inside = set(rng.choice(n, min(n, per_level), replace=False).tolist()) if d > 1 else set()
        for j in range(n):
            s += [GP.THR] + [GP.TEXT] * int(rng.integers(0, 4)) + (block(d - 1) if j in inside else [])
            s += [GP.TEXT] * int(rng.integers(0, 3)) + [GP.END_THR]
        return s + [GP.END_PAR]
    return [GP.THINK] + block(depth) + [GP.END_THINK]


def list_streams():
    """Rows whose levels' lists end at 16, 32, 64 and 128 entries and more, over
    every number of events per lane and up to the deepest row a wave holds."""
    rng = np.random.default_rng(17)
    shapes = [(6, 3, 1), (7, 3, 1), (14, 3, 1), (15, 3, 1), (30, 3, 1), (31, 3, 1), (62, 3, 1), (1, 20, 1), (1, 21, 1),
              (1, 62, 1), (1, 64, 1), (1, 65, 1), (2, 5, 2), (3, 4, 3), (2, 6, 2), (4, 3, 4), (5, 3, 4), (40, 2, 1),
              (60, 2, 1), (9, 2, 9), (2, 3, 1), (2, 12, 1), (3, 8, 1), (4, 13, 1)]
    return [nested_stream(rng, *x) for x in shapes for _ in range(4)]


@pytest.mark.parametrize("cus", [MANY, FEW])
def test_emulated_level_lists(emu_small_pool, cus):
    """With most lists of the scan unstored and with all of them stored."""
    streams = list_streams()
    for gap in (0, 60):  # text after each row, so that its segments' share of the pool holds its tags
        tokens, starts, lengths = pack([s + [GP.TEXT] * (gap * len(s)) for s in streams], TAGS)
        correct = (np.arange(lengths.size) % 3 != 0).astype(np.uint8)
        check(emu_small_pool, tokens, starts, lengths, correct, cus=cus, what="level lists cus %d" % cus)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1024, 20000])
def test_level_lists_on_the_gpu(n):
    import torch

    streams = list_streams()
    for gap in (0, 20):
        tokens, starts, lengths = pack([s + [GP.TEXT] * (gap * len(s)) for s in streams], S.CONTIGUOUS_TAGS)
        m = lengths.size
        pick = np.arange(n) % m
        co = (np.arange(n) % 3 != 0).astype(np.uint8)
        px = PX.Parason(S.CONTIGUOUS_TAGS, group_size=G, **DEFAULT_COEF)
        dev = [torch.as_tensor(x).cuda() for x in (tokens, starts[pick], lengths[pick], co)]
        got = {k: v.cpu().numpy() for k, v in px.run(*dev, total_tokens=int(lengths[pick].astype(np.int64).sum())).items()}
        got["flags"] = got["flags"].view(np.uint32)
        compare(got, *oracle_expect(tokens, starts[pick], lengths[pick], co, S.CONTIGUOUS_TAGS, G, DEFAULT_COEF, 0),
                what="level lists %d gap %d" % (n, gap))


def oracle_latency(streams):
    tokens, starts, lengths = pack(streams, TAGS)
    return O.eval_rows(tokens, starts, lengths, TAGS)["latency"]


@pytest.mark.gpu
@pytest.mark.parametrize("n,lo,hi,kind", [(2048, 1750, 5250, 0), (2056, 350, 1050, 0), (8192, 1, 2100, 1),
                                          (16384, 350, 1050, 0), (16392, 350, 1050, 0), (40000, 300, 900, 0)])
def test_rows_on_the_gpu(n, lo, hi, kind):
    """Outline-heavy batches over the sizes where the row kernels change."""
    import torch

    P = S.make_params(dict(seed=n, len_kind=kind, len_lo=lo, len_hi=hi, p_trigger=1.0, p_trunc=0.02))
    tok, st, ln, co = S.host_batch(P, n)
    dev = [torch.as_tensor(x).cuda() for x in (tok, st, ln, co)]
    for flags in (0, PX.CFG_LENIENT_GAPS):
        px = PX.Parason(S.CONTIGUOUS_TAGS, group_size=G, flags=flags, **DEFAULT_COEF)
        got = {k: v.cpu().numpy() for k, v in px.run(*dev, total_tokens=tok.size).items()}
        got["flags"] = got["flags"].view(np.uint32)
        compare(got, *oracle_expect(tok, st, ln, co, S.CONTIGUOUS_TAGS, G, DEFAULT_COEF, flags),
                what="rows %d flags %d" % (n, flags))


@pytest.mark.gpu
def test_adversarial_rows_in_a_large_batch_on_the_gpu():
    """17,000 rows (four per wave): strings of every kind the row kernels hand
    on, next to ones they hold, down to the deep tier."""
    import torch

    streams = adversarial_streams()
    tokens, starts, lengths = pack([streams[i % len(streams)] for i in range(17000)], S.CONTIGUOUS_TAGS)
    correct = (np.arange(lengths.size) % 3 != 0).astype(np.uint8)
    dev = [torch.as_tensor(x).cuda() for x in (tokens, starts, lengths, correct)]
    px = PX.Parason(S.CONTIGUOUS_TAGS, group_size=G, **DEFAULT_COEF)
    got = {k: v.cpu().numpy() for k, v in px.run(*dev, total_tokens=tokens.size).items()}
    got["flags"] = got["flags"].view(np.uint32)
    compare(got, *oracle_expect(tokens, starts, lengths, correct, S.CONTIGUOUS_TAGS, G, DEFAULT_COEF),
            what="adversarial, large batch")
    assert got["max_depth"].max() >= 1000


def with_deep_rows(n, seed, depths=(80, 80, 80, 80)):
    """Short rows with a few the deep tier evaluates, two of them in one group and one in the last."""
    rng = np.random.default_rng(seed)
    valid = [list(x) for x in GP.enumerate_valid(14)]
    streams = [valid[int(k)] for k in rng.integers(0, len(valid), n)]
    rows = sorted({0, 3, n // 2, n - 1} | {int(i) for i in rng.integers(0, n, max(0, len(depths) - 4))})
    for i, depth in zip(rows, depths):
        streams[i] = deep_stream(depth)
    return streams


@pytest.mark.gpu
@pytest.mark.parametrize("deep", [False, True])
@pytest.mark.parametrize("n", [8, 1024, 1032, 65536, 65544])
def test_batch_reductions_on_the_gpu(n, deep):
    """Metrics and batch-wide statistics where their blocks and records change:
    one block up to 1,024 rows, one row per thread up to 65,536."""
    import torch

    if deep:
        tok, st, ln = pack(with_deep_rows(n, n), S.CONTIGUOUS_TAGS)
        co = (np.arange(n) % 3 != 0).astype(np.uint8)
    else:
        tok, st, ln, co = short_rows(n, 20, 120, n)
    dev = [torch.as_tensor(x).cuda() for x in (tok, st, ln, co)]
    for flags in (0, PX.CFG_BATCH_STATS):
        px = PX.Parason(S.CONTIGUOUS_TAGS, group_size=G, flags=flags, **DEFAULT_COEF)
        out = px.run(*dev, total_tokens=tok.size, metrics=True)
        got = {k: v.cpu().numpy() for k, v in out.items()}
        got["flags"] = got["flags"].view(np.uint32)
        rows, R, rs, rt, eta = oracle_expect(tok, st, ln, co, S.CONTIGUOUS_TAGS, G, DEFAULT_COEF, flags)
        compare(got, rows, R, rs, rt, eta, what="n %d flags %d" % (n, flags), exact_reward=not flags)
        check_metrics(got["metrics"], rows, co, R)


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, PX.CFG_BATCH_STATS])
def test_millions_of_rows_on_the_gpu(flags):
    """Past 4,194,304 rows: the plan's own launch over the tiles (plan_top), and
    batch statistics whose number of records no longer grows with the batch.  Rows
    of two to four tokens (some cut off), every output and the metrics."""
    import torch

    n = (1 << 22) + 1032
    t = S.CONTIGUOUS_TAGS
    tok = np.tile(np.array([t[0], 5, 6, t[1]], np.int32), n)
    rng = np.random.default_rng(4)
    ln = np.where(rng.random(n) < 0.8, 4, rng.integers(0, 4, n)).astype(np.int32)
    st = np.arange(n, dtype=np.int64) * 4
    co = (rng.random(n) < 0.5).astype(np.uint8)
    px = PX.Parason(t, group_size=G, flags=flags, **DEFAULT_COEF)
    dev = [torch.as_tensor(x).cuda() for x in (tok, st, ln, co)]
    got = {k: v.cpu().numpy() for k, v in px.run(*dev, total_tokens=int(ln.sum()), metrics=True).items()}
    got["flags"] = got["flags"].view(np.uint32)
    rows, R, rs, rt, eta = oracle_expect(tok, st, ln, co, t, G, DEFAULT_COEF, flags)
    compare(got, rows, R, rs, rt, eta, what="millions", exact_reward=not flags)
    check_metrics(got["metrics"], rows, co, R)
