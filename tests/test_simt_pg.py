"""The policy-gradient step runs on the CPU, under AddressSanitizer and
UndefinedBehaviorSanitizer, against the oracle.

The library's own csrc/pg.hip (with csrc/parason.hip for the segment plan) is
compiled for the host with the SIMT emulation of tests/simt/hip/hip_runtime.h,
and tests/simt/emu_pg.cpp drives it through the C-ABI.  Every batch runs with
the waves of a block in step, and with each wave run to its next barrier before
the next wave starts, from the first wave and from the last: the GPU promises
no order between barriers, and a barrier missing between one wave's read of
LDS and another's write gives other results in one of them."""
import os
import subprocess

import numpy as np
import pytest

from oracle import pg_oracle as PG
from paper_2608_24658_amd import parason as PX
from paper_2608_24658_amd.synth import synth as S
from test_gpu_pg import EPS_HI, EPS_LO, TOL, check_rows
from test_simt_emulation import CLANG, CSRC, ROOT, SIMT

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="no host clang++ with the sanitizers")

ORDERS = ("lockstep", "ahead", "ahead-reverse")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("simt_pg") / "emu_pg")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined", "-ffp-contract=off", "-I", SIMT,
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++",
                           os.path.join(CSRC, "parason.hip"), os.path.join(CSRC, "pg.hip"),
                           os.path.join(SIMT, "emu_pg.cpp"), "-o", out])
    return out


def run_emu(binary, reward, new, old, starts, lengths, G, cus, shift=0, in_place=False, waves="lockstep", tmp="/tmp"):
    n, n_tok = len(starts), new.size
    body = (np.array([n, n_tok], np.int64).tobytes() + np.array([G, cus, shift, int(in_place)], np.int32).tobytes()
            + np.array([EPS_LO, EPS_HI]).tobytes()
            + b"".join(np.ascontiguousarray(x, np.float32).tobytes() for x in (reward, new, old))
            + np.asarray(starts, np.int64).tobytes() + np.asarray(lengths, np.int32).tobytes())
    fin, fout = (os.path.join(tmp, "emu_pg_%s_%d.bin" % (k, os.getpid())) for k in ("in", "out"))
    with open(fin, "wb") as f:
        f.write(body)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1:abort_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1", SIMT_WAVES=waves)
    r = subprocess.run([binary, fin, fout], env=env, capture_output=True, text=True, timeout=600)
    if r.returncode != 0:
        raise RuntimeError("emulation failed (%d):\n%s" % (r.returncode, r.stderr[-4000:]))
    b = open(fout, "rb").read()
    os.unlink(fin)
    os.unlink(fout)
    assert np.frombuffer(b, np.int32, 1)[0] == PX.OK
    adv, grad = np.frombuffer(b, np.float32, n, 4), np.frombuffer(b, np.float32, n_tok, 4 + 4 * n)
    return adv, grad, np.frombuffer(b, np.float64, 4, 4 + 4 * (n + n_tok))


def batch(n, lo, hi, seed):
    """n rows of lo to hi tokens with gaps between them, their rewards and log-probabilities."""
    rng = np.random.default_rng(seed)
    lengths = rng.integers(lo, hi + 1, n).astype(np.int32)
    starts = np.cumsum(lengths.astype(np.int64) + rng.integers(0, 4, n)) - lengths
    old, new = S.host_logp(S.make_params(dict(seed=seed, len_kind=0, len_lo=lo, len_hi=hi)), 0, int(starts[-1] + lengths[-1]))
    reward = rng.choice(np.array([-1.0, 1.0, 1.25, 0.8], np.float32), n)
    return reward, new, old, starts, lengths


def check(binary, args, G, cus, what, **kw):
    reward, new, old, starts, lengths = args
    adv, grad, stats = run_emu(binary, *args, G, cus, **kw)
    want = PG.advantages(reward, G)
    assert np.all(np.abs(adv - want) <= 2.0 ** -24 * np.abs(want)), what
    exp = PG.surrogate(new, old, starts, lengths, want.astype(np.float32), EPS_LO, EPS_HI)
    inside = ~np.isnan(exp["grad"])
    assert np.all(grad[~inside] == np.float32(1e30)), (what, "a position outside the rows was written")
    clipped, a, n_bnd = check_rows(grad.astype(np.float64), exp, want.astype(np.float32), lengths, what)
    assert stats[1] == exp["tokens"], (what, stats, exp["tokens"])
    assert stats[2] == np.sum(clipped & (a > 0)) and stats[3] == np.sum(clipped & (a < 0)), (what, stats)
    slack = n_bnd * 2.0 ** -20 * np.max(np.abs(want)) / exp["tokens"]
    assert abs(stats[0] - exp["loss"]) <= TOL * max(1e-6, abs(exp["loss"])) + slack, (what, stats[0], exp["loss"])


# rows planned in LDS (fewer segments than waves, and more), and by launches
BATCHES = [(8, 1, 40, 8, 2), (64, 300, 1500, 8, 2), (600, 0, 300, 3, 2), (2048, 1, 60, 8, 2), (2056, 1, 60, 8, 2)]


@pytest.mark.parametrize("waves", ORDERS)
@pytest.mark.parametrize("n,lo,hi,G,cus", BATCHES)
def test_emulated_step(emu, n, lo, hi, G, cus, waves):
    check(emu, batch(n, lo, hi, n), G, cus, "n %d, %s" % (n, waves), shift=n % 4, waves=waves)


@pytest.mark.parametrize("n", [64, 2048, 2056])
def test_advantages_over_the_rewards(emu, n):
    """The advantages may be written over the rewards, at any batch size: the
    same advantages and gradients, bit for bit.  (A block that reads rewards
    another one has written over normalises advantages a second time, which
    changes their last bits.)"""
    args = batch(n, 1, 60, n + 1)
    apart, over = (run_emu(emu, *args, 8, 2, in_place=x) for x in (False, True))
    assert np.array_equal(over[0], apart[0]) and np.array_equal(over[1], apart[1])
    assert np.array_equal(over[2][1:], apart[2][1:])
    assert abs(over[2][0] - apart[2][0]) <= 1e-12 * abs(apart[2][0])  # the same terms in double, in another order
