"""GPU parity of the pipelined decode (one lane per stage) where its blocks,
its feeding lanes and its key formats have edges, against the oracle
(integers: equal).

Rows around the eight-step blocks and the 32-entry padding; one stage (every
lane feeds the next), 21, 32 and 64 stages (lane 63 idle, the last stage of the
last group, the last stage of the only one); lists of up to 16 machines; the
three key formats: completions that always fit beside the index, that may
outgrow it (rows of both kinds in one wave), and that do not fit."""
import numpy as np
import pytest

import oracle
from gpu_util import ensure_built, make_ctx, say
from paper_1903_10722_amd import inputs
from paper_1903_10722_amd.binding import FFS_EINVAL

pytestmark = pytest.mark.gpu

ISLANDS = [inputs.cellular(3, 3, 0.9, 0.1), inputs.pseudo(2, 0.75, 0.0)]


def _check(m, p, perms, mapping=0):
    w = dict(m=m, p=p, islands=ISLANDS, interval=0)
    ctx = make_ctx([w], mapping=mapping)
    got = ctx.evaluate(0, perms).cpu().numpy()
    want = oracle.decode_many(m, p, perms)
    assert np.array_equal(got, want), f"first mismatch at row {np.argmax(got != want)}"
    ctx.close()
    return want


SHAPES = [(n, 3, [2, 1, 3], 99) for n in (1, 2, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 40, 63, 65)] + [
    (50, 1, [3], 99), (41, 1, [1], 99), (30, 21, [2] * 21, 99), (30, 32, [1, 2] * 16, 99), (25, 64, [1] * 64, 99),
    (40, 4, [16, 9, 16, 1], 2), (300, 5, [6, 5, 8, 7, 1], 2), (129, 6, [4, 4, 1, 2, 4, 3], 3000), (1100, 2, [3, 4], 9)]


@pytest.mark.parametrize("n,S,m,p_hi", SHAPES)
def test_pipe_decode_edges(n, S, m, p_hi):
    ensure_built()
    m, p = inputs.make_instance(n, S, 1, 1, p_hi=p_hi, seed=n + S, machines=m)
    say(f"[pipe] n={n} S={S} m={m.tolist()} p<={p_hi}")
    _check(m, p, inputs.random_perms(67, n, seed=n))


def test_pipe_decode_outgrows_the_index():
    """1000 jobs of three types, each long (500) on its own single-machine
    stage: the lower bound is 167 000, random rows stay near it, rows sorted by
    type take 500 000, beyond the 262 142 that fit beside the index.  Both
    kinds share waves."""
    ensure_built()
    n, S = 1000, 3
    m = np.ones(S, dtype=np.int32)
    p = np.ones((n, S), dtype=np.int32)
    p[np.arange(n), np.arange(n) % S] = 500
    rng = np.random.default_rng(3)
    by_type = np.argsort(np.arange(n) % S, kind="stable")
    perms = np.asarray([by_type if r % 7 == 0 else rng.permutation(n) for r in range(150)], dtype=np.int32)
    say("[pipe] outgrows the index")
    want = _check(m, p, perms)
    assert (want[::7] > 262142).all() and (np.delete(want, np.s_[::7]) < 262142).all()


def test_pipe_decode_beyond_the_index():
    """A lower bound above the completions that fit beside the index."""
    ensure_built()
    m, p = inputs.make_instance(1000, 3, 1, 1, p_lo=900, p_hi=999, seed=4, machines=[1, 2, 1])
    say("[pipe] beyond the index")
    want = _check(m, p, inputs.random_perms(70, 1000, seed=9))
    assert (want > 262142).all()


@pytest.mark.parametrize("n", [5, 32, 45])
def test_pipe_decode_rejects_non_permutations(n):
    ensure_built()
    m, p = inputs.make_instance(n, 4, 1, 3, seed=n)
    ctx = make_ctx([dict(m=m, p=p, islands=ISLANDS, interval=0)], mapping=0)
    perms = inputs.random_perms(90, n, seed=3)
    perms[7, 4] = n
    perms[16, 0] = -1
    perms[17, 3] = perms[17, 0]
    perms[89, n - 1] = perms[89, 1]
    say(f"[pipe] invalid rows n={n}")
    out, rc = ctx.evaluate(0, perms, check=False)
    assert rc == FFS_EINVAL
    got, bad = out.cpu().numpy(), [7, 16, 17, 89]
    assert (got[bad] == -1).all()
    ok = np.setdiff1d(np.arange(90), bad)
    assert np.array_equal(got[ok], oracle.decode_many(m, p, perms[ok]))
    ctx.close()


@pytest.mark.parametrize("n,S,m,p_hi", [(511, 3, [2, 1, 3], 99), (512, 3, [2, 1, 3], 99), (513, 3, [2, 1, 3], 99),
                                        (512, 2, [8, 7], 2), (20, 20, [5] * 20, 65535), (600, 4, [4] * 4, 999)])
def test_lane_decode_formats(n, S, m, p_hi):
    """One lane per chromosome: the nine-bit job field and beyond it."""
    ensure_built()
    m, p = inputs.make_instance(n, S, 1, 1, p_hi=p_hi, seed=n + S, machines=m)
    say(f"[lane formats] n={n} S={S} p<={p_hi}")
    _check(m, p, inputs.random_perms(131, n, seed=n), mapping=1)


@pytest.mark.parametrize("n,long,cap", [(1000, 200, 131071), (512, 800, 262143), (1000, 500, 131071)])
def test_lane_decode_outgrows_the_index(n, long, cap):
    """Three job types, each long on its own single-machine stage: rows sorted
    by type outgrow the completion field beside the index, random rows do not
    (last case: the lower bound itself is beyond it)."""
    ensure_built()
    S = 3
    m = np.ones(S, dtype=np.int32)
    p = np.ones((n, S), dtype=np.int32)
    p[np.arange(n), np.arange(n) % S] = long
    rng = np.random.default_rng(3)
    by_type = np.argsort(np.arange(n) % S, kind="stable")
    perms = np.asarray([by_type if r % 7 == 0 else rng.permutation(n) for r in range(150)], dtype=np.int32)
    say(f"[lane formats] outgrows n={n} long={long}")
    want = _check(m, p, perms, mapping=1)
    assert (want[::7] > cap).all()
