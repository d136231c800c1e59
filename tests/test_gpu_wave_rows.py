"""GPU parity of children built by a whole wave, against the oracle's
trajectories (integers: equal): rows at the ends of every count of genes per
lane (1, 2, 4, 8, 16; registers up to 2048 genes, passes above), one lane per
chromosome, and of the pre-screen's candidates at the same row lengths."""
import numpy as np
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import Context, inputs

pytestmark = pytest.mark.gpu

ROWS = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 1536, 2047, 2048,
        2049, 4096]


@pytest.mark.parametrize("n", ROWS)
def test_wave_rows(n):
    ensure_built()
    m, p = inputs.make_instance(n, 2, 1, 3, p_hi=20, seed=n)
    isl = [inputs.cellular(5, 4, 0.9, 0.5), inputs.pseudo(22, 0.8, 0.4)]
    w = dict(m=m, p=p, islands=isl, interval=3, theta=1.0, topology=0)
    say(f"[wave rows] n={n}")
    ctx, ga = make_ctx([w], mapping=1), oracle_ga(w)
    for g in (0, 1, 3, 2):
        ctx.evolve(g)
        ga.evolve(g)
        assert_same_state(ctx, ga, 0, 2, f"n={n} generation {ctx.generation}")
    ctx.close()


@pytest.mark.parametrize("n", [9, 512, 513, 1024, 1025, 2048, 2049])
def test_candidate_rows(n):
    """The candidates' features do not depend on the kernel that builds them:
    one wave per cell, and (asked for with exact makespans) a group per row."""
    ensure_built()
    m, p = inputs.make_instance(n, 3, 1, 3, p_hi=20, seed=n)
    ctx = Context(device=0)
    ctx.add_instance(m, p, [inputs.cellular(4, 4, 0.9, 0.5), inputs.pseudo(4, 0.8, 0.4)], interval=0, seed=3,
                     surrogate_k=4, surrogate_warmup=1)
    ctx.bind()
    say(f"[wave rows] candidates n={n}")
    for _ in range(2):
        a = ctx.surrogate_candidates(0, exact=False, features=True)
        b = ctx.surrogate_candidates(0, exact=True, features=True)
        assert np.array_equal(a["features"], b["features"]), n
        ctx.evolve(2)
    ctx.close()
