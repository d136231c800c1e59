"""Epochs of small islands run as one launch each, against the oracle's
trajectories and best-ever records (integers: equal): islands that fill one
workgroup's tile and of a few slots, rows at the ends of the vector
range, one and several stages per wave, both island kinds, intervals of one and
of none, several instances, and eager generations between the epochs."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu

# jobs, stages, machines per stage, interval, waves per workgroup, islands
CASES = [
    (20, 3, 3, 5, None, [inputs.cellular(8, 8, 0.9, 0.5), inputs.pseudo(64, 0.8, 0.4)]),
    (1, 1, 1, 1, None, [inputs.cellular(3, 3, 0.9, 0.5), inputs.pseudo(2, 0.8, 0.4)]),
    (9, 2, 8, 3, 1, [inputs.cellular(5, 6, 0.9, 0.5), inputs.cellular(3, 4, 0.9, 0.5)]),
    (72, 3, 2, 4, 8, [inputs.pseudo(160, 0.8, 0.4), inputs.cellular(4, 4, 0.9, 0.5)]),
    (24, 1, 16, 3, None, [inputs.cellular(10, 10, 0.9, 0.5)]),
    (300, 32, 2, 2, 8, [inputs.cellular(3, 5, 0.9, 0.5), inputs.pseudo(8, 0.8, 0.4)]),
    (9, 2, 2, 2, None, [inputs.cellular(16, 16, 0.9, 0.5), inputs.pseudo(258, 0.8, 0.4)]),   # counted on one workgroup, over several
    (9, 2, 2, 1, None, [inputs.cellular(37, 28, 0.9, 0.5), inputs.pseudo(4096, 0.8, 0.4)]),   # counted, over workgroups
    (9, 2, 2, 1, None, [inputs.cellular(4, 4, 0.9, 0.5), inputs.pseudo(4098, 0.8, 0.4)]),     # one too large for that
    (20, 3, 3, 0, None, [inputs.cellular(8, 8, 0.9, 0.5)]),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_epochs(case):
    ensure_built()
    n, S, mm, interval, wpb, isl = CASES[case]
    ws = []
    for i in range(2 if case in (0, 2) else 1):
        m, p = inputs.make_instance(n, S, 1, mm, p_hi=20, seed=n + S + i)
        ws.append(dict(m=m, p=p, islands=isl, interval=interval, theta=1.0, topology=0))
    say(f"[epochs] n={n} S={S} interval={interval} waves={wpb}")
    ctx = make_ctx(ws, waves_per_block=wpb, mapping=0)
    gas = [oracle_ga(w, inst=i) for i, w in enumerate(ws)]
    step = interval or 16
    for g in (step, 2 * step + 1, step - 1, 1, step, 3 * step):
        ctx.evolve(g)
        for i, ga in enumerate(gas):
            ga.evolve(g)
            what = f"instance {i} generation {ctx.generation}"
            b1, b2 = ctx.best(i), ga.best()
            assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), what
            assert b1["perm"].tolist() == b2["perm"].tolist(), what
            assert_same_state(ctx, ga, i, len(isl), what)
    ctx.close()


def test_epochs_between_tiles():
    """Tiles that make an island one workgroup's work and several's, in turn,
    and an eager start inside an epoch after each change."""
    ensure_built()
    w = inputs.workload("tiny", seed=9)
    ctx, ga = make_ctx([w], waves_per_block=8), oracle_ga(w)
    for waves, g in ((8, 20), (1, 10), (8, 13), (1, 7), (4, 25), (8, 15), (8, 20)):
        ctx.set_waves_per_block(waves)
        ctx.evolve(g)
        ga.evolve(g)
        say(f"[epochs] waves={waves} generation {ctx.generation}")
        b1, b2 = ctx.best(0), ga.best()
        assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), ctx.generation
        assert b1["perm"].tolist() == b2["perm"].tolist()
        assert ctx.migration_counters(0) == ga.counters()
        assert_same_state(ctx, ga, 0, 2, f"generation {ctx.generation}")
    ctx.close()
