"""Results read through the contexts' pinned blocks, and the best-ever records
when reads fall between eager generations, captured epochs and migrations: best
records, counters and makespans after every call equal the oracle's; contexts
created and destroyed in turn, and several alive at once, keep their results
apart; an invalid row's status is cleared for the next call and does not reach
another context."""
import numpy as np
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs
from paper_1903_10722_amd.binding import FFS_EINVAL, FFS_OK

pytestmark = pytest.mark.gpu


def test_reads_between_epochs():
    ensure_built()
    w = inputs.workload("tiny", seed=3)
    ctx, ga = make_ctx([w]), oracle_ga(w)
    for g in (0, 10, 1, 9, 20, 3, 7, 10, 10):     # captured epochs, eager generations, a mid-epoch start
        ctx.evolve(g)
        ga.evolve(g)
        for _ in range(2):
            b1, b2 = ctx.best(0), ga.best()
            assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), ctx.generation
            assert b1["perm"].tolist() == b2["perm"].tolist()
        assert ctx.migration_counters(0) == ga.counters()
        assert_same_state(ctx, ga, 0, 2, f"generation {ctx.generation}")
    ctx.close()


def test_contexts_side_by_side():
    ensure_built()
    ws = [inputs.workload("tiny", seed=s) for s in (4, 5, 6)]
    for _ in range(3):
        ctxs = [make_ctx([w]) for w in ws]
        bad = inputs.random_perms(70, 20, seed=1)
        bad[69, 0] = 20
        good = inputs.random_perms(70, 20, seed=2)
        assert ctxs[1].evaluate(0, bad, check=False)[1] == FFS_EINVAL
        assert ctxs[0].evaluate(0, good, check=False)[1] == FFS_OK
        assert ctxs[1].evaluate(0, good, check=False)[1] == FFS_OK
        for c, w in zip(ctxs, ws):
            c.evolve(12)
            ga = oracle_ga(w)
            ga.evolve(12)
            assert c.best(0)["makespan"] == ga.best()["makespan"]
            assert np.array_equal(c.population(0, 1)[1], ga.population(1)[1])
        for c in ctxs:
            c.close()
    say("[results] contexts side by side")
