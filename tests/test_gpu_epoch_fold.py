"""Best-ever records after one-launch epochs of many small instances, against
the oracle's (integers: equal): one wave of the folding workgroups per instance
(sixteen to a workgroup beside the migration, four where nothing migrates), and
more islands than lanes."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu

PAIR = [inputs.cellular(3, 4, 0.9, 0.5), inputs.pseudo(12, 0.8, 0.4)]


@pytest.mark.parametrize("count,interval,islands", [(33, 2, PAIR), (5, 0, PAIR), (2, 2, PAIR * 33), (2, 0, PAIR * 33)],
                         ids=["instances", "no_migration", "islands", "islands_no_migration"])
def test_records(count, interval, islands):
    ensure_built()
    kinds = sorted(islands, key=lambda x: x["kind"])          # pairs are (i, i + H)
    ws = []
    for i in range(count):
        m, p = inputs.make_instance(30, 4, 2, 3, seed=i)
        ws.append(dict(m=m, p=p, islands=kinds, interval=interval, theta=1.0, topology=0))
    say(f"[epoch fold] {count} instances of {len(kinds)} islands, interval {interval}")
    ctx = make_ctx(ws, mapping=0)
    gas = [oracle_ga(w, inst=i) for i, w in enumerate(ws)]
    found = set()
    for g in (16, 16, 5, 11, 32):
        ctx.evolve(g)
        for i, ga in enumerate(gas):
            ga.evolve(g)
            what = f"instance {i} generation {ctx.generation}"
            b1, b2 = ctx.best(i), ga.best()
            assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), what
            assert b1["perm"].tolist() == b2["perm"].tolist(), what
            found.add(b2["generation"])
    assert len(found) > 2, found
    for i in (0, count - 1):
        assert_same_state(ctx, gas[i], i, len(kinds), f"instance {i}")
    ctx.close()
