"""Contexts whose instances all migrate along the edges of the ring (topology 2,
no island pairs): populations, counters and best records against the oracle's,
with two and more islands, one and several workgroups an island, one and two
instances, in captured epochs and in eager generations."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs,side,count,graphs", [(1, 4, 1, True), (2, 8, 1, True), (3, 16, 2, True), (2, 4, 2, False)])
def test_only_ring_edges(pairs, side, count, graphs):
    ensure_built()
    isl = [inputs.cellular(side, side, 0.9, 0.3)] * pairs + [inputs.pseudo(side * side, 0.75, 0.2)] * pairs
    ws = []
    for i in range(count):
        m, p = inputs.make_instance(30, 4, 1, 4, seed=7 + i)
        ws.append(dict(m=m, p=p, islands=isl, interval=3, theta=1.0, topology=2))
    say(f"[ring edges] {count} instances of {len(isl)} islands of {side * side}")
    ctx = make_ctx(ws)
    ctx.set_graphs(graphs)
    gas = [oracle_ga(w, inst=i) for i, w in enumerate(ws)]
    for g in (3, 6, 2, 1):
        ctx.evolve(g)
        for i, ga in enumerate(gas):
            ga.evolve(g)
            assert_same_state(ctx, ga, i, len(isl), f"instance {i} generation {ctx.generation}")
            assert ctx.migration_counters(i) == ga.counters()
            b1, b2 = ctx.best(i), ga.best()
            assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"])
            assert b1["perm"].tolist() == b2["perm"].tolist()
    ctx.migrate(0)
    gas[0].migrate()
    assert_same_state(ctx, gas[0], 0, len(isl), "after a forced epoch")
    assert ctx.migration_counters(0) == gas[0].counters()
    ctx.close()
