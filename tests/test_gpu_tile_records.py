"""Best-ever records across changes of the launch chains, the mapping and the
tile that directly follow a generation, without a read in between: they equal
the oracle's."""
import pytest

from gpu_util import ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu

CHANGES = {
    "chains": [lambda c: c.set_chains(1), lambda c: c.set_chains(2)],
    "mapping": [lambda c: c.set_mapping(1), lambda c: c.set_mapping(0)],
    "tile": [lambda c: c.set_instance_tile(0, 1, 2), lambda c: c.set_instance_tile(0, 0, 8)],
}


@pytest.mark.parametrize("what", list(CHANGES))
def test_records_across_changes(what):
    ensure_built()
    for seed in range(4):
        isl = [inputs.cellular(6, 6, 0.9, 0.4)] * 2 + [inputs.pseudo(36, 0.8, 0.3)] * 2
        ws = []
        for i in range(1 if what == "chains" else 2):
            m, p = inputs.make_instance(40 - 10 * i, 6, 2, 4, seed=seed + 10 * i)
            ws.append(dict(m=m, p=p, islands=isl, interval=0))
        say(f"[tile records] {what} seed={seed}")
        ctx = make_ctx(ws, mapping=0)
        ctx.set_chains(2)
        gas = [oracle_ga(w, inst=i) for i, w in enumerate(ws)]
        for step, g in enumerate((1, 1, 1, 2, 1, 1, 3, 1, 1)):
            ctx.evolve(g)
            CHANGES[what][step % 2](ctx)
            for i, ga in enumerate(gas):
                ga.evolve(g)
                b1, b2 = ctx.best(i), ga.best()
                assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), (seed, step, i)
                assert b1["perm"].tolist() == b2["perm"].tolist()
        ctx.close()
