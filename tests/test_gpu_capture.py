"""Generations that the caller captures into a graph of their own (the context's
graphs off): after every replay, with eager generations and reads between them,
the best-ever record and the populations equal the oracle's."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interval,gens", [(0, 2), (4, 4)])
def test_reads_between_replays(interval, gens):
    import torch
    ensure_built()
    m, p = inputs.make_instance(80, 10, 3, 4, seed=5)
    isl = [inputs.cellular(6, 6, 0.9, 0.4), inputs.pseudo(36, 0.8, 0.3)]
    w = dict(m=m, p=p, islands=isl, interval=interval, theta=1.0, topology=0)
    ctx, ga = make_ctx([w]), oracle_ga(w)
    ctx.set_graphs(False)
    found = []

    def check(what):
        b1, b2 = ctx.best(0), ga.best()
        assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"]), what
        assert b1["perm"].tolist() == b2["perm"].tolist(), what
        assert_same_state(ctx, ga, 0, 2, what)
        found.append(b2["generation"])

    ctx.evolve(gens)
    ga.evolve(gens)
    check("eager")
    say(f"[capture] interval={interval} generations={gens}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=ctx.stream):
        ctx.evolve(gens)
    for rep in range(8):
        with torch.cuda.stream(ctx.stream):
            graph.replay()
        ga.evolve(gens)
        check(f"replay {rep}")
        if rep % 3 == 2:
            ctx.evolve(gens)
            ga.evolve(gens)
            check(f"eager after replay {rep}")
    torch.cuda.synchronize()
    del graph
    ctx.close()
    # records were found in replays that follow a read
    assert len(set(found)) > 4, found


def test_screened_epochs_one_after_another():
    """Pre-screened epochs with the context's launches one after another: the
    whole state equals that of launches side by side."""
    from test_gpu_surrogate import _ctx, _small
    ensure_built()
    say("[capture] pre-screened epochs, launches side by side and one after another")
    a, b = (_ctx(_small(seed=8), warmup=3, seed=5) for _ in range(2))
    b.set_concurrent(False)
    for g in (10, 10, 7, 3, 20):
        a.evolve(g)
        b.evolve(g)
        assert a.checkpoint() == b.checkpoint(), a.generation
    a.close()
    b.close()
