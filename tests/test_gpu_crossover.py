"""GPU parity of the order crossover on rows read as vectors, against the
oracle's trajectories (integers: equal): rows around the eight-gene vectors and
the register path's tiers (at most 3, 7 and 13 vectors per lane, longer rows in
passes), reversed parents (pseudo pairs, even and odd), children with and
without crossover and mutation, one lane per stage and one per chromosome."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2), (7, 3), (8, 1), (9, 3), (20, 3), (33, 1), (56, 1), (57, 1), (100, 5), (104, 1), (105, 1), (64, 64),
          (300, 4), (500, 5), (513, 2), (1000, 20), (1025, 3)]


@pytest.mark.parametrize("n,S", SHAPES)
@pytest.mark.parametrize("mapping", [0, 1])
def test_crossover_rows(n, S, mapping):
    ensure_built()
    m, p = inputs.make_instance(n, S, 1, 2, p_hi=20, seed=n + S)
    isl = [inputs.cellular(5, 4, 0.9, 0.5), inputs.pseudo(22, 0.8, 0.4)]
    w = dict(m=m, p=p, islands=isl, interval=3, theta=1.0, topology=0)
    say(f"[ox] n={n} S={S} mapping={mapping}")
    ctx = make_ctx([w], mapping=mapping)
    ga = oracle_ga(w)
    assert_same_state(ctx, ga, 0, 2, f"n={n} S={S} generation 0")
    for g in (1, 3, 4):
        ctx.evolve(g)
        ga.evolve(g)
        assert_same_state(ctx, ga, 0, 2, f"n={n} S={S} generation {ctx.generation}")
    ctx.close()
