"""Instances at the LDS limit of the per-stage mapping, against the oracle
(integers: equal): long rows of many stages with two-byte processing times,
where the times leave room for one chromosome's row but not for two, also when
the two bytes come from another instance of the context."""
import pytest

from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs

pytestmark = pytest.mark.gpu

ISLANDS = [inputs.cellular(3, 3, 0.9, 0.5), inputs.pseudo(4, 0.8, 0.4)]


@pytest.mark.parametrize("n,S", [(2721, 26), (4000, 17), (4064, 17)])
def test_one_row_beside_the_times(n, S):
    ensure_built()
    m, p = inputs.make_instance(n, S, 1, 2, p_hi=9, seed=n)
    p[7, 3] = 300
    w = dict(m=m, p=p, islands=ISLANDS, interval=2, theta=1.0, topology=0)
    say(f"[limits] n={n} S={S}")
    ctx, ga = make_ctx([w], mapping=0), oracle_ga(w)
    assert_same_state(ctx, ga, 0, 2, "generation 0")
    ctx.evolve(3)
    ga.evolve(3)
    assert_same_state(ctx, ga, 0, 2, "generation 3")
    ctx.close()


def test_two_byte_times_of_another_instance():
    ensure_built()
    n, S = 4000, 17
    m, p = inputs.make_instance(n, S, 1, 2, p_hi=9, seed=3)
    m2, p2 = inputs.make_instance(20, 3, 1, 2, p_hi=400, seed=4)
    ws = [dict(m=a, p=b, islands=ISLANDS, interval=2, theta=1.0, topology=0) for a, b in ((m, p), (m2, p2))]
    say("[limits] two-byte times of another instance")
    ctx = make_ctx(ws, mapping=0)
    gas = [oracle_ga(w, inst=i) for i, w in enumerate(ws)]
    ctx.evolve(2)
    for i, ga in enumerate(gas):
        ga.evolve(2)
        assert_same_state(ctx, ga, i, 2, f"instance {i}")
    ctx.close()
