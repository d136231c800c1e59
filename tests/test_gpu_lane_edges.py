"""GPU parity of the lane decode where its windows of sixteen slots have edges,
against the oracle (integers: equal): rows around one, two and more windows
with one, two and three stages, so that a stage's first, full, flush and last
windows coincide in each combination; runs and line sweeps of one stage whose
rows end on a window; and the automatic choice of ffs_evaluate and
ffs_evaluate_noalloc at row counts that take the lane kernel."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same_state, ensure_built, make_ctx, oracle_ga, say
from paper_1903_10722_amd import inputs
from paper_1903_10722_amd.binding import FFS_OK, evaluate_noalloc

pytestmark = pytest.mark.gpu

ISLANDS = [inputs.cellular(3, 3, 0.9, 0.1), inputs.pseudo(2, 0.75, 0.0)]
MACHINES = {1: [[1], [3], [8]], 2: [[1, 1], [2, 5], [8, 8]], 3: [[1, 1, 1], [3, 1, 4]]}


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("n", [15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 512, 528])
def test_lane_decode_windows(n, S):
    ensure_built()
    for machines in MACHINES[S]:
        for p_hi in (99, 999):       # one- and two-byte processing times
            m, p = inputs.make_instance(n, S, 1, 1, p_hi=p_hi, seed=n + S, machines=machines)
            say(f"[lane windows] n={n} S={S} m={machines} p<={p_hi}")
            ctx = make_ctx([dict(m=m, p=p, islands=ISLANDS, interval=0)], mapping=1)
            perms = inputs.random_perms(70, n, seed=n)
            got = ctx.evaluate(0, perms).cpu().numpy()
            ctx.close()
            want = oracle.decode_many(m, p, perms)
            assert np.array_equal(got, want), (machines, p_hi, got[:5], want[:5])


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("sweep", [0, 1])
def test_lane_trajectory_one_stage(n, sweep):
    ensure_built()
    m, p = inputs.make_instance(n, 1, 3, 3, p_hi=50, seed=n, machines=[3])
    isl = [dict(inputs.cellular(9, 8, 0.9, 0.5), sweep=sweep), inputs.pseudo(130, 0.8, 0.4)]
    w = dict(m=m, p=p, islands=isl, interval=4, theta=1.0, topology=0)
    say(f"[lane windows] trajectory n={n} sweep={sweep}")
    ctx, ga = make_ctx([w], mapping=1), oracle_ga(w)
    for g in (0, 3, 5):
        ctx.evolve(g)
        ga.evolve(g)
        assert_same_state(ctx, ga, 0, 2, f"n={n} generation {ctx.generation}")
        b1, b2 = ctx.best(0), ga.best()
        assert (b1["makespan"], b1["generation"]) == (b2["makespan"], b2["generation"])
        assert b1["perm"].tolist() == b2["perm"].tolist()
    ctx.close()


@pytest.mark.parametrize("n,machines,rows", [(256, [2], 98304), (48, [4], 524289), (100, [2, 5, 1, 4, 3], 100003),
                                             (100, [2, 5, 1, 4, 3] * 4, 100003),
                                             (20, [2, 3, 4, 5, 6] * 4, 65537), (500, [3, 3, 3, 5, 3, 5, 4, 5, 4, 5], 196609)])
def test_automatic_choice_of_many_rows(n, machines, rows):
    """Row counts from which the lane kernel is the automatic choice."""
    import torch
    ensure_built()
    S = len(machines)
    m, p = inputs.make_instance(n, S, 1, 1, p_hi=99, seed=n, machines=machines)
    perms = inputs.random_perms(rows, n, seed=n)
    at = np.union1d(np.random.default_rng(1).choice(rows, 500, replace=False), [0, rows - 1])
    want = oracle.decode_many(m, p, perms[at])
    say(f"[lane windows] automatic choice n={n} S={S} rows={rows}")
    ctx = make_ctx([dict(m=m, p=p, islands=ISLANDS, interval=0)])
    got = ctx.evaluate(0, perms).cpu().numpy()
    ctx.close()
    assert np.array_equal(got[at], want), (got[at][:5], want[:5])
    t = torch.from_numpy(perms).cuda()
    out = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    assert evaluate_noalloc(m, p, t, out) == FFS_OK
    assert np.array_equal(out.cpu().numpy(), got)
