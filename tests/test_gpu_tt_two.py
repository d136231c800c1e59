"""GPU parity of the tardiness decode for stages of at most two machines,
against its oracle (int64 objectives: equal): every count of positions per lane
and its ends, stages of one machine, all jobs on one machine, ties of
completions, genes out of range; and trajectories whose gene strings take one
and several passes of a wave."""
import numpy as np
import pytest

from gpu_util import ensure_built, say
from oracle import tardiness as ot
from paper_1903_10722_amd import inputs
from test_gpu_tardiness import _ctx, _random_genes, _same

pytestmark = pytest.mark.gpu

JOBS = [1, 2, 63, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 384, 385, 449, 512, 513, 768, 769, 1023, 1024]


@pytest.mark.parametrize("J", JOBS)
def test_decode_two(J):
    ensure_built()
    for M, hi, scale in (([2, 2, 2], 5, 1.0), ([1, 2, 1], 5, 0.1), ([1, 1], 3, 1.0), ([2, 2, 1], 1, 0.0)):
        inst = inputs.tardiness_instance(J, len(M), M, seed=J, p_hi=hi, release_scale=scale)
        say(f"[tt] J={J} M={M}")
        ctx = _ctx(inst, [inputs.pseudo(2, 0.75, 0.0)], interval=0)
        genes = _random_genes(inst, 7, seed=J)
        genes[0] = 0
        genes[1] = np.tile(np.asarray(M) - 1, J)
        got = ctx.evaluate(genes).cpu().numpy()
        want = np.array([ot.decode(inst, g)[0] for g in genes], dtype=np.int64)
        assert np.array_equal(got, want), (M, got, want)
        genes[2, -1] = M[-1]                # the last job's last stage
        genes[3, 0] = 255                   # the first job's first
        got = ctx.evaluate(genes).cpu().numpy()
        want[2] = want[3] = -1
        assert np.array_equal(got, want), (M, got, want)
        ctx.close()


@pytest.mark.parametrize("J,M", [(5, [2, 1]), (65, [2, 2, 2]), (300, [2, 2, 2, 2]), (1000, [2, 1, 2, 2, 2])])
def test_trajectory_two(J, M):
    ensure_built()
    inst = inputs.tardiness_instance(J, len(M), M, seed=J)
    isl = [inputs.cellular(3, 4, 0.8, 0.5), inputs.pseudo(12, 0.75, 0.5)]
    say(f"[tt] trajectory J={J} M={M}")
    ctx = _ctx(inst, isl, interval=3, runs=2, seed=7)
    gas = [ot.GA(inst, isl, interval=3, seed=7, inst_id=r) for r in range(2)]
    for g in (0, 1, 4):
        ctx.evolve(g)
        for r, ga in enumerate(gas):
            ga.evolve(g)
            _same(ctx, ga, r, 2, f"J={J} run {r} after {g} more generations")
    ctx.close()
