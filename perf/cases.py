"""The work that users of the framework have it do, as cases that can be timed.

Each case is one pass through public entry points (`Context`, `TtContext`): decodes of caller-supplied
permutations, runs of the island GA (one instance, many seeds of one instance, an uneven batch, with and
without the learned pre-screen), runs of the paper-faithful variant, and the pre-screen network's backward
pass.  Sizes are those of the repository's workloads, experiments and tests; `draw` spreads over the ranges
between and around them.

Every case is a dict of plain values.  `inst` seeds what defines the shape of the work (machine counts and,
in an uneven batch, sizes); the seed given to `prepare` draws everything else.
"""
from __future__ import annotations

import math

import numpy as np
import torch

DEVICE = "cuda"


def listed() -> list[dict]:
    return [
        # decode of caller-supplied permutations (Context.evaluate, device rows)
        # a handful of schedules checked at once inside a host-side search: launch and wait, nothing else
        dict(name="decode_few", kind="decode", n=20, S=3, m_lo=2, m_hi=2, p_hi=99, rows=64, inst=1),
        # the decode experiment's million rows at the medium shape
        dict(name="decode_medium_1m", kind="decode", n=100, S=5, m_lo=1, m_hi=5, p_hi=99, rows=1_000_000, inst=1),
        # a quarter million rows at the large shape (about one generation of the large workload)
        dict(name="decode_large_250k", kind="decode", n=500, S=10, m_lo=3, m_hi=5, p_hi=99, rows=250_007, inst=1),
        # an ordinary ragged batch of long rows (the surrogate workload's shape)
        dict(name="decode_long_4099", kind="decode", n=1000, S=20, m_lo=2, m_hi=6, p_hi=99, rows=4099, inst=1),
        # runs of the island GA (Context.evolve, then the best record, counters and the populations' makespans)
        # the tiny workload's whole run: launch-bound
        dict(name="ga_tiny", kind="ga", n=20, S=3, m_lo=2, m_hi=2, p_hi=99, islands="dual", side=8, seeds=1,
             gens=100, interval=10, genes=True, inst=1),
        # the medium workload's whole run, populations read back
        dict(name="ga_medium", kind="ga", n=100, S=5, m_lo=1, m_hi=5, p_hi=99, islands="dual", side=64, seeds=1,
             gens=500, interval=20, genes=True, inst=1),
        # two epochs of the large workload (sixteen islands, ring then pairs)
        dict(name="ga_large", kind="ga", n=500, S=10, m_lo=3, m_hi=5, p_hi=99, islands="ring16", side=128, seeds=1,
             gens=40, interval=20, genes=False, inst=1),
        # the island experiment: Section 5's sizes, fifty seeds side by side in one context
        dict(name="ga_seeds", kind="ga", n=300, S=4, m_lo=2, m_hi=2, p_hi=5, islands="dual", side=16, seeds=50,
             gens=1000, interval=500, genes=False, inst=1),
        # the uneven batch of 256 instances
        dict(name="ga_batch", kind="ga_batch", batch=256, side_lo=32, side_hi=128, gens=20, interval=10, inst=7),
        # the surrogate workload with the learned pre-screen (eight candidates per cell)
        dict(name="ga_prescreen", kind="prescreen", n=1000, S=20, m_lo=2, m_hi=6, p_hi=99, side=64, k=8, gens=20,
             interval=20, inst=1),
        # the paper-faithful variant: fifty runs of Section 5's setting (TtContext.evolve)
        dict(name="tardiness_runs", kind="tardiness", n=300, S=4, m=2, side=16, runs=50, gens=100, interval=500),
        # backward pass of the pre-screen's network on a training batch (Context.mlp_gradients)
        dict(name="mlp_gradients", kind="mlp", rows=4096),
    ]


def _log(rng, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    """One more case between the listed ones' sizes, odd sizes among them."""
    kind = rng.choice(["decode", "decode", "decode", "ga", "ga", "ga", "ga_batch", "prescreen", "tardiness", "mlp"])
    inst = rng.randrange(1, 1 << 20)
    if kind == "decode":
        n, S = _log(rng, 8, 1000), _log(rng, 1, 20)
        m_lo = rng.randint(1, 4)
        cap = 500_000_000 // (n * S)
        return dict(kind=kind, n=n, S=S, m_lo=m_lo, m_hi=rng.randint(m_lo, 6), p_hi=rng.choice([5, 99, 99, 999]),
                    rows=_log(rng, 16, min(1_000_000, cap)), inst=inst)
    if kind == "ga":
        n, S = _log(rng, 16, 600), _log(rng, 2, 16)
        m_lo = rng.randint(1, 3)
        islands = rng.choice(["dual", "dual", "dual", "cellular", "pseudo", "ring16"])
        side = _log(rng, 4, 64)
        seeds = rng.choice([1, 1, 1, _log(rng, 2, 50)])
        size = {"dual": 2, "cellular": 2, "pseudo": 2, "ring16": 16}[islands] * side * side * seeds
        gens = max(4, min(200, 4_000_000_000 // (size * n * S)))
        return dict(kind=kind, n=n, S=S, m_lo=m_lo, m_hi=rng.randint(m_lo, 6), p_hi=rng.choice([5, 99, 99, 999]),
                    islands=islands, side=side, seeds=seeds, gens=gens,
                    interval=rng.choice([0, 5, 10, 20]) if islands != "cellular" and islands != "pseudo" else 0,
                    genes=size * n <= 1_000_000, inst=inst)
    if kind == "ga_batch":
        return dict(kind=kind, batch=_log(rng, 4, 96), side_lo=rng.randint(8, 24), side_hi=rng.randint(32, 96),
                    gens=rng.choice([10, 20]), interval=rng.choice([5, 10]), inst=inst)
    if kind == "prescreen":
        return dict(kind=kind, n=_log(rng, 60, 1000), S=rng.randint(3, 20), m_lo=2, m_hi=rng.randint(2, 6), p_hi=99,
                    side=rng.randint(12, 64), k=rng.choice([2, 4, 8]), gens=rng.choice([10, 20]), interval=10,
                    inst=inst)
    if kind == "tardiness":
        return dict(kind=kind, n=_log(rng, 30, 500), S=rng.randint(2, 6), m=rng.choice([1, 2, 2, 3, 4]),
                    side=rng.randint(4, 16), runs=_log(rng, 1, 50), gens=rng.choice([20, 50]),
                    interval=rng.choice([10, 500]))
    return dict(kind="mlp", rows=128 * rng.randint(1, 32))


# ---- inputs -----------------------------------------------------------------
def _rng(*key: int) -> np.random.Generator:
    return np.random.default_rng([int(k) & 0xFFFFFFFF for k in key])


def _machines(case: dict) -> np.ndarray:
    return _rng(case["inst"], 1).integers(case["m_lo"], case["m_hi"] + 1, size=case["S"]).astype(np.int32)


def _times(n: int, S: int, p_hi: int, *key: int) -> np.ndarray:
    return _rng(*key, 2).integers(1, p_hi + 1, size=(n, S)).astype(np.int32)


def _perms(rows: int, n: int, seed: int) -> torch.Tensor:
    """rows x n int32 on the device, each row a uniformly random permutation."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    out = torch.empty((rows, n), dtype=torch.int32, device=DEVICE)
    step = max(1, 50_000_000 // n)
    for r in range(0, rows, step):
        k = min(step, rows - r)
        out[r:r + k] = torch.rand((k, n), generator=g, device=DEVICE).argsort(dim=1).to(torch.int32)
    return out


def _cellular(rows: int, cols: int, pc: float, pm: float) -> dict:
    return dict(kind=0, rows=rows, cols=cols, size=rows * cols, pc=pc, pm=pm)


def _pseudo(size: int, pc: float, pm: float) -> dict:
    return dict(kind=1, rows=0, cols=0, size=size, pc=pc, pm=pm)


def _islands(layout: str, side: int) -> list:
    cell, half = (0.9, 0.1), side * side - (side * side) % 2
    if layout == "cellular":
        return [_cellular(side, 2 * side, *cell)]
    if layout == "pseudo":
        return [_pseudo(2 * half, 0.75, 0.0)]
    pairs = 8 if layout == "ring16" else 1
    return [_cellular(side, side, *cell)] * pairs + [_pseudo(half, 0.75, 0.0)] * pairs


def _batch(case: dict) -> list:
    """(n, S, machines, side) of the uneven batch's instances."""
    g = _rng(case["inst"], 3)
    out = []
    for _ in range(case["batch"]):
        n, S = int(g.choice([20, 50, 100, 200, 500])), int(g.choice([5, 10, 20]))
        side = int(g.integers(case["side_lo"], case["side_hi"] + 1))
        out.append((n, S, g.integers(1, 6, size=S).astype(np.int32), side))
    return out


def _features(rows: int, seed: int):
    """Feature rows (BF16 bits: bucket loads around 1, scalars in [0, 1.2]) and targets (relative gaps)."""
    g = _rng(seed, 4)
    x = np.concatenate([g.normal(1.0, 0.25, size=(rows, 240)).clip(0.0), g.uniform(0.0, 1.2, size=(rows, 16))], axis=1)
    X = torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16)
    t = torch.from_numpy(g.uniform(0.0, 0.15, size=rows).astype(np.float32))
    return X, t


def _params(seed: int) -> np.ndarray:
    """Network parameters as they are initialised: weights uniform in +-sqrt(6 / fan in), small biases."""
    g = _rng(seed, 5)

    def uni(fan, *shape):
        return (g.uniform(-1.0, 1.0, size=shape) * math.sqrt(6.0 / fan)).ravel()

    parts = [uni(256, 512, 256), g.normal(0, 0.01, 512), uni(512, 512, 512), g.normal(0, 0.01, 512), uni(512, 512),
             g.normal(0, 0.01, 1)]
    return np.concatenate(parts).astype(np.float32)


def prepare(case: dict, seed: int) -> dict:
    from paper_1903_10722_amd import Context, inputs
    from paper_1903_10722_amd.tardiness import TtContext
    kind = case["kind"]
    if kind == "tardiness":
        inst = inputs.tardiness_instance(case["n"], case["S"], [case["m"]] * case["S"], seed=seed)
        isl = [_cellular(case["side"], case["side"], 1.0, 0.05),
               _pseudo(case["side"] ** 2 - case["side"] ** 2 % 2, 0.75, 0.0)]
        ctx = TtContext(inst, isl, interval=case["interval"], seed=seed, runs=case["runs"])
        return dict(case=case, ctx=ctx)
    ctx = Context(device=0)
    state = dict(case=case, ctx=ctx)
    if kind == "ga_batch":
        for i, (n, S, m, side) in enumerate(_batch(case)):
            ctx.add_instance(m, _times(n, S, 99, seed, i), _islands("dual", side), interval=case["interval"],
                             seed=seed)
    elif kind == "mlp":
        m = np.array([2, 2, 2], dtype=np.int32)
        ctx.add_instance(m, _times(20, 3, 99, seed), _islands("dual", 4), interval=0, seed=seed, surrogate_k=2)
    elif kind == "decode":
        # decoding needs no population: the smallest islands
        ctx.add_instance(_machines(case), _times(case["n"], case["S"], case["p_hi"], seed), _islands("dual", 3),
                         interval=0, seed=seed)
        state["perms"] = _perms(case["rows"], case["n"], seed)
    elif kind == "prescreen":
        ctx.add_instance(_machines(case), _times(case["n"], case["S"], case["p_hi"], seed),
                         _islands("dual", case["side"]), interval=case["interval"], seed=seed, surrogate_k=case["k"])
    else:
        p = _times(case["n"], case["S"], case["p_hi"], seed)
        for r in range(case["seeds"]):
            ctx.add_instance(_machines(case), p, _islands(case["islands"], case["side"]), interval=case["interval"],
                             topology=1 if case["islands"] == "ring16" else 0, seed=seed + r)
    ctx.bind()
    if kind == "mlp":
        ctx.set_surrogate_params(_params(seed))
        X, t = _features(case["rows"], seed)
        state["X"], state["t"] = X.view(torch.int16).to(DEVICE), t.to(DEVICE)
    return state


# ---- one pass -----------------------------------------------------------------
def _makespans(ctx, inst: int, island: int) -> np.ndarray:
    """Every individual's makespan of one island (ffs_get_population without the genes)."""
    import ctypes
    mk = np.zeros(ctx.instances[inst]["sizes"][island], dtype=np.int32)
    ctx._check(ctx.lib.ffs_get_population(ctx._h, inst, island, None, mk.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))))
    return mk


def run(state: dict):
    case, ctx, kind = state["case"], state["ctx"], state["case"]["kind"]
    if kind == "decode":
        return ctx.evaluate(0, state["perms"])
    if kind == "mlp":
        g, dZ2, dZ1 = ctx.mlp_gradients(state["X"], state["t"])
        return dict(grad=g, dZ2=dZ2.view(torch.bfloat16), dZ1=dZ1.view(torch.bfloat16))
    ctx.evolve(case["gens"])
    if kind == "tardiness":
        best = [ctx.best(r) for r in range(case["runs"])]
        genes, objs = zip(*[ctx.population(0, i) for i in range(2)])
        return dict(best=np.array([[b["objective"], b["generation"], b["island"], b["slot"]] for b in best]),
                    best_genes=np.stack([b["genes"] for b in best]), genes=np.concatenate(genes),
                    objectives=np.concatenate(objs))
    # what the end of a run reads: the best records, the migration counters and the final populations (genes too
    # where the case asks for them: at the large sizes their download would hide the run)
    insts = range(len(ctx.instances))
    best = [ctx.best(i) for i in insts]
    out = dict(best=np.array([[b["makespan"], b["generation"]] for b in best]),
               perms=np.concatenate([b["perm"] for b in best]),
               counters=np.array([ctx.migration_counters(i) for i in insts]))
    where = [(i, x) for i in insts for x in range(len(ctx.instances[i]["sizes"]))]
    if case.get("genes"):
        pops = [ctx.population(i, x) for i, x in where]
        out["genes"] = np.concatenate([g for g, _ in pops])
        out["makespans"] = np.concatenate([m for _, m in pops])
    else:
        out["makespans"] = np.concatenate([_makespans(ctx, i, x) for i, x in where])
    if kind == "prescreen":
        out["params"] = ctx.surrogate_params()
        out["choices"] = ctx.surrogate_choices()
    return out


# ---- what a pass cannot do without -----------------------------------------------
def _ga_work(n: int, m: np.ndarray, individuals: int, gens: int):
    """Two parent rows in and one child row out (16-bit genes) and a makespan each way; n (m_k + 6) integer
    operations per stage of a decode (an m_k-way minimum and about six more per job and stage)."""
    return individuals * gens * (6.0 * n + 8), individuals * gens * n * float((np.asarray(m) + 6).sum())


def work(case: dict) -> dict:
    kind = case["kind"]
    if kind == "decode":
        m = _machines(case)
        return dict(bytes=case["rows"] * (4.0 * case["n"] + 4) + 4.0 * case["n"] * case["S"],
                    flops=case["rows"] * case["n"] * float((m + 6).sum()))
    if kind == "mlp":
        r = case["rows"]
        fwd = 2.0 * r * (256 * 512 + 512 * 512 + 512)
        # features and targets in, gradients and both back-propagated activations out, weights in
        return dict(bytes=r * (2.0 * 256 + 4 + 2 * 2 * 512) + 394753 * 8.0, flops=3 * fwd - 2.0 * r * 256 * 512)
    if kind == "tardiness":
        J, N = case["n"], 2 * case["side"] ** 2 * case["runs"]
        per = case["S"] * J * (6.0 + (case["m"] - 1) * math.ceil(math.log2(max(2, J))))
        return dict(bytes=N * case["gens"] * (3.0 * J * case["S"] + 24), flops=N * case["gens"] * per)
    if kind == "ga_batch":
        parts = [_ga_work(n, m, 2 * side * side, case["gens"]) for n, S, m, side in _batch(case)]
        return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))
    m = _machines(case)
    if kind == "prescreen":
        b, f = _ga_work(case["n"], m, 2 * case["side"] ** 2, case["gens"])
        cells, n, S = case["side"] ** 2, case["n"], case["S"]
        mlp = 2.0 * (256 * 512 + 512 * 512 + 512)
        # per generation: k candidates per cell built, summed over stages and scored, and a training step
        b += case["gens"] * (cells * case["k"] * 4.0 * n + 4096 * 2.0 * 256 + 394753 * 26.0)
        f += case["gens"] * (cells * case["k"] * (float(n) * S + mlp) + 3.0 * 4096 * mlp)
        return dict(bytes=b, flops=f)
    per = {"dual": 2, "cellular": 2, "pseudo": 2, "ring16": 16}[case["islands"]] * case["side"] ** 2
    b, f = _ga_work(case["n"], m, per * case["seeds"], case["gens"])
    return dict(bytes=b, flops=f)


# ---- exact values -----------------------------------------------------------------
def _exact_decode(case: dict, seed: int) -> torch.Tensor:
    """Makespans by list scheduling in 64-bit integers, all rows at a time: stage 1 in permutation order, later
    stages in the order of the previous completions (ties: earlier dispatch), earliest free machine first."""
    m, n, S = _machines(case), case["n"], case["S"]
    p = torch.from_numpy(_times(n, S, case["p_hi"], seed).astype(np.int64)).to(DEVICE)
    perms = _perms(case["rows"], n, seed)
    outs = []
    step = max(1, 60_000_000 // n)
    for r0 in range(0, case["rows"], step):
        jobs = perms[r0:r0 + step].to(torch.int64)
        rows = jobs.shape[0]
        ready = torch.zeros((n, rows), dtype=torch.int64, device=DEVICE)
        for s in range(S):
            pt = p[:, s][jobs].t().contiguous()
            free = [torch.zeros(rows, dtype=torch.int64, device=DEVICE) for _ in range(int(m[s]))]   # ascending
            done = torch.empty_like(ready)
            for t in range(n):
                c = torch.maximum(free[0], ready[t]) + pt[t]
                done[t] = c
                for q in range(1, len(free)):
                    free[q - 1], c = torch.minimum(free[q], c), torch.maximum(free[q], c)
                free[-1] = c
            ready, order = torch.sort(done, dim=0, stable=True)
            jobs = torch.gather(jobs, 1, order.t())
        outs.append(ready[-1].to(torch.int32))
    return torch.cat(outs)


def _exact_mlp(case: dict, seed: int) -> dict:
    w = torch.from_numpy(_params(seed)).double().to(DEVICE)
    X, t = _features(case["rows"], seed)
    X, t, rows = X.double().to(DEVICE), t.double().to(DEVICE), case["rows"]
    cuts = torch.split(w, [512 * 256, 512, 512 * 512, 512, 512, 1])
    W1, W2 = cuts[0].view(512, 256), cuts[2].view(512, 512)
    H1 = (X @ W1.T + cuts[1]).clamp(min=0)
    H2 = (H1 @ W2.T + cuts[3]).clamp(min=0)
    d = 2.0 * (H2 @ cuts[4] + cuts[5] - t) / rows
    dZ2 = torch.outer(d, cuts[4]) * (H2 > 0)
    dZ1 = (dZ2 @ W2) * (H1 > 0)
    grad = torch.cat([(dZ1.T @ X).ravel(), dZ1.sum(0), (dZ2.T @ H1).ravel(), dZ2.sum(0), d @ H2, d.sum().view(1)])
    return dict(grad=grad, dZ2=dZ2, dZ1=dZ1)


def exact(case: dict, seed: int):
    if case["kind"] == "decode":
        return _exact_decode(case, seed) if case["n"] * case["S"] <= 6000 else None
    return _exact_mlp(case, seed) if case["kind"] == "mlp" else None
