"""Timed cases of the annealer: whole anneals of one graph, batched runs of many
graphs, and read-outs, each through the package's public calls.

A case is a dict of plain values.  Its inputs (graph and annealing seed) come
from the case and a seed alone.  Kinds:

    single    one graph, T trials, all steps of the schedule, then energy, cut
              and spins.  `entry` says how a program calls it: "job" keeps a
              psa.Job and steps it (outputs on the device), "call" is the one
              call psa.anneal (outputs on the host), "noalloc" is
              psa.anneal_noalloc (outputs on the device).
    batch     many graphs of uneven size advanced together by
              psa.jobs_step_batch and read out by psa.jobs_energy_cut.
    readout   energy, cut, local fields and spins of given spins.
"""
import math
import random

import numpy as np
import torch

from paper_2601_14476_amd import psa

_context = []


def _ctx():
    if not _context:
        _context.append(psa.Context(0))
    return _context[0]


# ---------------------------------------------------------------------------
# Graphs
# ---------------------------------------------------------------------------
def _gnm(rng, n, m):
    """m distinct pairs u < v, drawn uniformly."""
    m = min(m, n * (n - 1) // 2)
    keys = np.zeros(0, np.int64)
    while keys.size < m:
        k = int(1.2 * (m - keys.size)) + 32
        a, b = rng.integers(0, n, size=(2, k))
        new = (np.minimum(a, b) * n + np.maximum(a, b))[a != b]
        keys = np.unique(np.concatenate([keys, new]))
    keys = np.sort(rng.permutation(keys)[:m])
    return (keys // n).astype(np.int32), (keys % n).astype(np.int32)


def _torus(rows, cols):
    r, c = np.meshgrid(np.arange(rows), np.arange(cols), indexing="ij")
    node = (r * cols + c).ravel()
    right = (r * cols + (c + 1) % cols).ravel()
    down = (((r + 1) % rows) * cols + c).ravel()
    return np.concatenate([node, node]).astype(np.int32), np.concatenate([right, down]).astype(np.int32)


def _graph(case, seed):
    """(n, u, v, w) of a case's graph; MAX-CUT weights +1, +-1, or +-1..+-7."""
    rng = np.random.Generator(np.random.PCG64([seed, case["n"]]))
    n = case["n"]
    if case["graph"] == "torus":
        u, v = _torus(case["rows"], n // case["rows"])
    else:
        u, v = _gnm(rng, n, case["edges"])
    if case["weights"] == "one":
        w = np.ones(u.size, np.int32)
    elif case["weights"] == "pm1":
        w = rng.choice(np.array([-1, 1], np.int32), size=u.size)
    else:
        w = (rng.integers(1, 8, size=u.size) * rng.choice([-1, 1], size=u.size)).astype(np.int32)
    return n, u, v, w


def _mix(case):
    """The runs of a batch: the same sizes for every seed.

    "er_and_sparse": graphs of 800 to 5,000 p-bits, in turn with mean degree
    2 to 10 % of n and +1 weights, and with degree 4 to 8 and +-1 weights, one
    trial count, no variability.  "requests": 800 to 20,000 p-bits of degree
    4 to 50, +-1 weights, 32 to 256 trials, some with device variability."""
    rng = random.Random(case["mix_seed"])
    runs = []
    for j in range(case["count"]):
        if case["mix"] == "er_and_sparse":
            n = rng.randint(800, 5000)
            if j % 2 == 0:
                edges, weights = int(rng.uniform(0.02, 0.1) * n * (n - 1) / 2), "one"
            else:
                edges, weights = n * rng.randint(4, 8) // 2, "pm1"
            trials, sigma = case["trials"], 0.0
        else:
            n = rng.randint(800, 20000)
            edges, weights = n * rng.randint(4, 50) // 2, "pm1"
            trials, sigma = rng.randint(32, 256), rng.choice([0.0, 0.05, 0.1, 0.2])
        runs.append(dict(graph="gnm", n=n, edges=edges, weights=weights, trials=trials, sigma=sigma))
    return runs


def _options(case):
    """Keyword arguments of the run: variability and update rule."""
    s = case.get("sigma", 0.0)
    kw = dict(sigma_lambda=s, sigma_delta=s, sigma_nu=s, p_mean=0.8 if s > 0 else 1.0)
    rule = case.get("rule", "psa")
    if rule == "spsa":
        kw.update(algorithm=psa.PSA_ALG_SPSA, p_stall=0.5)
    elif rule == "tapsa":
        kw.update(algorithm=psa.PSA_ALG_TAPSA, window=4)
    elif rule == "period":
        kw.update(t_res=10)
    return kw


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    sparse = dict(kind="single", entry="job", graph="gnm", n=2000, edges=6000, weights="pm1", trials=100, sigma=0.1)
    torus = dict(kind="single", entry="job", graph="torus", n=20000, rows=100, weights="pm1", sigma=0.1)
    return [
        # the smallest use: one call on a little problem, results on the host
        dict(name="small_call", kind="single", entry="call", graph="gnm", n=250, edges=750, weights="pm1",
             trials=16, steps=200, sigma=0.1, rule="psa"),
        # the paper's random graph of 800 p-bits and +1 weights, 10 trials
        dict(name="er800_t10", kind="single", entry="job", graph="gnm", n=800, edges=19176, weights="one",
             trials=10, steps=1000, sigma=0.0, rule="psa"),
        # a sparse graph with device variability, 100 trials: the ordinary run,
        # with each input stage and with timing as periods
        dict(sparse, name="gnm2000_t100", steps=2000, rule="psa"),
        dict(sparse, name="gnm2000_tapsa", steps=1000, rule="tapsa"),
        dict(sparse, name="gnm2000_period", steps=500, rule="period"),
        # the paper's 100 x 200 torus: the largest run of the benchmark, and the
        # paper's 100 trials
        dict(torus, name="torus20000_t1024", trials=1024, steps=5000, rule="psa"),
        dict(torus, name="torus20000_t100", trials=100, steps=1000, rule="psa"),
        # one graph of long rows (matrix path)
        dict(name="er3000_t64", kind="single", entry="job", graph="gnm", n=3000, edges=269910, weights="one",
             trials=64, steps=500, sigma=0.0, rule="psa"),
        # integer weights, an odd size and trial count
        dict(name="weights4001_t37", kind="single", entry="job", graph="gnm", n=4001, edges=24006, weights="int",
             trials=37, steps=500, sigma=0.05, rule="psa"),
        # many graphs of uneven size run together
        dict(name="batch24", kind="batch", mix="er_and_sparse", count=24, mix_seed=4, trials=64, steps=500),
        # one serving quantum over the resident requests
        dict(name="requests16", kind="batch", mix="requests", count=16, mix_seed=5, trials=0, steps=250),
        # results of a finished run on a sparse graph
        dict(name="readout20000_t256", kind="readout", graph="gnm", n=20000, edges=200000, weights="pm1",
             trials=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST = 1.5e9  # p-bit updates of a drawn case, longer rows counting for more


def draw(rng):
    kind = rng.choice(["single"] * 7 + ["batch", "readout"])
    if kind == "batch":
        mix = rng.choice(["er_and_sparse", "requests"])
        return dict(kind=kind, mix=mix, count=rng.randint(3, 16), mix_seed=rng.randint(100, 10**6),
                    trials=_log(rng, 8, 100) if mix == "er_and_sparse" else 0, steps=_log(rng, 50, 250))
    shape = rng.choice(["gnm", "gnm", "torus", "er"])
    if shape == "torus":
        rows = _log(rng, 5, 140)
        n = rows * _log(rng, 5, 140)
        graph = dict(graph="torus", n=n, rows=rows)
        degree = 4.0
    elif shape == "gnm":
        n = _log(rng, 60, 20000)
        edges = n * rng.randint(4, 50) // 2
        degree = 2.0 * edges / n
        graph = dict(graph="gnm", n=n, edges=edges)
    else:
        n = _log(rng, 100, 5000)
        edges = max(n, int(rng.uniform(0.02, 0.1) * n * (n - 1) / 2))
        degree = 2.0 * edges / n
        graph = dict(graph="gnm", n=n, edges=edges)
    graph["weights"] = rng.choice(["one", "pm1", "pm1", "int"])
    if kind == "readout":
        return dict(kind=kind, trials=_log(rng, 4, 512), **graph)
    rule = rng.choice(["psa", "psa", "psa", "psa", "spsa", "tapsa", "period"])
    sigma = rng.choice([0.0, 0.05, 0.1, 0.2])
    trials = _log(rng, 1, 1024)
    cost = n * trials * (1.0 + min(degree, 80.0) / 8.0) * (10 if rule == "period" else 1)
    steps = max(10, min(_log(rng, 100, 2000), int(_MOST / cost)))
    entry = rng.choice(["job", "job", "job", "call", "noalloc"])
    if entry == "noalloc" and (n * trials > 4_000_000 or rule == "tapsa"):
        entry = "job"
    return dict(kind=kind, entry=entry, trials=trials, steps=steps, sigma=sigma, rule=rule, **graph)


# ---------------------------------------------------------------------------
# What a program has in hand, and one pass
# ---------------------------------------------------------------------------
def _outputs(trials, n):
    return dict(energy=torch.zeros(trials, dtype=torch.int64, device="cuda"),
                cut=torch.zeros(trials, dtype=torch.int64, device="cuda"),
                spins=torch.zeros((trials, n), dtype=torch.int8, device="cuda"))


def _spins(case, seed):
    rng = np.random.Generator(np.random.PCG64([seed, 77]))
    return (2 * rng.integers(0, 2, size=(case["trials"], case["n"]), dtype=np.int8) - 1).astype(np.int8)


def prepare(case, seed):
    ctx = _ctx()
    if case["kind"] == "batch":
        runs = _mix(case)
        jobs, outs = [], []
        for j, r in enumerate(runs):
            g = psa.Graph.from_edges(ctx, *_graph(r, seed * 1000 + j))
            jobs.append(psa.Job(ctx, g, case["steps"], r["trials"], seed * 1000 + j, **_options(r)))
        total = sum(r["trials"] for r in runs)
        energy, cut = (torch.zeros(total, dtype=torch.int64, device="cuda") for _ in range(2))
        spins = torch.zeros(sum(r["trials"] * r["n"] for r in runs), dtype=torch.int8, device="cuda")
        k = s = 0
        for r in runs:
            outs.append((energy[k:k + r["trials"]], cut[k:k + r["trials"]], spins[s:s + r["trials"] * r["n"]]))
            k += r["trials"]
            s += r["trials"] * r["n"]
        return dict(case=case, ctx=ctx, jobs=jobs, outs=outs, energy=energy, cut=cut, spins=spins)
    n, u, v, w = _graph(case, seed)
    g = psa.Graph.from_edges(ctx, n, u, v, w)
    state = dict(case=case, ctx=ctx, graph=g, seed=seed)
    if case["kind"] == "readout":
        job = psa.Job(ctx, g, 10, case["trials"], seed)
        job.write_spins(_spins(case, seed), 10)
        field = torch.zeros((case["trials"], n), dtype=torch.int32, device="cuda")
        state.update(job=job, field=field, **_outputs(case["trials"], n))
        return state
    if case["entry"] == "job":
        state.update(job=psa.Job(ctx, g, case["steps"], case["trials"], seed, **_options(case)))
    if case["entry"] != "call":
        state.update(_outputs(case["trials"], n))
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "batch":
        jobs, outs = state["jobs"], state["outs"]
        for job in jobs:
            job.reset()
        psa.jobs_step_batch(ctx, jobs, case["steps"])
        psa.jobs_energy_cut(ctx, jobs, [o[0] for o in outs], [o[1] for o in outs])
        for job, o in zip(jobs, outs):
            job.read_spins(o[2])
        return dict(energy=state["energy"], cut=state["cut"], spins=state["spins"])
    if case["kind"] == "readout":
        job = state["job"]
        job.energy_cut(state["energy"], state["cut"])
        job.local_field(state["field"])
        job.read_spins(state["spins"])
        return {k: state[k] for k in ("energy", "cut", "field", "spins")}
    if case["entry"] == "call":
        spins, energy, cut = psa.anneal(ctx, state["graph"], case["steps"], case["trials"], state["seed"],
                                        **_options(case))
        return dict(energy=energy, cut=cut, spins=spins)
    if case["entry"] == "noalloc":
        psa.anneal_noalloc(ctx, state["graph"], case["steps"], case["trials"], state["seed"],
                           spins_out=state["spins"], energy_out=state["energy"], cut_out=state["cut"],
                           **_options(case))
    else:
        job = state["job"]
        job.reset()
        job.step(case["steps"])
        job.energy_cut(state["energy"], state["cut"])
        job.read_spins(state["spins"])
    return {k: state[k] for k in ("energy", "cut", "spins")}


# ---------------------------------------------------------------------------
# What a pass cannot do without, and reference values
# ---------------------------------------------------------------------------
def _edges(case):
    return 2 * case["n"] if case["graph"] == "torus" else min(case["edges"], case["n"] * (case["n"] - 1) // 2)


def work(case):
    """Bytes: the edges once (a column and a weight in each direction), the
    per-p-bit factors once, every output once.  Operations of an update: a
    quarter of a 40-operation random block (two quarters with the timing
    gate), 18 for the uniform number, the pre-activation and the decision, and
    an add for each neighbour."""
    runs = _mix(case) if case["kind"] == "batch" else [case]
    nbytes = flops = 0.0
    for r in runs:
        n, trials, edges = r["n"], r["trials"], _edges(r)
        nbytes += 16.0 * edges + 16.0 * n + n * trials + 16.0 * trials
        if case["kind"] == "readout":
            nbytes += 5.0 * n * trials
            flops += 4.0 * edges * trials
            continue
        gated = r.get("sigma", 0.0) > 0 and r.get("rule", "psa") != "period"
        per_update = 28.0 + (12.0 if gated else 0.0) + 2.0 * edges / n
        flops += per_update * n * trials * case["steps"]
    return {"bytes": nbytes, "flops": flops}


def exact(case, seed):
    """Energy, cut and fields of a read-out in 64-bit integers.  An anneal has
    no value of its own in 64 bits: each decision is taken in single precision
    and every later one depends on it; its outputs are whole numbers."""
    if case["kind"] != "readout":
        return None
    n, u, v, w = (torch.as_tensor(x) for x in _graph(case, seed))
    m = torch.from_numpy(_spins(case, seed)).to(torch.int64)
    field = torch.empty_like(m)
    cut = torch.empty(m.shape[0], dtype=torch.int64)
    u, v, w = u.long(), v.long(), w.long()
    for k in range(m.shape[0]):
        mk = m[k]
        L = torch.zeros_like(mk)
        L.index_add_(0, u, -w * mk[v])
        L.index_add_(0, v, -w * mk[u])
        field[k] = L
        cut[k] = (w * (mk[u] != mk[v])).sum()
    energy = -(field * m).sum(dim=1) // 2
    return dict(energy=energy, cut=cut, field=field, spins=m)
