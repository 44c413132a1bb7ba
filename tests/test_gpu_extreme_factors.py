"""Factors at the ends of the float range (lambda and delta need only be
finite) against the oracle, bit for bit: products of a factor, the field bound
and the decision's constants that overflow, subnormal factors, and schedules
that overflow beside fields that are all zero."""
import numpy as np
import pytest

import oracle
from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    from paper_2601_14476_amd import psa as mod
    return mod


@pytest.fixture(scope="module")
def ctx(psa):
    c = psa.Context(0)
    yield c
    c.close()


SHAPES = {"streaming, one trial": dict(trials_per_group=1, lanes_per_task=1), "streaming, four trials": dict(trials_per_group=4),
          "two lanes per task": dict(trials_per_group=1, lanes_per_task=2),
          "four lanes per task": dict(trials_per_group=1, lanes_per_task=4), "automatic": dict()}


def _check(psa, ctx, n, u, v, j, lam, delta, i0, h=None, gate=False, batch=False, rule="psa", **shape):
    rng = np.random.default_rng(3)
    lam = np.full(n, lam, np.float32) if np.isscalar(lam) else np.asarray(lam, np.float32)
    delta = np.full(n, delta, np.float32) if np.isscalar(delta) else np.asarray(delta, np.float32)
    thr = rng.integers(1 << 23, 1 << 24, n).astype(np.uint32) if gate else np.full(n, 1 << 24, np.uint32)
    i0 = np.asarray(i0, np.float32)
    T, S = 6, i0.size
    kw = dict(spsa=dict(algorithm=psa.PSA_ALG_SPSA), tapsa=dict(algorithm=psa.PSA_ALG_TAPSA, window=3)).get(rule, {})
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    job = psa.Job(ctx, g, S, T, seed=9, i0=i0, lam=lam, delta=delta, thr24=thr, path=psa.PSA_PATH_CSR, **shape, **kw)
    if batch:
        psa.jobs_step_batch(ctx, [job], S)
    else:
        job.step(S)
    if rule == "spsa":
        ref = oracle.run_spsa(n, u, v, j, h, i0, lam, delta, thr, 1 << 23, 9, 0, T, 0, S, oracle.init_spins(n, 9, 0, T), None)[0]
    elif rule == "tapsa":
        ref = oracle.run_tapsa(n, u, v, j, h, i0, lam, delta, thr, 3, 9, 0, T, 0, S, oracle.init_spins(n, 9, 0, T), None)[0]
    else:
        ref = oracle.anneal(n, u, v, j, h, i0, lam, delta, thr, 9, 0, T)[0]
    np.testing.assert_array_equal(job.read_spins(), ref)
    job.close()
    g.close()


# (lambda, delta, I0): the exponent's factor 2 lambda log2 e past the float
# range; in it, but not times the field; lambda delta past it, with I0 = 0 too;
# subnormal lambda beside a huge delta
FACTORS = {"lambda past the range": (6.5e37, 0.0, [2e-38, 1.5e-38, 3e-38]),
           "lambda at the end": (3.4e38, 0.0, [1.2e-38, 2e-38, 5e-39]),
           "lambda times the field": (1e37, 0.0, [3e-38, 1e-38, 6e-38]),
           "lambda times half the field": (-2.5e37, 0.25, [2e-38, 1.3e-38]),
           "lambda delta past the range": (1.0, 1.3e38, [0.0, 1e-38, 0.0, 5e-39]),
           "lambda delta in double only": (1e30, 1e30, [0.0, 1e-45, 0.0]),
           "subnormal lambda": (2.8e-45, 3e38, [1e6, 3e6, 2e6])}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("name", FACTORS)
@pytest.mark.parametrize("top", [1, 5])
def test_factors_past_the_range(psa, ctx, shape, name, top):
    lam, delta, i0 = FACTORS[name]
    n, u, v, w = inputs.gnm(1501, 5000, 8)
    j = (w * np.random.default_rng(2).integers(1, top + 1, w.size)).astype(np.int32)
    _check(psa, ctx, n, u, v, j, lam, delta, i0, **SHAPES[shape])
    _check(psa, ctx, n, u, v, j, lam, delta, i0, gate=True, batch=True, **SHAPES[shape])


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("rule", ["psa", "spsa", "tapsa"])
def test_one_extreme_p_bit_in_each_task(psa, ctx, shape, rule):
    n, u, v, w = inputs.gnm(1203, 4000, 4)
    lam = np.ones(n, np.float32)
    lam[::4] = 1e38
    _check(psa, ctx, n, u, v, w, lam, 0.0, np.geomspace(1e-38, 1e-36, 5), rule=rule, **SHAPES[shape])


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("top", [1, 5])
@pytest.mark.parametrize("batch", [False, True])
def test_schedule_past_the_range_on_zero_fields(psa, ctx, shape, top, batch):
    """I0 times the exponent's factor overflows and the fields of whole
    wavefronts are 0: each such p-bit is up with probability one half."""
    n = 1500
    u, v = np.arange(0, 40, 2, dtype=np.int32), np.arange(1, 41, 2, dtype=np.int32)
    j = np.where(np.arange(u.size) % 2 == 0, top, -top).astype(np.int32)
    _check(psa, ctx, n, u, v, j, 1.0, 0.0, [1e38, 3e38, 6e37, 1e38], batch=batch, **SHAPES[shape])
