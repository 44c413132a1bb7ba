"""The tuning cache tells runs on different sweeps apart, and the tuner times what
an untuned run would take."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    from paper_2601_14476_amd import psa as mod
    return mod


@pytest.fixture()
def ctx(psa):
    c = psa.Context(0)
    yield c
    c.close()


KW = dict(sigma_lambda=0.1, sigma_delta=0.1, sigma_nu=0.1, p_mean=0.8)


def test_classes(psa, ctx):
    n, u, v, w = inputs.gnm(700, 2100, 5)
    g = psa.Graph.from_edges(ctx, n, u, v, w)
    count = 0
    for kw in (dict(), dict(t_res=4), dict(t_res=9), dict(algorithm=psa.PSA_ALG_TAPSA, window=2),
               dict(algorithm=psa.PSA_ALG_TAPSA, window=30)):
        for _ in range(2):
            psa.tune_get(ctx, g, 20, 12, 1, **KW, **kw)
        count += 1
        assert psa.tune_cache_size(ctx) == count, kw
    # sums of |J| past the four-trial sums' halves and past the spin-bit rows'
    for mag in (30000, 60):
        gw = psa.Graph.from_edges(ctx, n, u, v, (w * mag).astype(np.int32) + np.arange(w.size, dtype=np.int32) % 3)
        psa.tune_get(ctx, gw, 20, 12, 1, i0_min=1e-4, i0_max=1e-2, **KW)
        count += 1
        assert psa.tune_cache_size(ctx) == count, mag
        gw.close()
    g.close()


def test_tuned_run_alone_draws_ahead_as_the_untuned_one(psa, ctx):
    """800 p-bits of degree 48, 10 trials: the untuned run takes a third of the
    time of any fixed shape, so the tuned one has to be it."""
    n, u, v, w = inputs.gnm(800, 19176, 2)
    g = psa.Graph.from_edges(ctx, n, u, v, w)
    r = psa.autotune(ctx, g, 400, 10, 1, **KW)
    assert (r["path"], r["trials_per_group"], r["lanes_per_task"]) == (psa.PSA_PATH_CSR, 0, 0), r
    assert r["us_per_step"] == min(x for x in (r["csr_us_per_step"], r["dense_us_per_step"]) if x > 0)
    tuned, plain = (psa.Job(ctx, g, 400, 10, 1, tune=t, **KW) for t in (True, False))
    ctx.set_timing(True)
    launches = []
    for job in (tuned, plain):
        ctx.timing()
        job.step(400)
        launches.append(ctx.timing()["anneal_launches"])
    ctx.set_timing(False)
    assert launches[0] == launches[1] > 1
    np.testing.assert_array_equal(tuned.read_spins(), plain.read_spins())
    g2 = psa.Graph.from_edges(ctx, n, u, v, w)
    # a schedule shorter than the sweep's least call is timed as it would run
    assert psa.autotune(ctx, g2, 40, 10, 1, **KW)["candidates"] >= 5


def test_tuned_jobs_of_a_batch_leave_the_shape_to_it(psa, ctx):
    """Twelve graphs of 3,000 p-bits, degree 6, 64 trials: a batch takes four trials
    per workgroup for them, tuned or not."""
    runs = []
    for s in range(12):
        n, u, v, w = inputs.gnm(3000 + 7 * s, 9000, 40 + s)
        runs.append(psa.Graph.from_edges(ctx, n, u, v, w))
    r = psa.autotune(ctx, runs[0], 120, 64, 1, batch=True, **KW)
    assert r["path"] == psa.PSA_PATH_CSR and r["candidates"] >= 5, r
    plain = psa.anneal_batch(ctx, [(g, 60, 64, 3, dict(KW)) for g in runs], spins=True)
    tuned = psa.anneal_batch(ctx, [(g, 60, 64, 3, dict(KW, tune=True)) for g in runs], spins=True)
    for a, b in zip(plain, tuned):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
