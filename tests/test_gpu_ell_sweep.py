"""Streaming sweeps (rows as wavefront-ordered ELL groups in device memory)
against the oracle, bit for bit: one and four trials per workgroup, each form
of the neighbour sums, row counts around a wavefront's 64 tasks and a
workgroup's lanes, long and empty rows, odd trial counts, factors past the
decision estimate's bound, and every input stage."""
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


def _weights(m, lo, hi, seed):
    rng = np.random.default_rng(seed)
    return (rng.integers(lo, hi + 1, m) * rng.choice([-1, 1], m)).astype(np.int32)


def _check(psa, ctx, n, u, v, j, trials, steps, tpw, h=None, batch=False, i0=(0.02, 0.5), sig=(0.2, 0.3, 0.2, 0.7), **kw):
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    sched = oracle.schedule(steps, *i0)
    lam, dl, thr = oracle.variability(n, 21, *sig)
    job = psa.Job(ctx, g, steps, trials, seed=21, i0=sched, sigma_lambda=sig[0], sigma_delta=sig[1],
                  sigma_nu=sig[2], p_mean=sig[3], trials_per_group=tpw, lanes_per_task=1 if tpw == 1 else 0,
                  path=psa.PSA_PATH_CSR, **kw)
    k = steps // 2
    for part in (k, steps - k):
        if batch:
            psa.jobs_step_batch(ctx, [job], part)
        else:
            job.step(part)
    ref = oracle.anneal(n, u, v, j, h, sched, lam, dl, thr, 21, 0, trials)
    np.testing.assert_array_equal(job.read_spins(), ref[0])
    E, C = job.energy_cut()
    np.testing.assert_array_equal(E, ref[1])
    np.testing.assert_array_equal(C, ref[2])
    job.close()
    g.close()


# one task; 64 tasks and one more; 1,024 lanes and one task more; odd counts
@pytest.mark.parametrize("n,m", [(2, 1), (5, 7), (256, 900), (257, 900), (4096, 9000), (4097, 9000), (6001, 14000)])
@pytest.mark.parametrize("tpw", [1, 4])
@pytest.mark.parametrize("top", [1, 7, 900])
def test_sizes_and_sums(psa, ctx, n, m, tpw, top):
    _, u, v, _ = inputs.gnm(n, m, 3 + n)
    j = _weights(u.size, 1, top, 5)
    h = np.random.default_rng(6).integers(-2, 3, n).astype(np.int32)
    _check(psa, ctx, n, u, v, j, 5, 6, tpw, h=h, batch=n % 2 == 0, i0=(0.02 / top, 0.5 / top))


# rows of 255 / 256 entries (byte and half sums), magnitudes at the halves'
# 13 bits and past it, at 15 bits and past it, a stored zero coupling
@pytest.mark.parametrize("deg,mag", [(255, 1), (256, 1), (51, 5), (52, 5), (8, 8191), (8, 8192), (3, 32767), (3, 32768),
                                     (6, 0)])
@pytest.mark.parametrize("tpw", [1, 4])
def test_row_sums_at_their_limits(psa, ctx, deg, mag, tpw):
    n = 301
    u = np.concatenate([np.zeros(deg, np.int32), np.arange(1, 40, dtype=np.int32)])
    v = np.concatenate([np.arange(1, deg + 1), 300 - np.arange(1, 40)]).astype(np.int32)
    keep = u != v
    pair = np.unique(np.stack([np.minimum(u, v), np.maximum(u, v)])[:, keep], axis=1)
    u, v = pair.astype(np.int32)
    j = np.where(np.arange(u.size) % 3 == 0, -mag, mag).astype(np.int32)
    if mag == 0:
        j[1::2] = 2
    s = max(mag, 1)
    _check(psa, ctx, n, u, v, j, 7, 8, tpw, i0=(0.02 / s, 0.4 / s))


@pytest.mark.parametrize("tpw", [1, 4])
@pytest.mark.parametrize("sig,i0", [((0.0, 0.0, 0.0, 1.0), (0.02, 0.5)),      # no gate, no factors
                                    ((0.0, 0.0, 0.5, 0.2), (0.02, 0.5)),      # update probabilities clipped to 0
                                    ((0.3, 400.0, 0.1, 0.8), (0.05, 2.0)),    # past the estimate's bound part-way
                                    ((0.2, 0.2, 0.0, 1.0), (1e-30, 3e38))])   # extreme schedule
def test_factors(psa, ctx, tpw, sig, i0):
    n, u, v, w = inputs.gnm(1501, 5000, 8)
    _check(psa, ctx, n, u, v, -w, 6, 12, tpw, sig=sig, i0=i0)


@pytest.mark.parametrize("tpw", [1, 4])
@pytest.mark.parametrize("rule", ["spsa", "tapsa", "period"])
@pytest.mark.parametrize("top", [1, 9, 2000])
def test_input_stages(psa, ctx, tpw, rule, top):
    n, u, v, _ = inputs.gnm(4203, 9000, 12)
    j = _weights(u.size, 1, top, 4)
    g = psa.Graph.from_edges(ctx, n, u, v, j, maxcut=False)
    S, T, sig = 9, 5, (0.1, 0.2, 0.1, 0.8)
    i0 = oracle.schedule(S, 0.02 / top, 0.9 / top)
    lam, dl, thr = oracle.variability(n, 13, *sig)
    kw = {"spsa": dict(algorithm=psa.PSA_ALG_SPSA), "tapsa": dict(algorithm=psa.PSA_ALG_TAPSA, window=3),
          "period": dict(t_res=4)}[rule]
    if rule == "period":  # more distinct periods than the class sweep takes
        per = (1 + np.random.default_rng(3).integers(0, 200, n)).astype(np.uint32)
        kw["period"] = per
    job = psa.Job(ctx, g, S, T, seed=13, i0=i0, sigma_lambda=sig[0], sigma_delta=sig[1], sigma_nu=sig[2],
                  p_mean=sig[3], trials_per_group=tpw, lanes_per_task=1 if tpw == 1 else 0, path=psa.PSA_PATH_CSR, **kw)
    ref, state, t = oracle.init_spins(n, 13, 0, T), None, 0
    for k in (2, 3, 4):
        job.step(k)
        if rule == "spsa":
            ref, state = oracle.run_spsa(n, u, v, j, None, i0, lam, dl, thr, 1 << 23, 13, 0, T, t, t + k, ref, state)
        elif rule == "tapsa":
            ref, state = oracle.run_tapsa(n, u, v, j, None, i0, lam, dl, thr, 3, 13, 0, T, t, t + k, ref, state)
        else:
            ref = oracle.run_period(n, u, v, j, None, i0, lam, dl, per, 4, 13, 0, T, t, t + k, ref)
        t += k
        np.testing.assert_array_equal(job.read_spins(), ref, err_msg=f"after step {t}")
