"""Runs of few trials, whose thresholds are drawn ahead of the steps, against
the oracle bit for bit: task counts around a wavefront and a workgroup, rows
around the registers' share, row sums at the byte's limit, chunks that end
anywhere, gates and factors, saturated schedules, padding trials, and the
conditions under which the other sweeps take the run."""
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


def _check(psa, ctx, n, u, v, j, trials, parts, i0, sig=(0.1, 0.2, 0.1, 0.8), h=None, seed=31):
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    S = sum(parts)
    sched = np.asarray(oracle.schedule(S, *i0) if isinstance(i0, tuple) else i0, np.float32)
    lam, dl, thr = oracle.variability(n, seed, *sig)
    job = psa.Job(ctx, g, S, trials, seed=seed, i0=sched, sigma_lambda=sig[0], sigma_delta=sig[1], sigma_nu=sig[2],
                  p_mean=sig[3], path=psa.PSA_PATH_CSR)
    for k in parts:
        job.step(k)
    some = min(trials, 6)
    ref = oracle.anneal(n, u, v, j, h, sched, lam, dl, thr, seed, 0, some)
    got = job.read_spins()
    np.testing.assert_array_equal(got[:some], ref[0])
    # every trial: the one-trial sweep
    other = psa.Job(ctx, g, S, trials, seed=seed, i0=sched, sigma_lambda=sig[0], sigma_delta=sig[1],
                    sigma_nu=sig[2], p_mean=sig[3], path=psa.PSA_PATH_CSR, trials_per_group=1)
    other.step(S)
    np.testing.assert_array_equal(got, other.read_spins())
    job.close()
    other.close()
    g.close()


def _weights(m, top, seed):
    rng = np.random.default_rng(seed)
    return (rng.integers(1, top + 1, m) * rng.choice([-1, 1], m)).astype(np.int32)


# one to four p-bits per lane, a position more; the last is one p-bit too many
@pytest.mark.parametrize("n,m", [(2, 1), (5, 7), (64, 300), (65, 200), (256, 900), (257, 900), (513, 4000),
                                 (800, 20000), (897, 20000), (1024, 9000), (1024, 3000), (1025, 3000), (2048, 12000),
                                 (2049, 12500), (4032, 25000), (4033, 12000)])
@pytest.mark.parametrize("top", [1, 5])
@pytest.mark.parametrize("trials", [1, 6, 100])
def test_sizes(psa, ctx, n, m, top, trials):
    _, u, v, _ = inputs.gnm(n, m, n)
    h = np.random.default_rng(6).integers(-2, 3, n).astype(np.int32)
    _check(psa, ctx, n, u, v, _weights(u.size, top, 5), trials, (65, 3, 70), (0.05 / top, 2.0 / top), h=h)


# rows of 48 entries fill the registers' share, one or three more are read at
# every step; sums at 126 and, past it, the other sweeps
@pytest.mark.parametrize("deg,mag", [(12, 9), (16, 1), (17, 1), (48, 1), (49, 1), (51, 1), (126, 1), (127, 1), (3, 42), (3, 43), (1, 126),
                                     (1, 127), (8, 2), (9, 2), (48, 2), (49, 2), (63, 2)])
def test_rows_at_their_limits(psa, ctx, deg, mag):
    n = 301
    u = np.concatenate([np.zeros(deg, np.int32), np.arange(1, 40, dtype=np.int32)])
    v = np.concatenate([np.arange(1, deg + 1), 300 - np.arange(1, 40)]).astype(np.int32)
    j = np.where(np.arange(u.size) % 3 == 0, -mag, mag).astype(np.int32)
    _check(psa, ctx, n, u, v, j, 5, (80,), (0.02 / mag, 1.5 / mag))


# chunks of 16, 32, 64, .. steps: calls that end in and at their edges
@pytest.mark.parametrize("parts", [(64,), (67,), (112, 113), (500, 64, 63), (1201,)])
def test_chunks(psa, ctx, parts):
    n, u, v, w = inputs.gnm(600, 1800, 8)
    _check(psa, ctx, n, u, v, -w, 9, parts, (0.05, 5.0))


@pytest.mark.parametrize("sig", [(0.0, 0.0, 0.0, 1.0), (0.0, 0.0, 0.5, 0.2), (0.1, 300.0, 0.1, 0.8), (0.2, 0.2, 0.2, 0.8),
                                 (0.6, 0.0, 0.0, 1.0)])
@pytest.mark.parametrize("i0", [(0.0003, 0.001), (0.05, 5.0), (1.0, 1e4), (1e6, 1e9), (1e-6, 1e-3), (1e-30, 3e38)])
def test_factors(psa, ctx, sig, i0):
    n, u, v, w = inputs.gnm(801, 2500, 8)
    _check(psa, ctx, n, u, v, -w, 37, (150,), i0, sig=sig)


def test_pre_activations_in_the_tail(psa, ctx):
    """x from 5 to 9 on most updates, where tanh rounds to a few values below 1
    and the threshold is taken from the decision itself."""
    n, u, v, w = inputs.gnm(2000, 6000, 3)
    _check(psa, ctx, n, u, v, -w, 8, (300,), np.full(300, 1.4, np.float32), h=np.full(n, 3, np.int32))


@pytest.mark.parametrize("n,trials", [(500, 127), (500, 128), (500, 129), (1500, 112), (1500, 113), (2500, 128), (2500, 129)])
def test_trials_around_half_the_units(psa, ctx, n, trials):
    _, u, v, w = inputs.gnm(n, 3 * n, 3)
    _check(psa, ctx, n, u, v, -w, trials, (70,), (0.05, 3.0))


def test_two_jobs_in_turn(psa, ctx):
    """Calls of two jobs of one context follow each other on its buffer."""
    n, u, v, w = inputs.gnm(900, 2700, 4)
    g = psa.Graph.from_edges(ctx, n, u, v, -w, maxcut=False)
    sched = oracle.schedule(200, 0.05, 3.0)
    kw = dict(i0=sched, sigma_lambda=0.1, sigma_delta=0.1, sigma_nu=0.1, p_mean=0.8, path=psa.PSA_PATH_CSR)
    jobs = [psa.Job(ctx, g, 200, 11, seed=s, **kw) for s in (1, 2)]
    for _ in range(2):
        for job in jobs:
            job.step(100)
    for s, job in zip((1, 2), jobs):
        lam, dl, thr = oracle.variability(n, s, 0.1, 0.1, 0.1, 0.8)
        np.testing.assert_array_equal(job.read_spins(), oracle.anneal(n, u, v, -w, None, sched, lam, dl, thr, s, 0, 11)[0])
