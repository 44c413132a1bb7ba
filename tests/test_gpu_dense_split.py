"""Dense steps over 64-row items (the waves split the columns) against the
oracle on sampled trials and, for every trial, against the CSR path: one run
alone and several in a list, each coupling encoding, trial tiles of 16, 32 and
64, chunk counts below and past the four waves' share, identity factors and
the general epilogue."""
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


# n around the chunks (256 columns for +-1 and +1 weights, 128 for others):
# 1 to 9 chunks; trials that take 16-, 32- (and, int8 only, 64-) trial tiles
@pytest.mark.parametrize("n,trials,kind", [(64, 5, "one"), (257, 33, "pm1"), (700, 2048, "int"), (1000, 1024, "one"),
                                           (1000, 1030, "pm1"), (2100, 40, "pm1"), (1100, 64, "int"), (300, 700, "int")])
@pytest.mark.parametrize("sig", [(0.0, 0.0, 0.0, 1.0), (0.1, 0.2, 0.1, 0.8)])
@pytest.mark.parametrize("runs", [1, 2])
def test_split_steps(psa, ctx, n, trials, kind, sig, runs):
    rng = np.random.default_rng(n)
    _, u, v, _ = inputs.gnm(n, n * min(n - 1, 24) // 2, n)
    j = {"one": -np.ones(u.size), "pm1": rng.choice([-1, 1], u.size), "int": rng.integers(1, 6, u.size) * rng.choice([-1, 1], u.size)}
    j = j[kind].astype(np.int32)
    h = rng.integers(-2, 3, n).astype(np.int32)
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    S = 5
    i0 = oracle.schedule(S, 0.05, 0.6)
    kw = dict(i0=i0, sigma_lambda=sig[0], sigma_delta=sig[1], sigma_nu=sig[2], p_mean=sig[3])
    jobs = [psa.Job(ctx, g, S, trials, 11 + r, path=psa.PSA_PATH_DENSE, **kw) for r in range(runs)]
    for k in (2, 3):
        if runs == 1:
            jobs[0].step(k)
        else:
            psa.jobs_step_batch(ctx, jobs, k)
    for r, job in enumerate(jobs):
        got = job.read_spins()
        ref = psa.Job(ctx, g, S, trials, 11 + r, path=psa.PSA_PATH_CSR, **kw)
        ref.step(S)
        np.testing.assert_array_equal(got, ref.read_spins())
        lam, dl, thr = oracle.variability(n, 11 + r, *sig)
        some = min(trials, 3)
        np.testing.assert_array_equal(got[:some], oracle.anneal(n, u, v, j, h, i0, lam, dl, thr, 11 + r, 0, some)[0])
