"""Which sweep steps a run alone, seen in the launches that the context's timing
counts: one per call, or one per chunk of 16, 32, 64, ... steps and one more where
the thresholds are drawn ahead.  Both sides of every limit of that rule."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    from paper_2601_14476_amd import psa as mod
    return mod


@pytest.fixture(scope="module")
def ctx(psa):
    c = psa.Context(0)
    c.set_timing(True)
    yield c
    c.close()


def _launches(psa, ctx, n, u, v, j, trials, steps=80, i0=(0.05, 3.0), **kw):
    g = psa.Graph.from_edges(ctx, n, u, v, j, maxcut=False)
    opt = dict(sigma_lambda=0.1, sigma_delta=0.1, sigma_nu=0.1, p_mean=0.8, i0_min=i0[0], i0_max=i0[1], path=psa.PSA_PATH_CSR)
    opt.update(kw)
    job = psa.Job(ctx, g, max(steps, 80), trials, 1, **opt)
    ctx.timing()
    job.step(steps)
    count = ctx.timing()["anneal_launches"]
    job.close()
    g.close()
    return count


AHEAD = 4  # 80 steps: chunks of 16, 32 and 32, and the last one's steps


@pytest.mark.parametrize("n,trials,ahead", [(500, 127, True), (500, 128, True), (500, 129, False), (1500, 112, True), (1500, 113, False),
                                            (2500, 128, True), (2500, 129, False), (4032, 8, True), (4033, 8, False)])
def test_sizes(psa, ctx, n, trials, ahead):
    _, u, v, w = inputs.gnm(n, 3 * n, 3)
    assert _launches(psa, ctx, n, u, v, -w, trials) == (AHEAD if ahead else 1)


@pytest.mark.parametrize("deg,mag,ahead", [(126, 1, True), (127, 1, False), (3, 42, True), (3, 43, False)])
def test_row_sums(psa, ctx, deg, mag, ahead):
    u, v = np.zeros(deg, np.int32), np.arange(1, deg + 1, dtype=np.int32)
    assert _launches(psa, ctx, 301, u, v, np.full(deg, mag, np.int32), 5, i0=(0.02 / mag, 1.5 / mag)) == (AHEAD if ahead else 1)


def test_long_rows_past_two_per_lane(psa, ctx):
    for m, ahead in ((20000, True), (20008, False)):  # mean degree 16 at 2,500 p-bits
        _, u, v, w = inputs.gnm(2500, m, 3)
        assert _launches(psa, ctx, 2500, u, v, -w, 8) == (AHEAD if ahead else 1)


@pytest.mark.parametrize("steps,count", [(63, 1), (64, 4), (112, 4), (113, 5), (496, 6), (500, 7)])
def test_chunks(psa, ctx, steps, count):
    _, u, v, w = inputs.gnm(600, 1800, 3)
    assert _launches(psa, ctx, 600, u, v, -w, 9, steps=steps) == count


def test_other_rules_and_options(psa, ctx):
    n, u, v, w = inputs.gnm(600, 1800, 3)
    run = lambda **kw: _launches(psa, ctx, n, u, v, -w, 9, **kw)
    assert run() == AHEAD
    assert run(algorithm=psa.PSA_ALG_SPSA) == run(algorithm=psa.PSA_ALG_TAPSA) == run(t_res=2) == 1
    assert run(trials_per_group=1) == run(lanes_per_task=2) == run(block=512) == 1
    assert run(i0=(1e-5, 1.0)) == 1      # I0 lambda below 2^-12
    assert run(delta=np.full(n, 2.0 ** 21, np.float32)) == 1
