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
