"""Sweep with thresholds drawn ahead on graphs whose last wavefronts hold only
p-bits without neighbours, one to four p-bits per lane, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    from paper_2601_14476_amd import psa as mod
    return mod


@pytest.mark.parametrize("n,edges", [(65, 1), (257, 100), (1025, 512), (1100, 3), (2048, 600), (2049, 1024), (4032, 5)])
def test_empty_wavefronts(psa, n, edges):
    ctx = psa.Context(0)
    u = (2 * np.arange(edges) % (n - 1)).astype(np.int32)
    v = u + 1
    j = np.where(np.arange(edges) % 2 == 0, 2, -3).astype(np.int32)
    h = np.random.default_rng(1).integers(-2, 3, n).astype(np.int32)
    S, T, sig = 70, 5, (0.1, 0.2, 0.1, 0.8)
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    i0 = oracle.schedule(S, 0.02, 1.0)
    job = psa.Job(ctx, g, S, T, seed=5, i0=i0, sigma_lambda=sig[0], sigma_delta=sig[1], sigma_nu=sig[2], p_mean=sig[3],
                  path=psa.PSA_PATH_CSR)
    job.step(S)
    lam, dl, thr = oracle.variability(n, 5, *sig)
    np.testing.assert_array_equal(job.read_spins(), oracle.anneal(n, u, v, j, h, i0, lam, dl, thr, 5, 0, T)[0])
    job.close()
    g.close()
    ctx.close()
