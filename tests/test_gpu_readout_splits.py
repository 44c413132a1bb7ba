"""Read-outs around the lines between their splits (spins of four and sixteen
trials per lane, lanes side by side and on a row's edges) against numpy's 64-bit
integers, alone and in a batch."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


# 350,000 spins (energy) and 1,200,000 (fields) from both sides, rows below and
# above mean degree 12, trial counts that leave chunks of four lanes incomplete
@pytest.mark.parametrize("n,m,trials", [(1, 0, 3), (3499, 20000, 100), (3500, 20000, 100), (1750, 12000, 197), (1001, 12000, 349),
                                        (1001, 12000, 353), (3000, 9000, 396), (3000, 9000, 405), (61, 1500, 5741), (2400, 30000, 499),
                                        (2400, 30000, 501)])
def test_around_the_lines(n, m, trials):
    from paper_2601_14476_amd import psa
    ctx = psa.Context(0)
    rng = np.random.default_rng(n + trials)
    u, v, j = (inputs.gnm(n, m, 5)[1:] if m else (np.zeros(0, np.int32),) * 3)
    j = (j * rng.integers(1, 5, j.size)).astype(np.int32)
    h = rng.integers(-3, 4, n).astype(np.int32)
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    job = psa.Job(ctx, g, 4, trials, 1, i0_min=0.1, i0_max=1.0, path=psa.PSA_PATH_CSR)
    s = (2 * rng.integers(0, 2, (trials, n), dtype=np.int8) - 1).astype(np.int8)
    job.write_spins(s, 2)
    J = np.zeros((n, n), np.int64)
    np.add.at(J, (u, v), j)
    np.add.at(J, (v, u), j)
    m64 = s.astype(np.float64)  # exact: sums below 2^53
    field = (m64 @ J.astype(np.float64)).astype(np.int64) + h
    pair = ((field - h) * s).sum(axis=1)
    energy = -(s * h.astype(np.int64)).sum(axis=1) - pair // 2
    cut = (pair - J.sum()) // 4
    for E, C in (job.energy_cut(), tuple(x[0] for x in psa.jobs_energy_cut(ctx, [job]))):
        np.testing.assert_array_equal(E, energy)
        np.testing.assert_array_equal(C, cut)
    np.testing.assert_array_equal(job.local_field(), field)
    job.close()
    g.close()
    ctx.close()
