"""Read-outs of graphs with long rows around the lines between their splits,
against numpy's 64-bit integers, alone and in a batch with a short-rowed run."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


def reference(n, u, v, j, s):
    J = np.zeros((n, n), np.int64)
    np.add.at(J, (u, v), j)
    np.add.at(J, (v, u), j)
    field = (s.astype(np.float64) @ J.astype(np.float64)).astype(np.int64)  # exact: sums below 2^53
    pair = (field * s).sum(axis=1)
    return field, -pair // 2, (pair - J.sum()) // 4


# mean degrees 32, 48, 90 and 300, 150,000 and 400,000 spins, 4 and 16 trials, a
# million spins, each from both sides
@pytest.mark.parametrize("n,d,trials", [(701, 33, 3), (701, 47, 16), (701, 49, 17), (999, 89, 150), (1000, 91, 150), (1001, 91, 149),
                                        (999, 299, 61), (901, 301, 445), (999, 91, 401), (2003, 310, 15), (1100, 310, 4), (2700, 60, 371)])
def test_long_rows(n, d, trials):
    from paper_2601_14476_amd import psa
    ctx = psa.Context(0)
    rng = np.random.default_rng(n + d + trials)
    jobs, want = [], []
    for nn, dd, tt in ((n, d, trials), (60, 4, 5)):
        u, v, j = inputs.gnm(nn, nn * dd // 2 + 1, 5)[1:]
        g = psa.Graph.from_edges(ctx, nn, u, v, j, maxcut=False)
        job = psa.Job(ctx, g, 4, tt, 1, i0_min=0.1, i0_max=1.0, path=psa.PSA_PATH_CSR)
        s = (2 * rng.integers(0, 2, (tt, nn), dtype=np.int8) - 1).astype(np.int8)
        job.write_spins(s, 2)
        jobs.append((g, job))
        want.append(reference(nn, u, v, j, s))
        field, energy, cut = want[-1]
        E, C = job.energy_cut()
        np.testing.assert_array_equal(E, energy)
        np.testing.assert_array_equal(C, cut)
        np.testing.assert_array_equal(job.local_field(), field)
    for E, C, (_, energy, cut) in zip(*psa.jobs_energy_cut(ctx, [job for _, job in jobs]), want):
        np.testing.assert_array_equal(E, energy)
        np.testing.assert_array_equal(C, cut)
    for g, job in jobs:
        job.close()
        g.close()
    ctx.close()
