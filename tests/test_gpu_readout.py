"""Read-outs (energy, cut, local fields, spins) of given spins against numpy's
64-bit integers: every split of the read-out lanes -- sixteen or four trials
per lane, chunks side by side, shares of long rows --, row blocks and chunks
left over, 32- and 64-bit sums, with and without biases."""
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
    yield c
    c.close()


def _reference(n, u, v, j, h, m):
    m = m.astype(np.int64)
    field = np.tile(h.astype(np.int64), (m.shape[0], 1))
    pair = np.zeros(m.shape[0], np.int64)
    cut = np.zeros(m.shape[0], np.int64)
    for k in range(m.shape[0]):
        np.add.at(field[k], u, j * m[k, v])
        np.add.at(field[k], v, j * m[k, u])
        same = m[k, u] * m[k, v]
        pair[k] = (j * same).sum()
        cut[k] = (-j * (same < 0)).sum()
    return -(m @ h.astype(np.int64)) - pair, cut, field


# few waves (four trials per lane) and many (sixteen, 1 to 16 chunks side by
# side); degrees below 12, below 48 and above; 256-row blocks with a remainder
@pytest.mark.parametrize("n,m,trials,scale", [
    (1, 0, 1, 1), (255, 900, 5, 1), (256, 8000, 64, 1), (257, 13000, 17, 3), (700, 20000, 300, 1),
    (5003, 15000, 1000, 1), (3001, 45000, 515, 1), (2100, 120000, 260, 2), (1500, 9000, 2048, 1),
    (600, 3000, 40, 300000), (4000, 16000, 1030, 300000), (1024, 4096, 1552, 1)])
@pytest.mark.parametrize("bias", [False, True])
def test_readouts(psa, ctx, n, m, trials, scale, bias):
    rng = np.random.default_rng(n + trials)
    if m:
        _, u, v, w = inputs.gnm(n, m, 7)
    else:
        u = v = w = np.zeros(0, np.int32)
    j = (w * scale).astype(np.int32)
    h = rng.integers(-3, 4, n).astype(np.int32) if bias else np.zeros(n, np.int32)
    g = psa.Graph.from_edges(ctx, n, u, v, j, h=h, maxcut=False)
    jobs = [psa.Job(ctx, g, 4, t, 1, i0_min=0.1, i0_max=1.0, path=psa.PSA_PATH_CSR) for t in (trials, max(1, trials // 3))]
    spins = [(2 * rng.integers(0, 2, (job.trials, n), dtype=np.int8) - 1).astype(np.int8) for job in jobs]
    refs = []
    for job, s in zip(jobs, spins):
        job.write_spins(s, 2)
        refs.append(_reference(n, u, v, j.astype(np.int64), h, s))
        E, C = job.energy_cut()
        np.testing.assert_array_equal(E, refs[-1][0])
        np.testing.assert_array_equal(C, refs[-1][1])
        np.testing.assert_array_equal(job.local_field(), refs[-1][2])
        np.testing.assert_array_equal(job.read_spins(), s)
    for (E, C), ref in zip(zip(*psa.jobs_energy_cut(ctx, jobs)), refs):
        np.testing.assert_array_equal(E, ref[0])
        np.testing.assert_array_equal(C, ref[1])
