"""A kept job of few steps has the dense path from the start; single runs of the
same schedule come to it and give the same results on either path."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


def test_kept_and_single():
    from paper_2601_14476_amd import psa
    ctx = psa.Context(0)
    n, u, v, j = inputs.gnm(3000, 270000, 5)
    first = None
    g = psa.Graph.from_edges(ctx, n, u, v, j, maxcut=True)
    for _ in range(40):
        got = psa.anneal(ctx, g, 12, 27, 9)
        first = first or got
        for a, b in zip(got, first):
            np.testing.assert_array_equal(a, b)
    fresh = psa.Graph.from_edges(ctx, n, u, v, j, maxcut=True)
    for graph in (fresh, g):
        job = psa.Job(ctx, graph, 12, 27, 9)
        assert job.info()["path"] == psa.PSA_PATH_DENSE
        job.step(12)
        E, C = job.energy_cut()
        job.close()
    np.testing.assert_array_equal(C, [x for x in first if x.ndim == 1][-1])
    fresh.close()
    g.close()
    ctx.close()
