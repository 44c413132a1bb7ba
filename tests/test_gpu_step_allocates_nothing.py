"""Device memory is taken when a job is created: stepping it takes none, whatever
sweep its steps run, and jobs that are only stepped in batches take no buffer
that stepping alone would need."""
import numpy as np
import pytest

from paper_2601_14476_amd import inputs

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("n,m,trials", [(500, 1500, 20), (2000, 6000, 100), (4000, 12000, 8), (6000, 18000, 8)])
def test_step_takes_no_memory(n, m, trials):
    from paper_2601_14476_amd import psa
    n, u, v, w = inputs.gnm(n, m, 1)
    for first in (True, False):  # the runtime loads the kernels at their first launch
        ctx = psa.Context(0)
        g = psa.Graph.from_edges(ctx, n, u, v, w)
        job = psa.Job(ctx, g, 300, trials, 1, path=psa.PSA_PATH_CSR)
        ctx.synchronize()
        before = _free()
        job.step(40)
        job.step(200)
        ctx.synchronize()
        assert first or _free() == before
        job.close()
        g.close()
        ctx.close()


def test_batch_entry_takes_no_step_buffer():
    from paper_2601_14476_amd import psa
    ctx = psa.Context(0)
    n, u, v, w = inputs.gnm(500, 1500, 1)
    g = psa.Graph.from_edges(ctx, n, u, v, w)
    items = [(g, 100, 8, s, dict(path=psa.PSA_PATH_CSR)) for s in (1, 2)]
    before = _free()
    psa.anneal_batch(ctx, items)
    ctx.synchronize()
    assert before - _free() < (32 << 20)  # tables; the step buffer is 64 MiB
    g.close()
    ctx.close()
