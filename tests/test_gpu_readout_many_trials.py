"""Read-outs of a few p-bits and very many trials: grids past 2^32 threads or
65,535 workgroups of one dimension (the largest trial count is 2^28)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psa():
    from paper_2601_14476_amd import psa as mod
    return mod


@pytest.mark.parametrize("n,trials,field", [(2, 1 << 28, False), (3, 65537 * 16, True), (3, 65537 * 64 - 1, True)])
def test_many_trials(psa, n, trials, field):
    import torch
    ctx = psa.Context(0)
    g = psa.Graph.from_edges(ctx, n, np.array([0], np.int32), np.array([1], np.int32), np.array([3], np.int32),
                             h=np.arange(n, dtype=np.int32), maxcut=False)
    job = psa.Job(ctx, g, 4, trials, 1, i0_min=0.1, i0_max=1.0, path=psa.PSA_PATH_CSR)
    spins = torch.zeros((trials, n), dtype=torch.int8, device="cuda")
    energy, cut, e2, c2 = (torch.zeros(trials, dtype=torch.int64, device="cuda") for _ in range(4))
    m = (2 * torch.randint(0, 2, (trials, n), dtype=torch.int8, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) - 1)
    torch.cuda.synchronize()
    job.write_spins(m, 1)
    job.read_spins(spins)
    job.energy_cut(energy, cut)
    psa.jobs_energy_cut(ctx, [job], [e2], [c2])
    ctx.synchronize()
    assert torch.equal(spins, m)
    pair = 3 * m[:, 0].long() * m[:, 1]
    want = -pair
    for i in range(n):
        want -= i * m[:, i].long()
    assert torch.equal(energy, want) and torch.equal(e2, want)
    want = torch.where(pair < 0, -3, 0)  # w = -J
    assert torch.equal(cut, want) and torch.equal(c2, want)
    if field:
        L = torch.zeros((trials, n), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        job.local_field(L)
        ctx.synchronize()
        want = torch.arange(n, dtype=torch.int32, device="cuda").repeat(trials, 1)
        want[:, 0] += 3 * m[:, 1]
        want[:, 1] += 3 * m[:, 0]
        assert torch.equal(L, want)
    job.close()
    g.close()
    ctx.close()
    torch.cuda.empty_cache()
