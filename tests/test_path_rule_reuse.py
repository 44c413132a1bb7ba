"""Path of runs whose graph has no dense matrix yet: kept jobs take it at once,
runs that are over after their schedule once they make up for it (host rule)."""
import host_harness
import pytest

BODY = """
    static char some[16];
    psa_graph gr;
    psa::DevGraph &g = gr.dev;
    gr.info.n = g.n = g.n4 = 5000;
    g.nnz = 500000;
    g.max_degree = 150;
    g.pk32 = g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
    g.ux16 = reinterpret_cast<const uint16_t *>(some);
    g.e4_mode = 0;
    gr.val_host = {1, -1};
    psa::DevRun run;
    run.trials = run.t4 = 8;
    run.steps = 10;
    psa::AnnealPlan p;
    if (!psa::plan_anneal(g, run, 0, 0, 0, 163840, 256, &p, nullptr)) return 1;
"""


def test_kept_jobs(tmp_path):
    out = host_harness.run(BODY + 'std::printf("%d %g\\n", psa::prefer_dense(&gr, run, p, true, false) ? 1 : 0, gr.dense_gain); return 0;', tmp_path)
    assert out == ["1 0"]


@pytest.mark.parametrize("steps,first", [(10, (2, 40)), (2000, (0, 0))])
def test_repeated_single_runs(steps, first, tmp_path):
    body = BODY + f"run.steps = {steps};" + 'for (int k = 0; k < 50; ++k) std::printf("%d\\n", psa::prefer_dense(&gr, run, p, true, true) ? 1 : 0); return 0;'
    out = [int(x) for x in host_harness.run(body, tmp_path)]
    at = out.index(1)  # rows before it, the dense matrix from then on
    assert first[0] <= at <= first[1] and out == [0] * at + [1] * (50 - at)
