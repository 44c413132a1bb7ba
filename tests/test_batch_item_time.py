"""Modelled step of one workgroup of a batch against steps measured alone: streamed
SpSA inputs of small graphs stay in L2 (host rule, no GPU)."""
import host_harness

# p-bits, degree, us measured alone with weights, one trial per workgroup, SpSA
RUNS = [(1786, 4, 1.87), (2000, 6, 2.35), (1500, 12, 2.87)]


def test_streamed_inputs(tmp_path):
    body = "static char some[16];"
    for n, d, _ in RUNS:
        body += f"""{{
        psa::DevGraph g;
        g.n = {n};
        g.n4 = ({n} + 3) / 4 * 4;
        g.nnz = int64_t{{{n}}} * {d};
        g.max_degree = {d};
        g.pk32 = g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
        g.e4_mode = 1;
        psa::DevRun run;
        run.trials = run.t4 = 140;
        run.xs = reinterpret_cast<float *>(some);
        psa::AnnealPlan p;
        int32_t variant = 0;
        if (!psa::plan_batch_item(g, run, 1, 1, 163840, &p, &variant, nullptr) || !p.ell) return 1;
        std::printf("%g\\n", 1e6 * psa::batch_item_time(g, run, p).alone);
        }}"""
    out = [float(x) for x in host_harness.run(body + "return 0;", tmp_path)]
    for (n, d, us), model in zip(RUNS, out):
        assert us / 1.5 <= model <= 1.5 * us, (n, d, us, model)
