"""Lanes per task and trials per workgroup of weighted graphs whose tasks have two
lanes each, at sizes where one form was measured faster (host rule, no GPU)."""
import host_harness

# p-bits, degree, rows all of it, weights +-1, rule, trials: trials per workgroup, lanes per task
CASES = [(1786, 4, 1, 0, "psa", 140, 1, 1), (1786, 4, 1, 0, "psa", 400, 1, 1), (1786, 4, 1, 0, "spsa", 233, 1, 1), (1100, 6, 0, 0, "psa", 140, 1, 1),
         (1100, 6, 0, 0, "spsa", 140, 1, 2), (1100, 6, 0, 0, "spsa", 400, 1, 1), (1100, 24, 0, 0, "spsa", 140, 1, 1), (2000, 24, 0, 0, "psa", 400, 1, 1),
         (2000, 6, 0, 0, "psa", 520, 4, 1), (2000, 6, 0, 0, "tapsa", 140, 1, 2), (1786, 4, 1, 0, "period", 140, 1, 2), (1786, 4, 1, 1, "psa", 140, 1, 2),
         (1000, 6, 0, 0, "psa", 140, 1, 4)]


def test_measured_runs(tmp_path):
    body = "static char some[16];"
    for n, d, uniform, unit, rule, t, *_ in CASES:
        body += f"""{{
        psa::DevGraph g;
        g.n = {n};
        g.n4 = ({n} + 3) / 4 * 4;
        g.nnz = int64_t{{{n}}} * {d};
        g.max_degree = {d if uniform else d * 3 // 2 + 4};
        g.pk32 = g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
        g.ux16 = {unit} ? reinterpret_cast<const uint16_t *>(some) : nullptr;
        g.e4_mode = {0 if unit else 1};
        psa::DevRun run;
        run.trials = {t};
        run.t4 = ({t} + 3) / 4 * 4;
        if ({int(rule == "spsa")}) run.xs = reinterpret_cast<float *>(some);
        if ({int(rule == "tapsa")}) {{ run.ring = reinterpret_cast<int32_t *>(some); run.alpha = 4; }}
        if ({int(rule == "period")}) run.t_res = 10;
        psa::AnnealPlan p;
        if (!psa::plan_anneal(g, run, 0, 0, 0, 163840, 256, &p, nullptr)) return 1;
        std::printf("%d %d\\n", p.tpw, p.lpt);
        }}"""
    out = [tuple(map(int, ln.split())) for ln in host_harness.run(body + "return 0;", tmp_path)]
    assert out == [c[6:] for c in CASES]
