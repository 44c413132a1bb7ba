"""Trials per workgroup that the planner takes for a run stepped alone, at
sizes where one or four were measured faster (host rule, no GPU)."""
import host_harness

# p-bits, degree, weights +-1, rule, trials: trials per workgroup
CASES = [
    # resident lanes with cached rows
    (600, 6, 1, "psa", 520, 1), (600, 6, 1, "psa", 768, 1), (600, 6, 1, "psa", 800, 4), (1200, 6, 1, "spsa", 760, 1),
    (1500, 6, 1, "spsa", 780, 4), (1200, 6, 1, "psa", 760, 1), (2000, 6, 1, "psa", 760, 4), (2000, 6, 1, "spsa", 760, 1), (800, 12, 1, "tapsa", 1000, 1), (2000, 6, 1, "tapsa", 1000, 1), (2000, 6, 1, "tapsa", 1030, 4),
    (800, 24, 1, "tapsa", 700, 1),
    # rows weighted, or past the cached slots
    (1000, 6, 0, "psa", 520, 4), (2000, 24, 1, "psa", 520, 4), (2000, 6, 0, "tapsa", 600, 4), (2000, 24, 1, "tapsa", 700, 4),
    # streaming sweep
    (4000, 6, 1, "psa", 512, 1), (4000, 6, 1, "psa", 600, 4), (4000, 12, 0, "psa", 520, 4), (8000, 6, 1, "tapsa", 520, 4),
    # period classes
    (600, 6, 1, "period", 1000, 1), (800, 12, 1, "period", 760, 1), (1000, 6, 0, "period", 760, 1), (1500, 6, 1, "period", 760, 1),
    (2000, 6, 1, "period", 760, 1), (2000, 6, 1, "period", 780, 4), (2000, 24, 1, "period", 520, 4), (800, 24, 1, "period", 700, 1),
    (4000, 6, 1, "period", 500, 1), (4000, 6, 1, "period", 1000, 4), (250, 6, 1, "period", 1030, 4), (300, 6, 1, "period", 1000, 1),
    (300, 60, 1, "period", 700, 1), (800, 60, 1, "period", 700, 4)]


def test_measured_runs(tmp_path):
    body = """
    struct C { int n, deg, unit, rule, trials; };
    const C cases[] = {%s};
    static char some[16];
    for (const C &c : cases) {
        psa::DevGraph g;
        g.n = c.n;
        g.n4 = (c.n + 3) / 4 * 4;
        g.nnz = static_cast<int64_t>(c.n) * c.deg;
        g.max_degree = c.deg * 3 / 2 + 4;
        g.pk32 = reinterpret_cast<const uint32_t *>(some);
        g.ux16 = c.unit ? reinterpret_cast<const uint16_t *>(some) : nullptr;
        g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
        g.e4_mode = c.unit ? 0 : 1;
        psa::DevRun run;
        run.trials = c.trials;
        run.t4 = (c.trials + 3) / 4 * 4;
        if (c.rule == 1) run.xs = reinterpret_cast<float *>(some);
        if (c.rule == 2) { run.ring = reinterpret_cast<int32_t *>(some); run.alpha = 4; }
        if (c.rule == 3) run.t_res = 10;
        psa::AnnealPlan p;
        if (!psa::plan_anneal(g, run, 0, 0, 0, 163840, 256, &p, nullptr)) return 1;
        std::printf("%%d\\n", p.tpw);
    }
    return 0;""" % ", ".join("{%d, %d, %d, %d, %d}" % (n, d, u, ["psa", "spsa", "tapsa", "period"].index(r), t) for n, d, u, r, t, _ in CASES)
    out = host_harness.run(body, tmp_path)
    wrong = [(c, int(o)) for c, o in zip(CASES, out) if c[-1] != int(o)]
    assert len(out) == len(CASES) and not wrong, wrong
