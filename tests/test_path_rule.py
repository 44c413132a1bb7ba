"""Path (row sweeps or dense product) that AUTO takes at sizes where either was
measured faster by a third or more, and with the coupling matrix still to be
built (host rule, no GPU)."""
import host_harness

# p-bits, degree, weights +-1, rule, trials, steps, dense matrix there: dense
CASES = [
    (4500, 6, 1, "period", 500, 30, 1, 0), (3000, 12, 1, "period", 500, 30, 1, 0), (3000, 24, 1, "period", 128, 30, 1, 0),
    (2000, 60, 1, "period", 64, 30, 1, 0), (3000, 180, 1, "period", 128, 30, 1, 1),
    (800, 12, 1, "tapsa", 2048, 30, 1, 0), (2000, 12, 1, "tapsa", 1000, 30, 1, 0), (1500, 24, 1, "tapsa", 700, 30, 1, 0),
    (3000, 12, 1, "tapsa", 700, 30, 1, 0), (2000, 24, 1, "spsa", 2048, 30, 1, 0), (2000, 180, 0, "tapsa", 32, 30, 1, 1),
    (4500, 6, 1, "spsa", 256, 30, 1, 0),
    (800, 180, 0, "psa", 64, 30, 1, 1), (2000, 180, 0, "psa0", 32, 30, 1, 1), (1500, 60, 0, "psa0", 128, 30, 1, 0),
    (3000, 180, 1, "psa", 128, 30, 1, 1), (3000, 24, 1, "psa", 128, 30, 1, 0), (4500, 6, 1, "psa", 1000, 30, 1, 0),
    (800, 24, 1, "psa", 500, 30, 1, 0), (300, 6, 1, "psa0", 64, 1000, 1, 0),
    # 2.7 ms of encoding against 10 or 2,000 steps
    (5000, 100, 1, "psa0", 8, 10, 0, 0), (5000, 100, 1, "psa0", 8, 10, 1, 1), (5000, 100, 1, "psa0", 8, 2000, 0, 1),
    (4000, 80, 0, "psa0", 32, 10, 0, 0)]


def test_measured_runs(tmp_path):
    body = """
    struct C { int n, deg, unit, rule, trials, steps, built; };
    const C cases[] = {%s};
    static char some[16];
    for (const C &c : cases) {
        psa_graph gr;
        psa::DevGraph &g = gr.dev;
        gr.info.n = g.n = c.n;
        g.n4 = (c.n + 3) / 4 * 4;
        g.nnz = static_cast<int64_t>(c.n) * c.deg;
        g.max_degree = c.deg * 3 / 2 + 4;
        g.pk32 = reinterpret_cast<const uint32_t *>(some);
        g.ux16 = c.unit ? reinterpret_cast<const uint16_t *>(some) : nullptr;
        g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
        g.e4_mode = c.unit ? 0 : 1;
        gr.val_host = c.unit ? std::vector<int32_t>{1, -1} : std::vector<int32_t>{1, -7};
        gr.d_dense = c.built ? some : nullptr;
        psa::DevRun run;
        run.trials = c.trials;
        run.t4 = (c.trials + 3) / 4 * 4;
        run.steps = c.steps;
        if (c.rule == 2) run.xs = reinterpret_cast<float *>(some);
        if (c.rule == 3) { run.ring = reinterpret_cast<int32_t *>(some); run.alpha = 4; }
        if (c.rule == 4) run.t_res = 10;
        psa::AnnealPlan p;
        if (!psa::plan_anneal(g, run, 0, 0, 0, 163840, 256, &p, nullptr)) return 1;
        std::printf("%%d\\n", psa::prefer_dense(&gr, run, p, c.rule == 0) ? 1 : 0);
    }
    return 0;""" % ", ".join("{%d, %d, %d, %d, %d, %d, %d}" % (n, d, u, ["psa0", "psa", "spsa", "tapsa", "period"].index(r), t, s, b)
                             for n, d, u, r, t, s, b, _ in CASES)
    out = host_harness.run(body, tmp_path)
    wrong = [(c, int(o)) for c, o in zip(CASES, out) if c[-1] != int(o)]
    assert len(out) == len(CASES) and not wrong, wrong
