"""Which runs of a batch take four trials per workgroup, at mixes where all with
one, or all with four, were measured faster (host rule, no GPU)."""
import random

import host_harness
import pytest


def _choose(tmp_path, runs):
    """runs: (n, mean degree, weights +-1, rule, trials); returns the choice of each."""
    body = """
    struct C { int n, deg, unit, rule, trials; };
    const std::vector<C> runs = {%s};
    static char some[16];
    psa_ctx ctx;
    ctx.num_cu = 256;
    ctx.max_lds = 163840;
    std::vector<psa_graph> graphs(runs.size());
    std::vector<psa_job> jobs(runs.size());
    std::vector<psa_job *> ptr;
    std::vector<int32_t> idx, t_end;
    for (size_t x = 0; x < runs.size(); ++x) {
        const C &c = runs[x];
        psa::DevGraph &g = graphs[x].dev;
        g.n = c.n;
        g.n4 = (c.n + 3) / 4 * 4;
        g.nnz = static_cast<int64_t>(c.n) * c.deg;
        g.max_degree = c.deg * 3 / 2 + 4;
        g.pk32 = reinterpret_cast<const uint32_t *>(some);
        g.ux16 = c.unit ? reinterpret_cast<const uint16_t *>(some) : nullptr;
        g.e1 = g.e4 = reinterpret_cast<const uint32_t *>(some);
        g.e1j = c.unit ? nullptr : g.e1;
        g.e4_mode = c.unit ? 0 : 1;
        psa_job &j = jobs[x];
        j.g = &graphs[x];
        j.auto_tpw = true;
        j.run.trials = c.trials;
        j.run.t4 = (c.trials + 3) / 4 * 4;
        j.run.pps = reinterpret_cast<const uint32_t *>(some);
        if (c.rule == 1) j.run.xs = reinterpret_cast<float *>(some);
        if (c.rule == 2) { j.run.ring = reinterpret_cast<int32_t *>(some); j.run.alpha = 4; }
        if (c.rule == 3) j.run.t_res = 10;
        if (!psa::plan_anneal(g, j.run, 1, 0, 0, ctx.max_lds, 256, &j.plan, nullptr)) return 1;
        ptr.push_back(&j);
        idx.push_back(static_cast<int32_t>(x));
        t_end.push_back(100);
    }
    for (char f : psa::choose_four_trials(&ctx, ptr.data(), idx, t_end)) std::printf("%%d\\n", f);
    std::fflush(stdout);
    _Exit(0);""" % ", ".join("{%d, %d, %d, %d, %d}" % (n, d, u, ["psa", "spsa", "tapsa", "period"].index(r), t) for n, d, u, r, t in runs)
    return [int(x) for x in host_harness.run(body, tmp_path)]


def _mix(seed, count, n, deg, unit, rule, trials):
    rng = random.Random(seed)
    return [(rng.randint(*n), rng.randint(*deg), unit, rule, rng.randint(*trials)) for _ in range(count)]


@pytest.mark.parametrize("runs,want", [
    # few workgroups for the chip, all alike: one (six of 3,000 p-bits 4.9 and 5.6 us per step)
    ([(3000, 6, 1, "psa", 8)] * 6, 0), ([(3000, 6, 0, "spsa", 8)] * 6, 0), ([(3000, 6, 1, "psa", 64)] * 12, 1),
    # small graphs, input stages
    (_mix(1, 40, (60, 500), (4, 8), 1, "tapsa", (8, 64)), 0), (_mix(1, 40, (60, 500), (4, 8), 1, "spsa", (8, 64)), 0),
    (_mix(1, 20, (60, 500), (4, 8), 1, "psa", (100, 500)), 1), (_mix(1, 20, (60, 500), (4, 8), 1, "spsa", (100, 500)), 1),
    (_mix(1, 20, (300, 1000), (20, 40), 0, "spsa", (32, 128)), 1), (_mix(2, 8, (800, 2000), (4, 8), 0, "spsa", (200, 600)), 1),
    # large graphs
    (_mix(3, 16, (5000, 20000), (10, 50), 1, "psa", (100, 200)), 1), (_mix(4, 12, (2069, 4044), (4, 8), 1, "psa", (16, 16)), 0),
    (_mix(4, 12, (2069, 4044), (4, 8), 1, "psa", (64, 64)), 1)])
def test_measured_mixes(tmp_path, runs, want):
    four = _choose(tmp_path, runs)
    assert len(four) == len(runs)
    assert sum(four) / len(four) > 0.7 if want else sum(four) == 0, four
