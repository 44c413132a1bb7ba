"""Splits of the read-outs (host rule): over measured sizes, the chosen split of
the lanes takes at most 1.1 times as long as the fastest that was measured."""
import host_harness
import pytest

# (p-bits, mean degree, trials): us of the local fields by (trial groups per lane, chunks side by side, lanes on the edges)
FIELDS = {
    (500, 400, 16): {(1, 4, 4): 23.7, (1, 4, 16): 9.2, (4, 1, 16): 15.9},
    (2000, 20, 16): {(1, 4, 4): 5.4, (1, 4, 16): 5.5, (4, 1, 4): 8.2},
    (3000, 400, 4): {(1, 4, 4): 26.5, (1, 1, 16): 10.2, (4, 1, 16): 16.9},
    (3000, 400, 16): {(1, 4, 4): 26.5, (1, 4, 16): 11.2, (4, 1, 16): 16.3},
    (1500, 120, 64): {(1, 4, 4): 12.7, (1, 4, 16): 7.6, (4, 4, 4): 17.1, (4, 4, 16): 10.7},
    (3000, 60, 64): {(1, 4, 4): 9.2, (1, 4, 16): 10.2, (4, 4, 4): 12.1, (4, 4, 16): 10.1},
    (3000, 400, 64): {(1, 4, 4): 44.8, (1, 4, 16): 39.1, (4, 4, 4): 39.1, (4, 4, 16): 19.0},
    (4800, 60, 128): {(1, 4, 4): 23.0, (4, 4, 4): 13.7, (4, 4, 16): 18.7},
    (3000, 200, 256): {(1, 4, 4): 63.7, (4, 4, 4): 28.8, (4, 4, 16): 33.3},
    (4800, 400, 128): {(1, 4, 4): 128.6, (4, 4, 4): 64.9, (4, 4, 16): 44.4},
    (20000, 40, 16): {(1, 4, 4): 10.0, (4, 1, 4): 12.7, (4, 1, 16): 12.5},
}
# us of energy and cut
ENERGY = {
    (1500, 60, 16): {(1, 1, 4): 12.4, (1, 1, 16): 13.2, (4, 1, 4): 16.9, (4, 1, 16): 18.4},
    (3000, 200, 16): {(1, 1, 16): 25.0, (4, 1, 4): 31.9, (4, 1, 16): 33.4},
    (3000, 400, 16): {(1, 1, 16): 74.7, (4, 1, 4): 53.9, (4, 1, 16): 54.4},
    (4800, 200, 16): {(1, 1, 16): 42.5, (4, 1, 4): 33.0, (4, 1, 16): 34.4},
    (3000, 400, 4): {(1, 1, 4): 40.4, (1, 1, 16): 36.8, (4, 1, 16): 56.4},
    (1500, 400, 64): {(1, 1, 16): 78.0, (4, 1, 4): 55.7, (4, 1, 16): 56.5},
    (3000, 200, 64): {(1, 1, 16): 53.1, (4, 1, 4): 37.1, (4, 1, 16): 35.9},
    (1500, 400, 128): {(1, 1, 16): 87.7, (4, 1, 16): 101.4},
    (3000, 400, 64): {(1, 1, 16): 91.2, (4, 1, 16): 98.2},
    (3000, 400, 100): {(1, 1, 16): 192.5, (4, 1, 16): 105.1},
    (4800, 400, 64): {(1, 1, 16): 208.7, (4, 1, 4): 138.7, (4, 1, 16): 103.3},
    (4800, 120, 256): {(1, 4, 4): 98.3, (4, 1, 16): 79.9, (4, 4, 4): 65.6, (4, 4, 16): 72.8},
    (4800, 200, 256): {(1, 4, 4): 158.6, (4, 1, 16): 118.9, (4, 4, 4): 137.2, (4, 4, 16): 148.7},
}


def chosen(sizes, call, tmp_path):
    body = ""
    for n, d, t in sizes:
        body += (f"{{ psa::EnergyJob e; e.n = {n}; e.t4 = e.trials = {(t + 3) // 4 * 4}; e.blocks = ({n} + 255) / 256; e.degree = {d};"
                 "psa::read_out_split(e.t4, e.degree, &e.cpl, &e.lpr);" + call +
                 'std::printf("%d %d %d\\n", e.quads, e.cpl, e.lpr); }')
    return [tuple(map(int, ln.split())) for ln in host_harness.run(body + "return 0;", tmp_path)]


@pytest.mark.parametrize("table,call", [(FIELDS, "psa::field_split(&e);"),
                                        (ENERGY, "psa::energy_split(&e, psa::energy_waves(e), psa::energy_batch_wgs(e), true);")])
def test_measured_splits(table, call, tmp_path):
    for (size, us), split in zip(table.items(), chosen(table, call, tmp_path)):
        assert split in us, (size, split)
        assert us[split] <= 1.1 * min(us.values()), (size, split)


def test_runs_of_a_batch_share_a_kind_of_lane(tmp_path):
    # a batched launch has one number of trial groups per lane for all its runs
    for waves in (100, 4095, 4096):
        quads = {q for q, _, _ in chosen(ENERGY, f"psa::energy_split(&e, {waves}, 100, false);", tmp_path)}
        assert quads == ({1} if waves < 4096 else {4})
