"""The sweep over spin bits loads a fixed count of entries of every row: each
index it forms lies inside the graph's bit rows, also for wavefronts whose rows
are all empty (isolated p-bits sort last)."""
import host_harness
import pytest


@pytest.mark.parametrize("n,edges", [(2, 1), (65, 1), (257, 100), (1025, 512), (1100, 3), (2048, 600), (2049, 1024), (4032, 5)])
def test_every_entry_lies_inside(tmp_path, n, edges):
    out = host_harness.run(f"""
    psa::HostGraph g;
    std::vector<int32_t> u, v, w;
    for (int32_t e = 0; e < {edges}; ++e) {{ u.push_back(2 * e % ({n} - 1)); v.push_back(2 * e % ({n} - 1) + 1); w.push_back(2); }}
    if (psa::host_graph_from_edges({n}, {edges}, u.data(), v.data(), w.data(), nullptr, 0, &g) != PSA_OK) return 1;
    int32_t most = -1, least = 0;
    for (size_t k = 0; k + 1 < g.bofs.size(); ++k)
        for (int32_t e = 0; e < 48; ++e) {{
            const int32_t at = psa::bit_row_entry(g.bofs[k], g.bofs[k + 1] - g.bofs[k], e);
            most = std::max(most, at);
            least = std::min(least, at);
        }}
    std::printf("%zu %d %d %d\\n", g.bofs.size() - 1, least, most, g.bofs.back());
    return 0;""", tmp_path)
    waves, least, most, entries = map(int, out[-1].split())
    assert waves == (n + 63) // 64
    assert least >= 0 and 0 <= most < entries
