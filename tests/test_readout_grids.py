"""Grids of the read-outs stay within what a launch holds -- fewer than 2^32
threads along x, at most 65,535 workgroups along y -- for every count that a
read-out takes, and cover it."""
import host_harness


def test_wide_grids(tmp_path):
    out = host_harness.run("""
    for (int64_t count : {int64_t{1}, int64_t{79}, int64_t{4096}, (int64_t{1} << 20) - 1, int64_t{1} << 20, (int64_t{1} << 20) + 1,
                          int64_t{1} << 22, (int64_t{1} << 22) + 1, int64_t{1} << 26, (int64_t{1} << 26) + 12345, (int64_t{1} << 31) - 1}) {
        const dim3 g = psa::wide_grid(count);
        std::printf("%lld %u %u %u\\n", static_cast<long long>(count), g.x, g.y, g.z);
    }
    return 0;""", tmp_path)
    assert len(out) == 11
    for line in out:
        count, x, y, z = map(int, line.split())
        assert z == 1 and 1 <= y <= 65535 and x >= 1, line
        assert x * 1024 < 1 << 32, line
        assert count <= x * y < count + x, line
        assert count > 1 << 20 or y == 1, line
