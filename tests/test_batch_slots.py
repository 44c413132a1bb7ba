"""Work lists of batches whose workgroups have a compute unit each: no XCD gets
more of them than it has units (host rule, no GPU)."""
import host_harness
import pytest


@pytest.mark.parametrize("jobs,items,block", [(12, 10, 512), (12, 10, 256), (40, 6, 512), (25, 10, 256), (3, 80, 512)])
def test_one_workgroup_to_a_unit(jobs, items, block, tmp_path):
    out = host_harness.run(f"""
    std::vector<int32_t> items({jobs}, {items});
    std::vector<double> cost;
    for (int j = 0; j < {jobs}; ++j) cost.push_back(2.0 - 0.01 * j);
    std::vector<int2> work;
    psa::build_work_list(items, cost, psa::batch_slots({jobs * items}, 256, {block}), &work);
    int n[8] = {{}};
    for (size_t b = 0; b < work.size(); ++b) n[b % 8] += work[b].x >= 0;
    for (int x : n) std::printf("%d\\n", x);
    return 0;""", tmp_path)
    n = [int(x) for x in out]
    assert sum(n) == jobs * items and max(n) <= 32


def test_shared_units(tmp_path):
    out = host_harness.run('std::printf("%d %d %d\\n", psa::batch_slots(256, 256, 512), psa::batch_slots(257, 256, 512), psa::batch_slots(257, 256, 1024)); return 0;', tmp_path)
    assert out == ["32 64 32"]
