"""When a list of dense steps takes 64-row items (host rule): measured runs
with int8 couplings that are faster whole, or split, on either side of it."""
import host_harness


def test_measured_lists(tmp_path):
    # items, slots, fp4 couplings: split
    lists = [(24, 128, 1, 1), (128, 128, 1, 1), (255, 256, 1, 1), (256, 256, 1, 0), (96, 128, 0, 1), (128, 128, 0, 1),
             (132, 176, 0, 0), (144, 192, 0, 0), (192, 256, 0, 0), (198, 264, 0, 1), (255, 256, 0, 0), (256, 256, 0, 0),
             (288, 384, 0, 0)]
    body = "".join(f'std::printf("%d\\n", psa::dense_splits({i}, {s}, {f}) ? 1 : 0);' for i, s, f, _ in lists)
    out = host_harness.run(body + "return 0;", tmp_path)
    assert [int(x) for x in out] == [want for *_, want in lists]
