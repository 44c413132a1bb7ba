"""Lanes per task of short rows of unit weights once the trials outnumber the
compute units, at sizes where two or four were measured faster (host rule, no GPU)."""
import test_lanes_per_task_rule as rule

# p-bits, degree, rows all of it, weights +-1, rule, trials: trials per workgroup, lanes per task
CASES = [(1023, 4, 1, 1, "psa", 299, 1, 2), (600, 6, 0, 1, "spsa", 258, 1, 2), (1000, 6, 0, 1, "tapsa", 284, 1, 2), (1000, 6, 0, 1, "psa", 256, 1, 4),
         (250, 6, 0, 1, "psa", 300, 1, 4), (364, 4, 0, 1, "spsa", 330, 1, 2)]


def test_measured_runs(tmp_path, monkeypatch):
    monkeypatch.setattr(rule, "CASES", CASES)
    rule.test_measured_runs(tmp_path)
