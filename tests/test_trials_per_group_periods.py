"""Trials per workgroup under period timing around the lines by entries and
weights, at sizes where one or four were measured faster (host rule, no GPU)."""
import test_trials_per_group_rule as rule

# p-bits, degree, weights +-1, rule, trials: trials per workgroup
CASES = [(n, d, unit, "period", t, want) for n, d, unit, t, want in [
    (300, 72, 1, 760, 1), (300, 72, 1, 780, 4), (500, 48, 1, 600, 1), (500, 48, 1, 780, 4), (1000, 24, 1, 760, 1), (250, 120, 1, 520, 1),
    (250, 120, 1, 780, 4), (1000, 40, 1, 520, 4), (600, 100, 1, 760, 4), (1000, 12, 0, 1000, 1), (1000, 19, 0, 1000, 1),
    (300, 60, 0, 1000, 1), (200, 80, 0, 780, 1), (500, 48, 0, 1000, 1), (250, 120, 0, 1000, 1), (800, 60, 0, 780, 4), (500, 150, 0, 780, 4),
    (1200, 12, 1, 760, 1), (1100, 24, 1, 520, 4), (1200, 12, 0, 760, 1), (1500, 24, 0, 760, 1), (1500, 24, 0, 780, 4), (2000, 24, 0, 520, 4)]]


def test_measured_runs(tmp_path, monkeypatch):
    monkeypatch.setattr(rule, "CASES", CASES)
    rule.test_measured_runs(tmp_path)
