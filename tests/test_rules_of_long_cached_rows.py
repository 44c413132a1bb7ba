"""Path and trials per workgroup of runs with a row of unit weights per lane that
take two or three rounds of the compute units, where they were measured (host
rules, no GPU)."""
import test_path_rule
import test_trials_per_group_rule

# us per step on the rows and of the dense step: 4.4 and 5.3, 5.0 and 6.8, 5.9 and 7.0, 3.1 and 5.3
PATHS = [(950, 45, 1, "psa", 284, 30, 1, 0), (950, 29, 1, "psa", 520, 30, 1, 0), (800, 47, 1, "psa", 520, 30, 1, 0), (915, 26, 1, "psa", 284, 30, 1, 0)]
# us per step with one and four trials: 5.9 and 7.0, 5.3 and 7.1, 9.6 and 8.2
TRIALS = [(800, 47, 1, "psa", 520, 1), (700, 45, 1, "psa", 520, 1), (950, 63, 1, "psa", 520, 4)]


def test_paths(tmp_path, monkeypatch):
    monkeypatch.setattr(test_path_rule, "CASES", PATHS)
    test_path_rule.test_measured_runs(tmp_path)


def test_trials(tmp_path, monkeypatch):
    monkeypatch.setattr(test_trials_per_group_rule, "CASES", TRIALS)
    test_trials_per_group_rule.test_measured_runs(tmp_path)
