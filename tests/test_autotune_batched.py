"""Bookkeeping of the batched tuner on a plan that only counts (no device work):
the kernels do not depend on the launch shape, so a candidate is timed once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2607_17978_amd import autotune   # noqa: E402


class CountingPlan:
    calls = []

    def __init__(self, n_max, spline_order, max_spacing, **_):
        self.key = (spline_order, max_spacing)

    def solve_batched(self, **_):
        self.calls.append(self.key)
        return torch.zeros(3), torch.ones(1, 2), torch.ones(3, 3), [], 0

    def batched_config(self, threads, wg_per_cu):
        pass

    def close(self):
        pass


@pytest.mark.parametrize("shapes", [(1,), (1, 2), (4, 1, 2)])
def test_candidate_is_timed_once(monkeypatch, shapes):
    monkeypatch.setattr(autotune.qeq, "Plan", CountingPlan)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    CountingPlan.calls = []
    out = autotune.tune_batched({"offsets": np.array([0, 3])}, candidates=((6, 0.8), (8, 1.0)), wg_per_cu=shapes,
                                reps=5)
    # one solve for the accuracy, one to warm up, five timed
    assert CountingPlan.calls == [autotune.REFERENCE] + [(6, 0.8)] * 7 + [(8, 1.0)] * 7
    for row in out["candidates"]:
        assert len({row[f"ms_wg{wg}"] for wg in shapes}) == 1
    assert out["best"]["wg_per_cu"] == shapes[0]
