"""The autotuner's calls on a rasterizer (a stand-in without a GPU): every candidate is timed on a
workspace that holds a binning, which a count invalidates."""
import torch

from paper_2605_31419_amd import autotune


class _Event:
    def __init__(self, enable_timing):
        pass

    def record(self):
        pass

    def elapsed_time(self, other):
        return 1.0


class _Rast:
    n_views = 2

    def __init__(self):
        self.binned, self.trained = False, []

    def bin_and_sort(self, poses):
        self.binned = True

    def count(self, poses):
        self.binned = False
        return 100

    def grad_buffers(self):
        return None, None, None, None

    def train_l1(self, poses, target_color, target_depth, loss, out, schedule):
        assert self.binned, "a candidate was timed without a binning"
        loss.fill_(1.0)
        self.trained.append(schedule)


def test_candidates_are_timed_on_a_binned_workspace(monkeypatch):
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda n, device=None: zeros(n))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    rast = _Rast()
    best, times = autotune.tune(rast, None, None, None, reps=2)
    assert set(rast.trained) == set(autotune.CANDIDATES) and best in autotune.CANDIDATES
    assert len(times) == len(autotune.CANDIDATES)
