"""Host logic of the tuner on a stand-in for the library: inputs whose radix passes do
not run, or share one launch, are no measure of a tile shape, however long the idle
launches take."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


class Lib:
    """The parts of cvetl that the tuner reads."""

    def __init__(self, passes, ms):
        self.passes, self.ms, self.shape, self.sorted = passes, ms, 0, 0

    cv_sort_workspace_size = None

    def lib(self):
        return self

    def _size(self, fn, *args):
        return 256

    def workspace(self, n, device=None):
        return "ws"

    def cv_tuning_set(self, name, value):
        self.shape = value

    def cv_tuning_get(self, name):
        return {"sort_shapes": 3, "sort_tile": 4096, "radix_bits": 8, "sort_shape": self.shape}[name]

    def cv_sort_records(self, rec, max_journeys=None, ws=None, sync=True):
        self.sorted += 1
        return None, None, dict(flags=8, key_bits=24, packed_pass=0)

    def cv_sort_passes(self, ws):
        return self.passes

    def cv_timing_reset(self):
        pass

    def cv_timing_enable(self, on):
        pass

    def cv_timing_read(self, family):
        return self.ms[self.shape if len(self.ms) > 1 else 0], 1


class Column:
    device = "cpu"

    def __init__(self, n):
        self.n = n

    def numel(self):
        return self.n


def _sweep(monkeypatch, n, lib):
    import torch
    import paper_2305_07454_amd as pkg
    from paper_2305_07454_amd import tune
    monkeypatch.setattr(pkg, "cvetl", lib, raising=False)
    monkeypatch.setitem(sys.modules, "paper_2305_07454_amd.cvetl", lib)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    return tune.sweep_sort_shapes({"journey_id": Column(n)}, None, reps=1, log=lambda m: None)


def test_sweep_ranks_shapes_by_passes_that_ran(monkeypatch):
    res = _sweep(monkeypatch, 3_000_000, Lib(3, [3.0, 1.0, 2.0]))
    assert [r["passes"] for r in res] == [3, 3, 3] and min(res, key=lambda r: r["sort_ms"])["sort_shape"] == 1


@pytest.mark.parametrize("n,passes", [(3_000_000, 0), (1 << 21, 3), (1_000_000, 3)])
def test_sweep_refuses_what_says_nothing(monkeypatch, n, passes):
    with pytest.raises(ValueError):
        _sweep(monkeypatch, n, Lib(passes, [3.0, 1.0, 2.0]))
