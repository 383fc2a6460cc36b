"""The bench's choice of a roofline: by what the sort says of its passes, not by how
long their launches take."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


class Lib:
    """The parts of cvetl that the roofline reads; every pass took `ms`."""

    def __init__(self, ms):
        self.ms = ms

    def cv_tuning_get(self, name):
        return {"sort_tile": 4096, "radix_bits": 8}[name]

    def cv_timing_read(self, family):
        return self.ms, 1


@pytest.mark.parametrize("ms", [1e-4, 0.005, 10.0])
def test_roofline_follows_what_the_sort_says(ms):
    """1 M records, 16 MB a pass: at 5 us an idle launch is below the card's peak and at 0.1 us beyond it."""
    rs = dict(flags=8, key_bits=24, packed_pass=0)
    roof, total = bench.radix_roofline(Lib(ms), 1_000_000, rs, sorts=False)
    assert roof is None and total == pytest.approx(3 * ms)
    roof, total = bench.radix_roofline(Lib(ms), 1_000_000, rs, sorts=True)
    assert roof["launches"] == 3 and total == pytest.approx(3 * ms)
