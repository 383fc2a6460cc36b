"""The grid's emit where a block's range has one chunk of 1 024 partial rows and where
it has more than one (4 096 blocks): a row per record, compared with numpy."""
import numpy as np
import pytest

from paper_2305_07454_amd import gen

from _parity import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4_096 * 1_024 - 1, 4_096 * 1_024 + 1, 9_000_001])
@pytest.mark.parametrize("share", [1, 7])
def test_grid_rows_of_many_ranges(n, share):
    """Every record has a journey and a cell of its own, or `share` records one cell."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    print(f"[grid ranges] n={n} share={share}", flush=True)
    rng = np.random.default_rng(n)
    cell = rng.permutation(n) // share
    spd = rng.integers(0, 40, n).astype(np.float32)
    cols = (np.arange(n), np.full(n, gen.T0_MS), np.full(n, 36.5), -94.5 + cell, spd)
    grid = gen.GridSpec(36.0, -95.0, 1.0, 1.0, 1, n, gen.T0_MS, 1000, 1)
    got, r = cvetl.cv_grid_aggregate(cvetl.to_device(cols), grid, capacity=n)
    count = np.bincount(cell)
    assert r["count"] == len(count)
    assert np.array_equal(host(got["key"]), np.arange(len(count)))
    assert np.array_equal(host(got["count"]), count) and np.array_equal(host(got["n_journeys"]), count)
    assert np.array_equal(host(got["sum_speed"]), np.bincount(cell, spd.astype(np.float64)))
