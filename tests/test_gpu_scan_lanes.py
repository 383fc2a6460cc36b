"""Sums and segmented scans across the lanes of a wave, with segment starts at
every lane position (rows of 16 lanes, halves of 32, none at all): journeys of
one record up to several waves in the summary, runs of one to many records in
the grid.  Whole numbers, so every sum is exact; compared with numpy."""
import numpy as np
import pytest

from paper_2305_07454_amd import gen

from _parity import host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    return cvetl


@pytest.mark.parametrize("pattern", ["1", "15", "16", "17", "31", "32", "33", "63", "64", "65", "random"])
def test_segments_at_every_lane(cv, pattern):
    import torch
    print(f"[scan lanes] {pattern}", flush=True)
    n = 9_000
    rng = np.random.default_rng(7)
    head = rng.random(n) < 0.1 if pattern == "random" else np.arange(n) % int(pattern) == 0
    head[0] = True
    jid = np.cumsum(head)
    spd = rng.integers(-900, 900, n).astype(np.float32)
    lat, lon = rng.uniform(36, 40, n), rng.uniform(-95, -90, n)
    step = rng.integers(0, 1000, n).astype(np.float64)
    flags = np.where(head, 1, 6).astype(np.uint8)
    srt = cv.to_device((jid, gen.T0_MS + np.arange(n), lat, lon, spd))
    feat = {k: torch.from_numpy(v).cuda() for k, v in
            dict(step_m=step, speed_mps=step / 7.0, flags=flags).items()}
    at = np.nonzero(head)[0]
    got, r = cv.cv_journey_summary(srt, feat, capacity=len(at))
    assert r["count"] == len(at)
    spd64 = spd.astype(np.float64)
    for k, e in (("n_points", np.diff(np.append(at, n))), ("sum_speed", np.add.reduceat(spd64, at)),
                 ("distance_m", np.add.reduceat(step, at)), ("max_speed", np.maximum.reduceat(spd, at)),
                 ("lat_min", np.minimum.reduceat(lat, at)), ("lon_max", np.maximum.reduceat(lon, at)),
                 ("n_dt_zero", np.add.reduceat((flags >> 1 & 1).astype(np.int64), at))):
        assert np.array_equal(host(got[k]).astype(e.dtype), e), k
    # every journey in a cell of its own: the groups are the journeys
    grid = gen.GridSpec(36.0, -95.0, 4.1, 1.0, 1, n + 2, gen.T0_MS, 10 ** 9, 1)
    cell = cv.to_device((jid, gen.T0_MS + np.arange(n), lat, -94.5 + jid, spd))
    for fl in (None, feat["flags"]):
        g, r = cv.cv_grid_aggregate(cell, grid, flags=fl)
        assert r["count"] == len(at)
        for k, e in (("key", jid[at]), ("count", np.diff(np.append(at, n))), ("sum_speed", np.add.reduceat(spd64, at)),
                     ("min_speed", np.minimum.reduceat(spd, at)), ("max_speed", np.maximum.reduceat(spd, at))):
            assert np.array_equal(host(g[k]).astype(e.dtype), e), k
