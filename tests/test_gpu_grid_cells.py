"""Cells of coordinates on and next to a cell's edge (one and two ulps to either
side), next to zero, infinite and NaN, with times near and far (beyond 2^30 ms)
on both sides of the grid's start: the grid's quotients by reciprocal against
the oracle's divisions, in the plain, direction and batched forms, with tiles
and waves cut everywhere (51 records to a journey, odd speeds among them).
Every column equals the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2305_07454_amd import gen

from _parity import check_groups, host

pytestmark = pytest.mark.gpu

SPECS = {
    "hundredths": (36.0, -95.0, 0.01, 0.01, 300, 300),
    "thirds": (-10.0 / 3, 7.7, 1.0 / 3, 0.1, 21, 77),
    "origin": (0.0, 0.0, 1e-3, 7e-4, 1000, 900),
    "wide": (-90.0, -180.0, 45.0, 0.3, 5, 1200),
}


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    oracle.lib()
    return cvetl


def _near_edges(rng, x0, d, cells, n):
    x = x0 + rng.integers(-1, cells + 2, n) * d
    for _ in range(2):
        step = rng.integers(-1, 2, n)
        x = np.where(step < 0, np.nextafter(x, -np.inf), np.where(step > 0, np.nextafter(x, np.inf), x))
    x = np.where(rng.random(n) < 0.3, x0 + rng.uniform(-0.5, cells + 0.5, n) * d, x)
    odd = rng.integers(0, 200, n)
    special = [np.nan, np.inf, -np.inf, 5e-324, -5e-324, 1e-300, -1e-300, 0.0, -0.0, 1e300, -1e300]
    return np.where(odd < len(special), np.array(special)[np.minimum(odd, len(special) - 1)], x)


@pytest.mark.parametrize("name", sorted(SPECS))
@pytest.mark.parametrize("bin_ms,n_t", [(60_000, 50), (900_000, 30_000), ((1 << 30) + 7, 9)])
def test_cells_at_edges(cv, name, bin_ms, n_t):
    import torch
    print(f"[grid cells] {name} bin {bin_ms}", flush=True)
    lat0, lon0, dlat, dlon, n_lat, n_lon = SPECS[name]
    spec = gen.GridSpec(lat0, lon0, dlat, dlon, n_lat, n_lon, gen.T0_MS, bin_ms, n_t)
    rng = np.random.default_rng(11)
    n = 40_003
    jid = np.arange(n) // 51
    off = rng.integers(-2, 40, n) * bin_ms + rng.integers(-1, 2, n)
    off = np.where(rng.random(n) < 0.05, rng.integers(-(1 << 40), 1 << 40, n), off)
    ts = gen.T0_MS + off
    order = np.lexsort((ts, jid))
    ts = ts[order]
    lat, lon = _near_edges(rng, lat0, dlat, n_lat, n), _near_edges(rng, lon0, dlon, n_lon, n)
    spd = rng.integers(0, 40, n).astype(np.float32)
    spd[rng.integers(0, n, 40)] = np.float32(1e-30)  # outside the short sum format
    hd = rng.integers(0, 360, n).astype(np.float32)
    flags = torch.from_numpy((np.diff(jid, prepend=-1) != 0).astype(np.uint8)).cuda()
    cols = (jid, ts, lat, lon, spd)
    exp, n_out = oracle.grid(*cols, spec)
    d = cv.to_device(cols)
    for fl in (None, flags):
        got, r = cv.cv_grid_aggregate(d, spec, flags=fl)
        check_groups(got, r["n_out_of_grid"], exp, n_out)
    exp, n_out = oracle.grid_dir(*cols, spec, 8, 22.5, heading=hd)
    got, r = cv.cv_grid_aggregate_dir(d, spec, 8, 22.5, heading=torch.from_numpy(hd).cuda())
    check_groups(got, r["n_out_of_grid"], exp, n_out)
    # shards that end inside a tile, inside a wave and on a row's edge, two of
    # them empty; journeys cross them
    sizes = [1, 63, 0, 449, 2048, 5000, 0, 64, 20_000, n - 27_625]
    bp, _ = cv.cv_batch_run(d, sizes, spec)
    go, a = host(bp.group_offsets), 0
    for s, m in enumerate(sizes):
        if m:
            srt = [host(bp.sorted[k][a:a + m]) for k in ("journey_id", "ts_ms", "lat_deg", "lon_deg", "speed_mps")]
            exp, n_out = oracle.grid(*srt, spec)
            check_groups({k: v[int(go[s]):int(go[s + 1])] for k, v in bp.groups.items()},
                         int(host(bp.shard_n_out)[s]), exp, n_out)
        a += m
