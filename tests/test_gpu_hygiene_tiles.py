"""Record hygiene at the edges of its tiles (8 192 records, wave rows of 64):
runs of one (journey, time stamp) and their copies across lanes, waves and
tiles, NaN and signed zeros compared by bits, perm given or not.  Against the
oracle's definitions, exactly."""
import numpy as np
import pytest

import oracle
from paper_2305_07454_amd import gen

from _parity import assert_exact, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    oracle.lib()
    return cvetl


def _sorted(n, seed):
    rng = np.random.default_rng(seed)
    jid = np.cumsum(rng.random(n) < 1 / 900) - 3
    step = np.where(rng.random(n) < 0.6, 0, rng.integers(1, 90_000, n))  # runs of one time stamp, gaps
    ts = gen.T0_MS + np.cumsum(step)
    lat = rng.choice([38.0, 38.5, -0.0, 0.0, np.nan], n)
    lon = rng.choice([-92.0, -92.5], n)
    spd = rng.choice(np.array([0.0, -0.0, 7.0], np.float32), n)
    if n > 200:  # one run of a single (journey, time stamp) across waves
        a = n // 2
        jid[a:a + 150] = jid[a]
        jid[a + 150:] = np.maximum(jid[a + 150:], jid[a])
        ts[a:a + 150] = ts[a]
    return jid.astype(np.int64), ts, lat, lon, spd


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 8191, 8192, 8193, 16_385, 300_001])
def test_hygiene_tiles(cv, n):
    print(f"[hygiene tiles] n={n}", flush=True)
    import torch
    s = _sorted(n, n)
    rec = cv.to_device(s)
    perm = torch.randperm(n, dtype=torch.int32).cuda()
    keep = oracle.drop_duplicates(s)
    for p in (perm, None):
        kept, kperm, r = cv.cv_drop_duplicates(rec, p)
        assert r["count"] == len(keep) and r["n_late"] == 0
        if p is not None:
            assert_exact("perm", host(kperm), host(perm)[keep])
        for (k, _), c in zip(cv.RECORD_FIELDS, s):
            assert_exact(k, host(kept[k]).view(np.uint8), np.ascontiguousarray(c[keep]).view(np.uint8))
    for gap in (0, 45_000):
        et, ej = oracle.split_trips(s[0], s[1], gap)
        tid, tj, r = cv.cv_split_trips(rec, gap)
        assert r["count"] == len(ej) and r["n_late"] == 0
        assert_exact("trip_id", host(tid), et)
        assert_exact("trip_journey", host(tj), ej)
