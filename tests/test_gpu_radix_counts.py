"""Sorts whose number of keys is known on the device alone, around 2^20 and 2^21 keys
allowed: the grid's partial rows (nearly every record with a row of its own, or few) and
the record sort's distinct ids (all there or few).  Compared with numpy."""
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


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, (1 << 21) + 1])
@pytest.mark.parametrize("hold", [1, 64])
def test_grid_rows(cv, n, hold):
    """A cell held for `hold` records; journeys of 1 024 records, whole speeds."""
    print(f"[radix counts] grid n={n} hold={hold}", flush=True)
    rng = np.random.default_rng(n + hold)
    cells = 1 << 18
    cell = np.repeat(rng.integers(0, cells, n // hold + 1), hold)[:n]
    spd = rng.integers(0, 40, n).astype(np.float32)
    jid = np.arange(n) // 1024
    cols = (jid, np.full(n, gen.T0_MS), np.full(n, 36.5), -94.5 + cell, spd)
    grid = gen.GridSpec(36.0, -95.0, 1.0, 1.0, 1, cells, gen.T0_MS, 1000, 1)
    got, r = cv.cv_grid_aggregate(cv.to_device(cols), grid)
    uk, at = np.unique(cell, return_inverse=True)
    pairs = np.unique(cell * (1 << 32) + jid)
    assert r["count"] == len(uk) and r["n_out_of_grid"] == 0
    assert np.array_equal(host(got["key"]), uk)
    assert np.array_equal(host(got["count"]), np.bincount(at))
    assert np.array_equal(host(got["n_journeys"]), np.bincount(np.searchsorted(uk, pairs >> 32), minlength=len(uk)))
    assert np.array_equal(host(got["sum_speed"]), np.bincount(at, spd.astype(np.float64)))


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("ids", [7, 1 << 21])
def test_distinct_ids(cv, n, ids):
    print(f"[radix counts] ids={ids} n={n}", flush=True)
    rng = np.random.default_rng(n + ids)
    jid = (rng.permutation(n) * 3 - n) if ids > 7 else rng.integers(0, ids, n)
    cols = (jid, gen.T0_MS + rng.integers(0, 1 << 20, n), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
            np.zeros(n, np.float32))
    perm, srt, r = cv.cv_sort_records(cv.to_device(cols), max_journeys=n)
    exp = np.lexsort((cols[1], jid))
    assert r["count"] == len(np.unique(jid))
    assert np.array_equal(host(perm).astype(np.int64), exp)
    assert np.array_equal(host(srt["journey_id"]), jid[exp])
