"""Sorts of all passes in one launch whose number of keys is known on the device
alone (the grid's partial rows, the record sort's distinct ids): counts on both sides
of 2^19, where the launch changes its tiles, and bounds on both sides of 2^22, where
launches per pass take over.  Compared with numpy."""
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


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, 1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("rows", [1, 4_097, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1 << 21])
def test_grid_rows(cv, n, rows):
    """`rows` runs of one cell each, none across a tile's or a wave's edge (512 records): a row per run."""
    print(f"[radix counted] grid n={n} rows={rows}", flush=True)
    rng = np.random.default_rng(n + rows)
    # as many runs as blocks of 512 records at least
    blocks = -(-n // 512)
    rows = min(max(rows, blocks), n)
    start = np.zeros(n, bool)
    start[::512] = True
    free = np.nonzero(~start)[0]
    start[rng.permutation(free)[:rows - blocks]] = True
    which = np.cumsum(start) - 1
    cells = 1 << 22
    cell = (rng.permutation(cells)[:rows])[which]
    spd = rng.integers(0, 40, n).astype(np.float32)
    cols = (np.arange(n) // 2048, np.full(n, gen.T0_MS), np.full(n, 36.5), -94.5 + cell, spd)
    grid = gen.GridSpec(36.0, -95.0, 1.0, 1.0, 1, cells, gen.T0_MS, 1000, 1)
    got, r = cv.cv_grid_aggregate(cv.to_device(cols), grid, capacity=rows)
    uk, at = np.unique(cell, return_inverse=True)
    assert r["count"] == len(uk) == rows and r["n_out_of_grid"] == 0
    assert np.array_equal(host(got["key"]), uk)
    assert np.array_equal(host(got["count"]), np.bincount(at))
    assert np.array_equal(host(got["sum_speed"]), np.bincount(at, spd.astype(np.float64)))


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("ids", [16_385, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1 << 22])
def test_distinct_ids(cv, n, ids):
    print(f"[radix counted] ids={ids} n={n}", flush=True)
    rng = np.random.default_rng(n + ids)
    jid = rng.permutation(np.arange(n) % ids) * 4_000_037 - (1 << 40)
    cols = (jid, gen.T0_MS + rng.integers(0, 1 << 20, n), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
            np.zeros(n, np.float32))
    perm, srt, r = cv.cv_sort_records(cv.to_device(cols), max_journeys=n)
    exp = np.lexsort((cols[1], jid))
    assert r["count"] == min(n, ids)
    assert np.array_equal(host(perm).astype(np.int64), exp)
    assert np.array_equal(host(srt["journey_id"]), jid[exp])
