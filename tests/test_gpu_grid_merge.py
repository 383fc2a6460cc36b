"""The merge of the grid's partial rows at the edges of its ranges: tiles of
2 048 records (4 or more to a block of the compaction), chunks of 1 024 sorted
pairs (one or more to a block of the emit), groups that run over chunk and
block edges, a single group, a group per record, no group at all.  Compared
with numpy; speeds are whole numbers, so sums are exact."""
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


def _numpy_groups(jid, key, spd):
    ok = key >= 0
    uk, at = np.unique(key[ok], return_inverse=True)
    pairs = np.unique(np.stack([key[ok], jid[ok]], 1), axis=0) if ok.any() else np.zeros((0, 2), np.int64)
    lo = np.full(len(uk), np.inf, np.float32)
    hi = np.full(len(uk), -np.inf, np.float32)
    np.minimum.at(lo, at, spd[ok])
    np.maximum.at(hi, at, spd[ok])
    return dict(key=uk, count=np.bincount(at, minlength=len(uk)),
                n_journeys=np.bincount(np.searchsorted(uk, pairs[:, 0]), minlength=len(uk)),
                sum_speed=np.bincount(at, spd[ok].astype(np.float64), minlength=len(uk)), min_speed=lo, max_speed=hi)


@pytest.mark.parametrize("n", [1, 2047, 2049, 8192, 8193, 100_001, 1_050_000])
@pytest.mark.parametrize("shape", ["one", "each", "few", "mixed", "outside"])
def test_merge_of_partial_rows(cv, n, shape):
    print(f"[grid merge] n={n} {shape}", flush=True)
    rng = np.random.default_rng(n)
    jid = np.sort(rng.integers(0, max(1, n // 700) + 1, n))
    grid = gen.GridSpec(36.0, -95.0, 1.0, 1.0, 4, 1 << 21, gen.T0_MS, 1000, 4)
    cell = dict(one=np.zeros(n, np.int64), each=rng.permutation(n), few=rng.integers(0, 5, n),
                mixed=np.where(rng.random(n) < 0.5, 7, rng.integers(0, 2 * n, n)), outside=np.full(n, -5))[shape]
    ilat = rng.integers(0, 4, n) if shape == "mixed" else np.zeros(n, np.int64)
    spd = rng.integers(0, 40, n).astype(np.float32)
    cols = (jid, np.full(n, gen.T0_MS), 36.5 + ilat, -94.5 + cell, spd)
    key = np.where((cell >= 0) & (cell < grid.n_lon), ilat * grid.n_lon + cell, -1)
    got, r = cv.cv_grid_aggregate(cv.to_device(cols), grid)
    exp = _numpy_groups(jid, key, spd)
    assert r["count"] == len(exp["key"]) and r["n_out_of_grid"] == int((key < 0).sum())
    for k, e in exp.items():
        assert np.array_equal(host(got[k]).astype(e.dtype), e), k


@pytest.mark.parametrize("n", [1, 2049, 100_001, (1 << 19) - 100, (1 << 19) + 1, 2_200_000])
def test_merge_of_direction_rows(cv, n):
    """Directions that change at every record: a row for nearly each, in few and
    in many keys' sorts, chunks taken one to a block."""
    import torch
    print(f"[grid merge] directions n={n}", flush=True)
    rng = np.random.default_rng(n)
    jid = np.sort(rng.integers(0, max(1, n // 900) + 1, n))
    grid = gen.GridSpec(36.0, -95.0, 1.0, 1.0, 1, 1 << 12, gen.T0_MS, 1000, 4)
    cell, sector = rng.integers(0, 1 << 12, n), rng.integers(0, 8, n)
    spd = rng.integers(0, 40, n).astype(np.float32)
    cols = cv.to_device((jid, np.full(n, gen.T0_MS), np.full(n, 36.5), -94.5 + cell, spd))
    head = torch.from_numpy((sector * 45 + 10).astype(np.float32)).cuda()
    got, r = cv.cv_grid_aggregate_dir(cols, grid, 8, 0.0, heading=head)
    exp = _numpy_groups(jid, sector * (1 << 12) + cell, spd)
    assert r["count"] == len(exp["key"]) and r["n_out_of_grid"] == 0
    for k, e in exp.items():
        assert np.array_equal(host(got[k]).astype(e.dtype), e), k
