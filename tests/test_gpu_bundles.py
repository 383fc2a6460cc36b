"""Record sorts of bundled feeds: runs of a few records per vehicle, each in time
order, one vehicle's after another's, so that windows look like whole journeys until
an id comes a second time.  Order against numpy; and what the key's preparation takes,
beside a feed of single records."""
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


def _check(cv, jid, ts):
    n = len(jid)
    rng = np.random.default_rng(n)
    cols = (jid, ts, rng.uniform(36, 40, n), rng.uniform(-95, -90, n), np.zeros(n, np.float32))
    perm, srt, r = cv.cv_sort_records(cv.to_device(cols))
    exp = np.lexsort((ts, jid))
    assert r["count"] == len(np.unique(jid))
    assert np.array_equal(host(perm).astype(np.int64), exp)
    assert np.array_equal(host(srt["journey_id"]), jid[exp]) and np.array_equal(host(srt["lat_deg"]), cols[2][exp])


def _bundles(n, size, ids):
    """Rounds of one run per id, ids in another order each round."""
    rng = np.random.default_rng(n + size)
    rounds = -(-n // (size * ids))
    order = np.concatenate([rng.permutation(ids) for _ in range(rounds)])
    jid = (np.repeat(order, size) * 7919 - 3)[:n]
    t = np.repeat(np.arange(rounds), ids * size) * size + np.tile(np.arange(size), rounds * ids)
    return jid, gen.T0_MS + 1000 * t[:n]


@pytest.mark.parametrize("size", [4, 5, 16, 64, 100])
@pytest.mark.parametrize("n,ids", [(1_000, 3), (70_001, 40), (600_011, 2_000), (3_000_001, 70_000)])
def test_bundles(cv, n, ids, size):
    print(f"[bundles] n={n} ids={ids} size={size}", flush=True)
    _check(cv, *_bundles(n, size, ids))


@pytest.mark.parametrize("at", [2, 5, 13, 100, 20_000, 29_999])
@pytest.mark.parametrize("low", [False, True])
def test_one_id_twice(cv, at, low):
    """30 000 whole journeys of 20 records, one of which comes back as the run `at` (the id
    that has no slot of its own among them)."""
    print(f"[bundles] at={at} low={low}", flush=True)
    runs = np.arange(30_000) * 11 + 5
    runs[at] = runs[0]
    jid = np.repeat(runs, 20)
    if low:
        jid[jid == runs[0]] = np.iinfo(np.int64).min
    _check(cv, jid, gen.T0_MS + 1000 * np.arange(len(jid)))


def test_bundles_cost_no_more_than_single_records(cv):
    """20 M records of 8 000 ids: the preparation of runs of five and of single records.
    Following every run's start and end through the table, as for whole journeys, takes
    1.6 times the single records' time; without it, runs need fewer look-ups than those."""
    import torch
    n, ids, ms = 20_000_000, 8_000, {}
    for size in (5, 1):
        j, t = _bundles(n, size, ids)
        cols = dict(journey_id=j, ts_ms=t, lat_deg=np.zeros(n), lon_deg=np.zeros(n), speed_mps=np.zeros(n, np.float32))
        rec = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in cols.items()}
        ws = cv.workspace(cv._size(cv.lib().cv_sort_workspace_size, n, 2 * ids))
        cv.cv_sort_records(rec, max_journeys=2 * ids, ws=ws)
        took = []
        for _ in range(5):
            cv.cv_timing_reset()
            cv.cv_timing_enable(True)
            cv.cv_sort_records(rec, max_journeys=2 * ids, ws=ws, sync=False)
            torch.cuda.synchronize()
            cv.cv_timing_enable(False)
            took.append(cv.cv_timing_read("sort_prep")[0])
        ms[size] = min(took)
    print(f"[bundles] preparation {ms}", flush=True)
    assert ms[5] < 1.25 * ms[1]
