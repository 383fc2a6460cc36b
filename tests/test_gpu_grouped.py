"""Input of whole journeys, one run of records per id, in time order but for
near neighbours: its order without radix passes, on both sides of every
condition of that form.  Records moved by 1 to 9 places (3 is the limit, 4 the
first beyond it), gaps on either side of 2^27 ms, ids with a second run, the
id that has no dictionary slot, runs that end at every offset of a wave's window,
few ids (counted), many (sorted chunks, radix passes).  The order and every
sorted column equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2305_07454_amd import gen

from _parity import check_features, check_sort

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


def _runs(seed, lengths, step=1000):
    """Journeys one after the other, time stamps rising by 0 or 1 step."""
    rng = np.random.default_rng(seed)
    lengths = np.asarray(lengths)
    n = int(lengths.sum())
    ids = rng.choice(2 ** 40, len(lengths), replace=False) * 3 - 2 ** 41
    run = np.repeat(np.arange(len(lengths)), lengths)
    place = np.arange(n) - np.repeat(np.cumsum(lengths) - lengths, lengths)
    ts = gen.T0_MS + rng.integers(0, 1 << 20, len(lengths))[run] * step + place * step
    dup = (rng.random(n) < 0.05) & (place > 0)
    ts[dup] -= step
    return ids, run, place, ts, rng


def _check(cv, jid, ts, max_journeys=None, fused=True):
    import torch
    n = len(jid)
    rng = np.random.default_rng(n)
    cols = (np.ascontiguousarray(jid, np.int64), np.ascontiguousarray(ts, np.int64), rng.uniform(36, 40, n),
            rng.uniform(-95, -90, n), rng.uniform(0, 40, n).astype(np.float32))
    d = cv.to_device(cols)
    mj = max_journeys or len(np.unique(jid)) + 3
    perm, srt, r = cv.cv_sort_records(d, max_journeys=mj)
    exp = oracle.sort(cols[0], cols[1])
    es = oracle.sorted_records(cols, exp)
    check_sort(perm, srt, exp, es)
    assert r["count"] == len(np.unique(jid))
    if fused:
        perm, srt, feat, _ = cv.cv_sort_records_features(d, mj)
        check_sort(perm, srt, exp, es)
        check_features(feat, oracle.features(*es[:4]))
    torch.cuda.synchronize()
    return r


def _lengths(rng, n, mean):
    out = []
    while sum(out) < n:
        out.append(int(rng.integers(1, 2 * mean)))
    out[-1] -= sum(out) - n
    return out


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 4_097, 100_003])
@pytest.mark.parametrize("mean", [9, 77, 1_000, 300_000])
def test_whole_journeys(cv, n, mean):
    print(f"[grouped] n={n} mean={mean}", flush=True)
    rng = np.random.default_rng(n + mean)
    ids, run, place, ts, rng = _runs(3, _lengths(rng, n, mean))
    order = np.arange(n)
    a = np.nonzero((rng.random(n) < 0.02) & (np.roll(run, -1) == run) & (np.arange(n) < n - 1))[0]
    a = a[np.diff(a, prepend=-2) > 1]
    order[a], order[a + 1] = a + 1, a
    _check(cv, ids[run[order]], ts[order])


@pytest.mark.parametrize("far", [1, 2, 3, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("back", [False, True])
def test_records_out_of_place(cv, far, back):
    # single records moved by `far` places, at every offset of the windows
    n = 64 * 71
    ids, run, place, ts, rng = _runs(5, [70] * (n // 70) + [n % 70])
    order = np.arange(n)
    for at in range(11, n - 20, 37):
        src = at if not back else at + far
        dst = at + far if not back else at
        if run[src] != run[dst]:
            continue
        block = list(order[at:at + far + 1])
        order[at:at + far + 1] = block[1:] + block[:1] if not back else block[-1:] + block[:-1]
    print(f"[grouped] moved by {far} back={back}", flush=True)
    _check(cv, ids[run[order]], ts[order])
    # windows of far + 1 records in random order
    order = np.arange(n)
    for at in range(5, n - 20, 23):
        if run[at] == run[at + far]:
            order[at:at + far + 1] = at + rng.permutation(far + 1)
    _check(cv, ids[run[order]], ts[order])


@pytest.mark.parametrize("what", ["gap_below", "gap_at", "gap_back", "second_run", "min_id", "min_id_last", "one",
                                  "reversed", "equal_times", "wide_times", "capacity"])
def test_edges_of_the_form(cv, what):
    print(f"[grouped] {what}", flush=True)
    n = 30_011
    ids, run, place, ts, rng = _runs(9, _lengths(np.random.default_rng(1), n, 150))
    jid = ids[run]
    if what.startswith("gap"):
        d = dict(gap_below=(1 << 27) - 1, gap_at=1 << 27, gap_back=-(1 << 27))[what]
        ts = gen.T0_MS + place.astype(np.int64)
        ts[(place >= 20)] += d - 1
    elif what == "second_run":
        jid = jid.copy()
        jid[run == run[-1]] = ids[3]
    elif what.startswith("min_id"):
        ids[-1 if what == "min_id_last" else 4] = -2 ** 63
        jid = ids[run]
    elif what == "one":
        jid = np.full(n, 7)
        ts = gen.T0_MS + np.arange(n) * 1000
        ts[5::64], ts[6::64] = ts[6::64].copy(), ts[5::64].copy()
    elif what == "reversed":
        ts = ts[::-1].copy()
        jid = jid[::-1].copy()
    elif what == "equal_times":
        ts = np.full(n, gen.T0_MS)
    elif what == "wide_times":
        ts = ts + run.astype(np.int64) * (1 << 40)
    elif what == "capacity":
        with pytest.raises(cv.CvError):  # too few journeys: the call says so
            _check(cv, jid, ts, max_journeys=17)
    _check(cv, jid, ts)


@pytest.mark.parametrize("ids,max_journeys", [(16_384, None), (16_385, None), (70_001, None), (70_001, 100_000),
                                              (20_000, 600_000), (300, 20_000)])
def test_many_journeys(cv, ids, max_journeys):
    print(f"[grouped] ids={ids} capacity={max_journeys}", flush=True)
    names, run, place, ts, rng = _runs(13, np.random.default_rng(2).integers(6, 14, ids))
    ts = ts ^ (place % 2)  # (no common factor)
    order = np.arange(len(run))
    a = np.nonzero((place % 8 == 2) & (np.roll(run, -1) == run))[0]
    order[a], order[a + 1] = a + 1, a
    names[ids // 2] = -2 ** 63
    _check(cv, names[run[order]], ts[order], max_journeys=max_journeys)


@pytest.mark.parametrize("far", [2, 3, 4, 5, 6, 7, 8, 12])
@pytest.mark.parametrize("back", [False, True])
def test_one_record_out_of_place(cv, far, back):
    # a single record out of its place, at every lane of a window and across the
    # edge of the next, with the records around it in every close order
    print(f"[grouped] one record moved by {far} back={back}", flush=True)
    n = 600
    rng = np.random.default_rng(far)
    ts0 = gen.T0_MS + 1000 * np.arange(n)
    for at in range(380, 380 + 130):
        for near in (False, True):
            order = np.arange(n)
            block = list(order[at:at + far + 1])
            order[at:at + far + 1] = block[-1:] + block[:-1] if back else block[1:] + block[:1]
            if near:  # neighbours changed places around it
                for i in (at + 1, at + far - 2, at + far + 2):
                    if rng.random() < 0.5:
                        order[i], order[i + 1] = order[i + 1], order[i]
            ts = ts0[order]
            jid = (np.arange(n) >= 300).astype(np.int64) * 7
            cols = (jid, ts, np.full(n, 37.0), np.full(n, -92.0), np.zeros(n, np.float32))
            perm = cv.cv_sort_records(cv.to_device(cols), max_journeys=4)[0]
            assert np.array_equal(perm.cpu().numpy().astype(np.int64), np.lexsort((ts, jid))), (at, near)
