"""Calls captured once and replayed on other data of the same sizes, with eager work in
between: a record sort whose ids are few in one replay and more than 2^19 in the next
(one launch that picks its tiles by the count), the hygiene passes (tickets and
look-back words cleared by each replay) and text with rows that the whole block reads.
Every replay is compared with the eager call's definition."""
import ctypes

import numpy as np
import pytest

import oracle
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
    oracle.lib()
    return cvetl


def _copy(dst, cols):
    import torch
    for (k, d), c in zip(dst.items(), cols):
        d.copy_(torch.from_numpy(np.ascontiguousarray(c)))


def test_sort_of_a_counted_number_of_ids(cv):
    import torch
    n, room = 700_000, 700_000
    rng = np.random.default_rng(5)
    sets = []
    for ids in (50, 600_000, 30_000, n, 1):
        jid = rng.permutation(np.arange(n) % ids) * 97 - 5_000_000
        sets.append((jid, gen.T0_MS + rng.integers(0, 1 << 20, n), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
                     np.zeros(n, np.float32)))
    rec = cv.to_device(sets[0])
    ws = cv.workspace(cv._size(cv.lib().cv_sort_workspace_size, n, room))
    cv.cv_sort_records(rec, max_journeys=room, ws=ws)
    torch.cuda.synchronize()
    print("[captured] sort", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        perm = cv.cv_sort_records(rec, max_journeys=room, ws=ws, sync=False)[0]
    for k in (0, 1, 2, 3, 4, 1, 0):
        _copy(rec, sets[k])
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(perm).astype(np.int64), np.lexsort((sets[k][1], sets[k][0]))), k


def test_hygiene(cv):
    import torch
    n = 100_001
    rng = np.random.default_rng(6)
    sets = []
    for share in (0.5, 0.0, 1.0):
        ts = gen.T0_MS + np.cumsum(np.where(rng.random(n) < share, 0, 40_000))
        pos = rng.integers(0, 2, n).astype(np.float64)
        sets.append((np.arange(n) // 700, ts, 38 + pos, -92 - pos, np.zeros(n, np.float32)))
    rec = cv.to_device(sets[0])
    out, res = cv.empty_records(n), [cv.new_result(), cv.new_result()]
    trip, start = (torch.empty(n, dtype=torch.int64, device="cuda") for _ in range(2))
    need = cv._size(cv.lib().cv_hygiene_workspace_size, n)
    ws = cv.workspace(need)
    oo = cv.CvRecordsOut(*(cv._ptr(out[k]) for k, _ in cv.RECORD_FIELDS))

    def call():
        r = cv._records_struct(rec)
        assert cv.lib().cv_drop_duplicates(ctypes.byref(r), None, ctypes.byref(oo), None, cv._ptr(res[0]), cv._ptr(ws), need,
                                           cv._stream()) == 0
        assert cv.lib().cv_split_trips(ctypes.byref(r), 30_000, cv._ptr(trip), cv._ptr(start), n, cv._ptr(res[1]),
                                       cv._ptr(ws), need, cv._stream()) == 0

    call()
    torch.cuda.synchronize()
    print("[captured] hygiene", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for k in (0, 1, 2, 1, 0):
        _copy(rec, sets[k])
        g.replay()
        torch.cuda.synchronize()
        keep = oracle.drop_duplicates(sets[k])
        assert cv.read_result(res[0])["count"] == len(keep)
        assert np.array_equal(host(out["ts_ms"])[:len(keep)], sets[k][1][keep])
        et, ej = oracle.split_trips(sets[k][0], sets[k][1], 30_000)
        assert cv.read_result(res[1])["count"] == len(ej) and np.array_equal(host(trip), et)


def test_text_with_long_rows(cv):
    import torch
    size = 200_000
    texts = []
    for long in (7, 3_000, 40_000):
        rows = [b"k%d,2021-05-09 00:00:01,38.25,-92.5,%s,%d.5,90" % (i, b"7" * (long if i % 3 else 5), i % 60) for i in range(4_000)]
        texts.append((b"\n".join(rows) + b"\n")[:size])
    cap = max(t.count(b"\n") for t in texts) + 1
    buf = torch.from_numpy(np.frombuffer(texts[0], dtype=np.uint8).copy()).cuda()
    out = cv.empty_records(cap)
    hd, ok = torch.empty(cap, device="cuda"), torch.empty(cap, dtype=torch.uint8, device="cuda")
    ws = cv.workspace(cv._size(cv.lib().cv_csv_workspace_size, size, cap))
    call = lambda: cv.cv_csv_extract(buf, has_header=False, capacity=cap, out=out, heading=hd, row_ok=ok, ws=ws,  # noqa: E731
                                     sync=False)[3]
    call()
    torch.cuda.synchronize()
    print("[captured] text", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        res = call()
    for k in (0, 1, 2, 1, 0):
        buf.copy_(torch.from_numpy(np.frombuffer(texts[k], dtype=np.uint8).copy()))
        g.replay()
        torch.cuda.synchronize()
        (ej, _, _, _, esp), _, eok = oracle.csv_extract(texts[k], False)
        r = cv.read_result(res)
        assert r["count"] == len(eok) and r["n_bad"] == int((eok == 0).sum())
        assert np.array_equal(host(ok)[:len(eok)], eok) and np.array_equal(host(out["journey_id"])[:len(eok)], ej)
        assert np.array_equal(host(out["speed_mps"])[:len(eok)].view(np.uint32), esp.view(np.uint32))
