"""The hygiene calls' scratch lies in their workspace alone: calls on two streams
that share one result word (whose content is then either's) still write every row,
whatever the word holds beforehand, and keep within the workspace asked for."""
import ctypes

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


class Side:
    """One caller: its records, outputs, workspace of exactly the size asked for with a guard behind, and stream."""

    def __init__(self, cv, n, seed):
        import torch
        rng = np.random.default_rng(seed)
        jid = np.cumsum(rng.random(n) < 1 / 500)
        ts = gen.T0_MS + np.cumsum(rng.integers(0, 3, n) * 20_000)
        pos = rng.integers(0, 2, n).astype(np.float64)
        self.cols = (jid.astype(np.int64), ts, 38.0 + pos, -92.0 - pos, np.zeros(n, np.float32))
        self.rec = cv.to_device(self.cols)
        self.out = cv.empty_records(n)
        self.trip = torch.empty(n, dtype=torch.int64, device="cuda")
        self.start = torch.empty(n, dtype=torch.int64, device="cuda")
        self.need = cv._size(cv.lib().cv_hygiene_workspace_size, n)
        self.ws = torch.full((self.need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        self.stream = torch.cuda.Stream()
        self.n = n

    def enqueue(self, cv, res):
        L = cv.lib()
        rec = cv._records_struct(self.rec)
        oo = cv.CvRecordsOut(*(cv._ptr(self.out[k]) for k, _ in cv.RECORD_FIELDS))
        s = ctypes.c_void_p(self.stream.cuda_stream)
        assert L.cv_drop_duplicates(ctypes.byref(rec), None, ctypes.byref(oo), None, cv._ptr(res), cv._ptr(self.ws),
                                    self.need, s) == 0
        assert L.cv_split_trips(ctypes.byref(rec), 30_000, cv._ptr(self.trip), cv._ptr(self.start), self.n, cv._ptr(res),
                                cv._ptr(self.ws), self.need, s) == 0

    def check(self, cv):
        keep = oracle.drop_duplicates(self.cols)
        for (k, _), c in zip(cv.RECORD_FIELDS, self.cols):
            assert_exact(k, host(self.out[k])[:len(keep)], c[keep])
        et, ej = oracle.split_trips(self.cols[0], self.cols[1], 30_000)
        assert_exact("trip", host(self.trip), et)
        assert_exact("start", host(self.start)[:len(ej)], ej)
        assert bool((self.ws[self.need:] == 0xA5).all()), "bytes behind the workspace were written"
        return len(ej)


@pytest.mark.parametrize("n", [8_192, 8_193, 516_096, 524_289, 1_000_003])
def test_one_result_on_two_streams(cv, n):
    import torch
    print(f"[hygiene result] n={n}", flush=True)
    a, b = Side(cv, n, n), Side(cv, max(1, n // 3), n + 1)
    res = torch.full((64,), 0xFF, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for _ in range(20):
        a.enqueue(cv, res)
        b.enqueue(cv, res)
    torch.cuda.synchronize()
    trips = (a.check(cv), b.check(cv))
    a.enqueue(cv, res)
    torch.cuda.synchronize()
    r = cv.read_result(res)
    assert r == dict(r, status=0, count=trips[0], required=0, n_late=0, n_bad=0, flags=0)
