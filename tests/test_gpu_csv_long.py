"""Text extraction of rows that end past the bytes staged for their tile (16 384
bytes and 1 024 after them), which the whole block reads 4 096 bytes a step, and
of lines of 2^20 bytes and more, which are malformed without being read to their
end.  Against the oracle's definition, exactly."""
import numpy as np
import pytest

import oracle

from _parity import assert_exact, host

pytestmark = pytest.mark.gpu

TILE, HALO, STEP, ROW_MAX = 16_384, 1_024, 4_096, 1 << 20
BODY = b"k%d,2021-05-09 00:00:01.%d,38.25,-92.5,%s,10.5,90"


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    oracle.lib()
    return cvetl


def _check(cv, text, header=False):
    import torch
    print(f"[csv long] bytes={len(text)} header={header}", flush=True)
    dev = torch.from_numpy(np.frombuffer(text, dtype=np.uint8).copy()).cuda()
    rec, hd, ok, r = cv.cv_csv_extract(dev, has_header=header, capacity=max(1, text.count(b"\n") + 1))
    # (the oracle has no bound on a line: those of ROW_MAX bytes are malformed)
    lines = [x if len(x) - x.endswith(b"\r") < ROW_MAX else b"x" for x in text.split(b"\n")]
    (ej, et, ela, elo, esp), ehd, eok = oracle.csv_extract(b"\n".join(lines), header)
    assert r["count"] == len(eok) and r["n_bad"] == int((eok == 0).sum())
    assert_exact("row_ok", host(ok), eok)
    for k, e in (("journey_id", ej), ("ts_ms", et)):
        assert_exact(k, host(rec[k]), e)
    for k, e in (("lat_deg", ela), ("lon_deg", elo)):
        assert_exact(k, host(rec[k]).view(np.uint64), e.view(np.uint64))
    assert_exact("speed", host(rec["speed_mps"]).view(np.uint32), esp.view(np.uint32))
    assert_exact("heading", host(hd).view(np.uint32), ehd.view(np.uint32))
    return eok


def _row(i, size, fill=b"7"):
    """A row of `size` bytes."""
    row = BODY % (i, i % 10, b"")
    return BODY % (i, i % 10, fill * (size - len(row)))


@pytest.mark.parametrize("size", [HALO + 1, STEP - 1, STEP, STEP + 1, 2 * STEP + 16, TILE, TILE + HALO, TILE + HALO + 1,
                                  3 * TILE + 7])
@pytest.mark.parametrize("eol", [b"\n", b"\r\n"])
def test_csv_long_rows(cv, size, eol):
    """Rows of about `size` bytes, among them some with a comma too many or too few, or a quote, at either end."""
    rows = [_row(i, size + i % 5 - 2) for i in range(60)]
    for i in range(5, 60, 6):
        r = rows[i]
        rows[i] = [r + b",", b"," + r, r[:40] + b"," + r[40:], r[:-9] + b'"' + r[-9:], b'"' + r, r.replace(b",", b"", 1),
                   r[:-3] + b"x" + r[-3:], r.replace(b"2021", b"2021-", 1), r[:len(r) // 2], r + b"\r"][i // 6 % 10]
    for tail in (b"", eol):
        ok = _check(cv, eol.join(rows) + tail)
        assert ok.sum() >= 45
    _check(cv, eol.join(rows) + eol + b"short" + eol + rows[0], header=True)


@pytest.mark.parametrize("eol", [b"\n", b"\r\n"])
def test_csv_rows_at_the_length_limit(cv, eol):
    short = BODY % (7, 7, b"65536")
    for at in (0, 1, 15, 16, 16_000):
        for size in (ROW_MAX - 1, ROW_MAX, ROW_MAX + 1, ROW_MAX + STEP):
            text = b"x" * at + b"\n" + short + eol + _row(1, size) + eol + short
            ok = _check(cv, text)
            assert list(ok) == [0, 1, int(size < ROW_MAX), 1]
            assert list(_check(cv, text[:-len(short) - len(eol)]))[2:] == [int(size < ROW_MAX)]


@pytest.mark.parametrize("fill", [b"x", b"\r", b","])
def test_csv_line_without_end(cv, fill):
    """64 MB without a newline after a row: refused from its first 2^20 bytes, which a
    block reads in about a millisecond.  One thread read it to the end, some 0.2 us
    per byte, 13 s."""
    import torch
    row = np.frombuffer(BODY % (7, 7, b"65536") + b"\n", dtype=np.uint8)
    text = torch.full(((64 << 20) + len(row),), fill[0], dtype=torch.uint8, device="cuda")
    text[:len(row)] = torch.from_numpy(row.copy()).cuda()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for _ in range(2):
        e[0].record()
        rec, hd, ok, r = cv.cv_csv_extract(text, has_header=False, capacity=4)
        e[1].record()
    torch.cuda.synchronize()
    assert r["count"] == 2 and r["n_bad"] == 1 and list(host(ok))[:2] == [1, 0]
    assert e[0].elapsed_time(e[1]) < 100.0
