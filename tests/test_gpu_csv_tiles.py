"""Text extraction at the edges of its tiles (16 384 bytes and 1 024 bytes after
them), of its row lists (512 rows a round) and of the eight-character forms of
its fields, against the oracle's definition, exactly."""
import numpy as np
import pytest

import oracle

from _parity import assert_exact, host

pytestmark = pytest.mark.gpu

TILE, HALO = 16_384, 1_024


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    oracle.lib()
    return cvetl


def _check(cv, text, header=True):
    import torch
    print(f"[csv tiles] bytes={len(text)} header={header}", flush=True)
    dev = torch.from_numpy(np.frombuffer(text, dtype=np.uint8).copy()).cuda()
    (ej, et, ela, elo, esp), ehd, eok = oracle.csv_extract(text, header)
    rec, hd, ok, r = cv.cv_csv_extract(dev, has_header=header, capacity=max(1, len(eok)))
    assert r["count"] == len(eok) and r["n_bad"] == int((eok == 0).sum())
    assert_exact("row_ok", host(ok), eok)
    for k, e in (("journey_id", ej), ("ts_ms", et)):
        assert_exact(k, host(rec[k]), e)
    for k, e in (("lat_deg", ela), ("lon_deg", elo)):
        assert_exact(k, host(rec[k]).view(np.uint64), e.view(np.uint64))
    assert_exact("speed", host(rec["speed_mps"]).view(np.uint32), esp.view(np.uint32))
    assert_exact("heading", host(hd).view(np.uint32), ehd.view(np.uint32))


def _row(rng, i):
    """A valid row of uneven widths."""
    f = [b"%d%c" % (rng.integers(0, 10 ** rng.integers(1, 7)), rng.integers(97, 123)),
         b"2021-%02d-%02d %02d:%02d:%02d" % tuple(rng.integers([1, 1, 0, 0, 0], [13, 29, 24, 60, 60]))]
    f[1] += [b"", b".%d" % rng.integers(0, 10), b".%02d" % rng.integers(0, 100), b".%03d" % rng.integers(0, 1000)][i % 4]
    f += [b"%.*f" % (int(rng.integers(0, 9)), rng.uniform(36, 41)), b"%.*f" % (int(rng.integers(0, 8)), -rng.uniform(89, 96)),
          b"%d" % rng.integers(0, 10 ** rng.integers(1, 6)), b"%.2f" % rng.uniform(0, 45),
          [b"", b"%d" % rng.integers(0, 360)][i % 3 > 0]]
    return b",".join(f)


FORMS = [b"0", b"-0", b"+0.0", b".5", b"5.", b".", b"-", b"", b"+.", b"00000001", b"000000001", b"12345678.12345678",
         b"123456789.1", b"1.123456789", b"90071992.54740991", b"90071992.54740992", b"99999999.9999999", b"1..2", b"1.2.3",
         b"1 ", b" 1", b"1e3", b"0x10", b"--1", b"1-", b"12/3", b"1:2", b"0.0000000000000000000001",
         b"0.00000000000000000000001", b"9007199254740991", b"9007199254740992", b"9007199254740993.5", b"1,5", b'"1"']
STAMPS = [b"2021-05-09 00:00:00", b"2021-05-09 00:00:00.", b"2021-05-09 00:00:00.1", b"2021-05-09 00:00:00.12",
          b"2021-05-09 00:00:00.123", b"2021-05-09 00:00:00.1234", b"2021-05-09 00:00:00.1a3", b"2021-05-09T00:00:00",
          b"2021-13-09 00:00:00", b"2021-00-09 00:00:00", b"2021-04-31 00:00:00", b"2021-02-29 00:00:00",
          b"2024-02-29 23:59:59.999", b"1900-02-29 00:00:00", b"2000-02-29 00:00:00", b"0000-01-01 00:00:00",
          b"0001-01-01 00:00:00", b"9999-12-31 23:59:59", b"2021-05-09 24:00:00", b"2021-05-09 00:60:00",
          b"2021-05-09 00:00:60", b"2021-5-09 00:00:00", b"2021/05/09 00:00:00", b"1969-12-31 23:59:59.5",
          b"2021-05-09 0a:00:00", b"202 -05-09 00:00:00", b"2021-05-32 00:00:00", b"2021-05-00 00:00:00"]
IDS = [b"a", b"abcdefgh", b"abcdefghi", b"", b"\x7f\x01", b"\x80a", b"7 z", b"12345678"]


def test_csv_field_forms(cv):
    good = [b"33456rd", b"2021-05-09 03:48:42", b"37.664087", b"-92.6546", b"65536", b"105.98", b"33"]
    rows = []
    for at, forms in ((0, IDS), (1, STAMPS), (2, FORMS), (3, FORMS), (4, FORMS), (5, FORMS), (6, FORMS)):
        rows += [b",".join(good[:at] + [f] + good[at + 1:]) for f in forms]
    rows += [b",".join(good[:k]) for k in range(7)] + [b",".join(good) + b",", b",,,,,,"]
    for eol in (b"\n", b"\r\n"):
        _check(cv, eol.join(rows) + eol, header=False)
        _check(cv, b"\r" + eol + b"\r\r" + eol + eol.join(rows), header=True)


@pytest.mark.parametrize("size", [TILE - 1, TILE, TILE + 1, TILE + HALO, TILE + HALO + 1, 3 * TILE])
@pytest.mark.parametrize("tail", [b"", b"\n"])
def test_csv_text_ends_at_tile_edges(cv, size, tail):
    rng = np.random.default_rng(size)
    rows, n, i = [], 0, 0
    while n < size - 200:
        rows.append(_row(rng, i))
        n += len(rows[-1]) + 1
        i += 1
    text = b"\n".join(rows) + b"\n"
    last = _row(rng, 1)
    fill = size - len(text) - len(last) - len(tail) - 1
    _check(cv, text + b"x" * fill + b"\n" + last + tail)


@pytest.mark.parametrize("lead", [TILE - 60, TILE - 2, TILE - 1, TILE, TILE + 1])
@pytest.mark.parametrize("long", [50, 127, 128, 129, 1_000, 1_100, 2 * TILE + 5])
def test_csv_rows_across_tile_edges(cv, lead, long):
    """A row that starts at `lead`, with a postal code that makes it `long` bytes, between ordinary ones."""
    rng = np.random.default_rng(lead + long)
    body = b"k,2021-05-09 00:00:01,38.25,-92.5,%s,10.5,90"
    row = body % (b"7" * max(0, long - len(body) + 2))
    text = b"x" * (lead - 1) + b"\n" + row + b"\n" + b"\n".join(_row(rng, i) for i in range(40)) + b"\n"
    _check(cv, text)


@pytest.mark.parametrize("unit", [b"\n", b"a\n", b",,,,,,\n", b"\r\n"])
def test_csv_many_short_rows(cv, unit):
    n = (TILE + 3_000) // len(unit)
    _check(cv, unit * n + b"k,2021-05-09 00:00:01,38.25,-92.5,7,10.5,90", header=False)


def test_csv_capacity_across_tiles(cv):
    import torch
    rng = np.random.default_rng(8)
    rows = [_row(rng, i) for i in range(2_000)]
    text = b"h\n" + b"\n".join(rows) + b"\n"
    dev = torch.from_numpy(np.frombuffer(text, dtype=np.uint8).copy()).cuda()
    (ej, *_), _, _ = oracle.csv_extract(text)
    for cap in (1, 511, 1_999):
        out = {k: torch.full((cap + 8,), 77, dtype=dt, device="cuda") for k, dt in cv.RECORD_FIELDS}
        res = cv.cv_csv_extract(dev, capacity=cap, out=out, sync=False)[3]
        r = cv.read_result(res)
        assert r["status"] == cv.CV_ERR_CAPACITY and r["count"] == r["required"] == 2_000
        assert_exact("journey_id", host(out["journey_id"])[:cap], ej[:cap])
        assert all(bool((v[cap:] == 77).all()) for v in out.values())


def test_csv_text_beyond_self_summed_tiles(cv):
    """More tiles than a block sums itself: the scanned counts."""
    rng = np.random.default_rng(3)
    block = b"\n".join(_row(rng, i) for i in range(20_000)) + b"\n"
    reps = (2_049 * TILE) // len(block) + 1
    import torch
    text = torch.from_numpy(np.frombuffer(block, dtype=np.uint8).copy()).cuda().repeat(reps)
    rec, hd, ok, r = cv.cv_csv_extract(text, has_header=False, capacity=20_000 * reps)
    (ej, et, ela, elo, esp), ehd, eok = oracle.csv_extract(block, False)
    assert r["count"] == 20_000 * reps and r["n_bad"] == reps * int((eok == 0).sum())
    for got, e in ((rec["journey_id"], ej), (rec["ts_ms"], et), (rec["lat_deg"], ela), (rec["lon_deg"], elo),
                   (rec["speed_mps"], esp), (ok, eok)):
        assert bool((got.view(reps, -1) == torch.from_numpy(e).cuda()[None]).all())
