"""Text extraction with fewer rows of capacity than the text has (none at all
when only the count is asked for), in a workspace of exactly the size that the
query names: the rows counted, the first of them written, and every byte behind
the workspace left as it was."""
import ctypes

import numpy as np
import pytest

import oracle

from _parity import assert_exact, host

TILE = 16_384
GUARD = 64 * 1024


def _query(cvetl, nbytes, cap):
    return cvetl._size(cvetl.lib().cv_csv_workspace_size, nbytes, cap)


def test_csv_workspace_query_holds_the_tile_counts():
    """A count of 4 bytes per tile up to 2 048 tiles, of 12 per group of 4 tiles
    (each array aligned to 256 bytes) above; the capacity adds nothing, and a
    workspace of 4 bytes per tile, 8 per row and 256 is always enough."""
    from paper_2305_07454_amd import cvetl
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    for tiles in [1, 2, 63, 64, 65, 127, 128, 1_000, 2_047, 2_048, 2_049, 2_050, 4_097, 17_823, 1 << 20, (1 << 31) - 1]:
        for nbytes in {(tiles - 1) * TILE + 1, tiles * TILE - 1, tiles * TILE}:
            groups = (tiles + 3) // 4
            need = up(4 * tiles) if tiles <= 2_048 else up(up(8 * groups) + 4 * groups)
            for cap in (0, 1, 100, 10 ** 6):
                q = _query(cvetl, nbytes, cap)
                assert need <= q <= up(4 * (tiles + 1)) + up(8 * (cap + 3)) + 256, (tiles, nbytes, cap, q)


@pytest.mark.gpu
@pytest.mark.parametrize("cap", [0, 1, 100])
@pytest.mark.parametrize("tiles", [1, 64, 65, 640, 2_048, 2_049, 4_098])
def test_csv_small_capacity_stays_in_its_workspace(tiles, cap):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    oracle.lib()
    print(f"[csv workspace] tiles={tiles} cap={cap}", flush=True)
    rows = [b"k%05d,2021-05-09 00:00:%02d,38.25,-92.5,65536,%d.5,90" % (i % 99_991, i % 60, i % 70) for i in range(5_000)]
    block = b"\n".join(rows) + b"\n"
    size = tiles * TILE - 5
    text = torch.from_numpy(np.frombuffer(block, dtype=np.uint8).copy()).cuda().repeat(size // len(block) + 1)[:size].contiguous()
    total = size // len(block) * len(rows) + block[:size % len(block)].count(b"\n")
    total += 0 if (size % len(block)) == 0 or block[size % len(block) - 1:size % len(block)] == b"\n" else 1
    (ej, et, *_), _, _ = oracle.csv_extract(block, False)

    need = _query(cvetl, size, cap)
    buf = torch.full((need + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    out = {k: torch.empty(max(1, cap), dtype=dt, device="cuda") for k, dt in cvetl.RECORD_FIELDS}
    oo = cvetl.CvRecordsOut(*((cvetl._ptr(out[k]) if cap else None) for k, _ in cvetl.RECORD_FIELDS))
    res = cvetl.new_result("cuda")
    st = cvetl.lib().cv_csv_extract(cvetl._ptr(text), size, 0, ctypes.byref(oo), None, None, cap, cvetl._ptr(res),
                                    cvetl._ptr(buf), need, cvetl._stream())
    assert st == 0
    r = cvetl.read_result(res)
    assert r["status"] == cvetl.CV_ERR_CAPACITY and r["count"] == r["required"] == total
    assert bool((buf[need:] == 0xA5).all()), "bytes behind the workspace were written"
    if cap:
        assert_exact("journey_id", host(out["journey_id"]), ej[:cap])
        assert_exact("ts_ms", host(out["ts_ms"]), et[:cap])
    # a byte less is refused
    assert cvetl.lib().cv_csv_extract(cvetl._ptr(text), size, 0, ctypes.byref(oo), None, None, cap, cvetl._ptr(res),
                                      cvetl._ptr(buf), need - 1, cvetl._stream()) == cvetl.CV_ERR_WORKSPACE
