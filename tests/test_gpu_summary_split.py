"""The journey summary at the edges of its tiles and of the ranges of its three
splits (windows of 64 records per wave), and in the coarsest split that a
workspace without room for the finer ones gets.  Counts, sums, maxima and
boxes are compared with numpy; distances are sums of whole metres, so exact."""
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


def _case(seed, n, mean):
    """Sorted records and features (whole steps, so every sum is exact in float64)."""
    rng = np.random.default_rng(seed)
    head = rng.random(n) < 1.0 / mean
    head[0] = True
    jid = np.cumsum(head) * 7
    cols = [jid, gen.T0_MS + np.arange(n) * 1000, rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
            rng.integers(0, 40, n).astype(np.float32)]
    flags = np.where(head, 1, 4 + 2 * (rng.random(n) < 0.1)).astype(np.uint8)
    feat = dict(step_m=rng.integers(0, 50, n).astype(np.float64), speed_mps=rng.uniform(0, 30, n), flags=flags)
    return cols, feat, head


def _check(cv, cols, feat, head, got, count):
    at = np.nonzero(head)[0]
    assert count == len(at)
    add = np.add.reduceat
    exp = dict(journey_id=cols[0][at], first=at, n_points=np.diff(np.append(at, len(head))), distance_m=add(feat["step_m"], at),
               sum_speed=add(cols[4].astype(np.float64), at), max_speed=np.maximum.reduceat(cols[4], at),
               max_derived_speed=np.maximum.reduceat(np.where(feat["flags"] & 4, feat["speed_mps"], 0.0), at),
               n_dt_zero=add((feat["flags"] >> 1 & 1).astype(np.int64), at),
               t_start_ms=cols[1][at], t_end_ms=cols[1][np.append(at[1:], len(head)) - 1],
               lat_min=np.minimum.reduceat(cols[2], at), lat_max=np.maximum.reduceat(cols[2], at),
               lon_min=np.minimum.reduceat(cols[3], at), lon_max=np.maximum.reduceat(cols[3], at))
    for k, e in exp.items():
        assert np.array_equal(host(got[k]).astype(e.dtype), e), k


@pytest.mark.parametrize("n,mean", [(1, 5), (63, 5), (511, 1000), (512, 3), (513, 1000), (2047, 40), (2048, 5000), (2049, 5000),
                                    (100_003, 90), (4_194_304, 2000), (4_194_305, 2000), (33_554_433, 30_000)])
def test_summary_split(cv, n, mean):
    import torch
    print(f"[summary] n={n}", flush=True)
    cols, feat, head = _case(n, n, mean)
    srt = cv.to_device(tuple(cols))
    ft = {k: torch.from_numpy(v).cuda() for k, v in feat.items()}
    got, r = cv.cv_journey_summary(srt, ft, capacity=int(head.sum()))
    _check(cv, cols, feat, head, got, r["count"])


def test_summary_in_the_least_workspace(cv):
    """One size that only the coarsest split fits (three words per 16 384 records and 152 bytes per row, all rounded to 256)."""
    import torch
    n = 300_001
    cols, feat, head = _case(9, n, 400)
    J = int(head.sum())
    tiles = -(-n // 16384)
    up = lambda b: -(-b // 256) * 256  # noqa: E731
    need = up(4) + up(16 * tiles) + 2 * up(4 * tiles + 4) + up(104 * J) + up(48 * J)
    srt = cv.to_device(tuple(cols))
    ft = {k: torch.from_numpy(v).cuda() for k, v in feat.items()}
    out = {k: torch.empty(J, dtype=dt, device="cuda") for k, dt in cv.JOURNEY_FIELDS}
    import ctypes
    js = cv.CvJourneys(*(cv._ptr(out[k]) for k, _ in cv.JOURNEY_FIELDS))
    call = lambda ws, res: cv.lib().cv_journey_summary(  # noqa: E731
        ctypes.byref(cv._records_struct(srt)), ctypes.byref(cv._feat_struct(ft)), ctypes.byref(js), J, cv._ptr(res),
        cv._ptr(ws), ws.numel(), cv._stream())
    res = cv.new_result()
    assert call(cv.workspace(need - 256), res) == cv.CV_ERR_WORKSPACE
    assert call(cv.workspace(need), res) == 0
    _check(cv, cols, feat, head, out, cv.read_result(res)["count"])
