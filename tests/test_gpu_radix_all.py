"""Sorts of few keys, whose radix passes run in one launch: sizes at the edges of
its tiles (4 096 and 8 192 keys) and of its two ranges (2^19 and 2^21 records), keys
of one to eight digits, with a 9-bit first digit, packed with their index from the
first pass or a later one; the shapes of a launch per pass beyond.  The order
equals numpy's stable order, also from several streams at once and on replays of
a captured call."""
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


def _columns(n, ids, t_bits, seed=0):
    rng = np.random.default_rng(n + t_bits + seed)
    jid = rng.integers(0, ids, n) * 11 - 5
    ts = gen.T0_MS + rng.integers(0, 1 << t_bits, n)
    return jid, ts, rng.uniform(36, 40, n), rng.uniform(-95, -90, n), rng.uniform(0, 40, n).astype(np.float32)


def _check(cv, cols, mj):
    perm, srt, r = cv.cv_sort_records(cv.to_device(cols), max_journeys=mj)
    exp = np.lexsort((cols[1], cols[0]))
    assert np.array_equal(host(perm).astype(np.int64), exp)
    assert np.array_equal(host(srt["ts_ms"]), cols[1][exp]) and np.array_equal(host(srt["lat_deg"]), cols[2][exp])
    return r


@pytest.mark.parametrize("n", [2, 4_095, 4_096, 4_097, 200_003, 1 << 19, (1 << 19) + 1, 1_000_003, 1 << 21,
                               (1 << 21) + 1])
@pytest.mark.parametrize("ids,t_bits", [(1, 3), (3, 6), (300, 8), (5, 22), (900, 40), (2, 55), (200, 56)])
def test_all_passes_in_one_launch(cv, n, ids, t_bits):
    print(f"[radix all] n={n} ids={ids} t_bits={t_bits}", flush=True)
    r = _check(cv, _columns(n, ids, t_bits), ids + 1)
    if n >= 200_003:  # (as many key bits as asked for, all offsets without a common factor)
        assert r["key_bits"] == (ids - 1).bit_length() + t_bits


@pytest.mark.parametrize("shape", range(6))
def test_a_launch_per_pass(cv, shape):
    prev = cv.cv_tuning_get("sort_shape")
    try:
        cv.cv_tuning_set("sort_shape", shape)
        print(f"[radix all] shape {shape}", flush=True)
        for ids, t_bits in ((3, 6), (300, 8), (900, 40), (200, 56)):
            _check(cv, _columns((1 << 21) + 77, ids, t_bits), ids + 1)
    finally:
        cv.cv_tuning_set("sort_shape", prev)


def test_streams_and_replays(cv):
    import torch
    n, mj = 300_001, 500
    sets = [_columns(n, 400, 20, seed=k) for k in range(4)]
    exp = [np.lexsort((c[1], c[0])) for c in sets]
    dev = [cv.to_device(c) for c in sets]
    streams = [torch.cuda.Stream() for _ in sets]
    need = cv._size(cv.lib().cv_sort_workspace_size, n, mj)
    ws = [cv.workspace(need) for _ in sets]
    torch.cuda.synchronize()
    print("[radix all] four streams", flush=True)
    for _ in range(3):
        got = []
        for d, s, w in zip(dev, streams, ws):
            with torch.cuda.stream(s):
                got.append(cv.cv_sort_records(d, max_journeys=mj, ws=w, stream=s, sync=False)[0])
        torch.cuda.synchronize()
        for g, e in zip(got, exp):
            assert np.array_equal(host(g).astype(np.int64), e)
    print("[radix all] captured", flush=True)
    d = {k: v.clone() for k, v in dev[0].items()}
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        perm = cv.cv_sort_records(d, max_journeys=mj, ws=ws[0], sync=False)[0]
    for k in range(4):
        for name in d:
            d[name].copy_(dev[k][name])
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(perm).astype(np.int64), exp[k])


@pytest.mark.parametrize("n", [1, 1_023, 1_025, (1 << 17) - 1, (1 << 17) + 1, (1 << 19) - 1, (1 << 19) + 1, 1_048_577])
@pytest.mark.parametrize("ids", [1_000, 70_000])
def test_payload_tiles(cv, n, ids):
    # interleaved ids: the payloads regrouped in tiles of 1 024, 2 048 and 4 096
    # records, read by the gather of every column and by the one with the kinematics
    import torch
    print(f"[payload] n={n} ids={ids}", flush=True)
    cols = _columns(n, ids, 12)
    exp = np.lexsort((cols[1], cols[0]))
    d = cv.to_device(cols)
    perm, srt, _ = cv.cv_sort_records(d, max_journeys=ids + 1)
    fperm, fsrt, feat, _ = cv.cv_sort_records_features(d, ids + 1)
    for p, s in ((perm, srt), (fperm, fsrt)):
        assert np.array_equal(host(p).astype(np.int64), exp)
        for k, c in zip(("journey_id", "ts_ms", "lat_deg", "lon_deg", "speed_mps"), cols):
            assert np.array_equal(host(s[k]), c[exp]), k
    off, off_d = cv.shard_offsets([n // 3, 0, n - n // 3])
    sperm, ssrt, _, _ = cv.cv_sort_records_features(d, 2 * ids + 2, shard_offsets=off_d)
    a = n // 3
    lo, hi = np.lexsort((cols[1][:a], cols[0][:a])), np.lexsort((cols[1][a:], cols[0][a:]))
    assert np.array_equal(host(sperm).astype(np.int64), np.concatenate([lo, hi]))
    assert np.array_equal(host(ssrt["lon_deg"]), np.concatenate([cols[3][:a][lo], cols[3][a:][hi]]))
