"""The order of the distinct journey ids inside the record sort: by counting (up
to 16 384 ids), sorted chunks of 4 096 joined in one step (capacities up to
65 536) or two (up to 524 288), radix passes (capacities above), each at the
edges of its range.  The order is compared with numpy's stable sort."""
import numpy as np
import pytest

from paper_2305_07454_amd import gen

from _parity import assert_exact, host, u32

pytestmark = pytest.mark.gpu

I64 = np.iinfo(np.int64)


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_07454_amd import cvetl
    cvetl.lib()
    return cvetl


def _columns(seed, J, extra):
    """J distinct ids (the extremes of int64, small numbers and random ones
    among them), every id at least once, rows shuffled."""
    rng = np.random.default_rng(seed)
    ids = np.unique(np.concatenate([[I64.max, 0, 1, -1, I64.min][:J], rng.integers(I64.min, I64.max, J + 8)]))
    ids = rng.permutation(ids)
    keep = np.concatenate([[I64.min, I64.max, 0], ids[~np.isin(ids, [I64.min, I64.max, 0])]])[:J] if J >= 3 else ids[:J]
    jid = rng.permutation(np.concatenate([keep, keep[rng.integers(0, J, extra)]]))
    n = len(jid)
    ts = gen.T0_MS + 1000 * rng.integers(0, 50, n)
    return [jid, ts, rng.uniform(36, 40, n), rng.uniform(-95, -90, n), rng.uniform(0, 40, n).astype(np.float32)]


@pytest.mark.parametrize("J,capacity", [
    (1, 1), (2, 4096), (63, 4096), (64, 64), (65, 4097), (16_384, 16_384), (16_384, 20_000), (16_385, 16_385),
    (20_480, 65_536), (65_536, 65_536), (65_537, 65_537), (20_000, 524_288), (140_001, 524_288), (3, 600_000),
    (16_385, 600_000)])
def test_order_of_distinct_ids(cv, J, capacity):
    print(f"[dictionary] J={J} capacity={capacity}", flush=True)
    cols = _columns(J, J, J + 37)
    perm, srt, r = cv.cv_sort_records(cv.to_device(tuple(cols)), max_journeys=capacity)
    exp = np.lexsort((cols[1], cols[0]))
    assert r["count"] == J
    assert_exact("perm", u32(host(perm)), exp.astype(np.uint32))
    for (k, _), c in zip(cv.RECORD_FIELDS, cols):
        assert_exact(k, host(srt[k]), c[exp])


@pytest.mark.parametrize("spans", [False, True])
@pytest.mark.parametrize("J,capacity", [(40, 4096), (16_384, 16_384), (16_400, 20_000), (70_000, 90_000), (300, 600_000), (17_000, 600_000)])
def test_order_of_distinct_ids_with_shards(cv, J, capacity, spans):
    """Shards of uneven size (one empty); `spans`: an id in two of them."""
    print(f"[dictionary] shards J={J} capacity={capacity} spans={spans}", flush=True)
    rng = np.random.default_rng(J)
    ids = rng.permutation(np.unique(rng.integers(I64.min + 1, I64.max, J + 8))[:J])
    cuts = [0, J // 7, J // 7, J // 2, J]
    parts = []
    for a, b in zip(cuts, cuts[1:]):
        own = ids[a:b]
        parts.append(rng.permutation(np.concatenate([own, own[rng.integers(0, b - a, b - a + 3)]]) if b > a else own))
    if spans:
        parts[-1][0] = parts[0][0]
        parts[-1][1:][parts[-1][1:] == parts[0][0]] = parts[-1][-1]
    jid = np.concatenate(parts)
    n = len(jid)
    cols = [jid, gen.T0_MS + 1000 * rng.integers(0, 50, n), rng.uniform(36, 40, n), rng.uniform(-95, -90, n),
            rng.uniform(0, 40, n).astype(np.float32)]
    off_h, off_d = cv.shard_offsets([len(p) for p in parts])
    perm, srt, _, r = cv.cv_sort_records_features(cv.to_device(tuple(cols)), capacity, shard_offsets=off_d)
    exp = [a + np.lexsort((cols[1][a:b], jid[a:b])) for a, b in zip(map(int, off_h), map(int, off_h[1:]))]
    order = np.concatenate(exp)
    base = np.repeat(off_h[:-1].astype(np.int64), np.diff(off_h.astype(np.int64)))
    assert_exact("perm", u32(host(perm)), (order - base).astype(np.uint32))
    for (k, _), c in zip(cv.RECORD_FIELDS, cols):
        assert_exact(k, host(srt[k]), c[order])


@pytest.mark.parametrize("capacity", [10, 4096, 5000])
def test_more_ids_than_the_capacity(cv, capacity):
    cols = _columns(1, capacity + 1, 5)
    with pytest.raises(cv.CvError) as e:
        cv.cv_sort_records(cv.to_device(tuple(cols)), max_journeys=capacity)
    assert e.value.status == cv.CV_ERR_CAPACITY


@pytest.mark.parametrize("n,capacity", [(33_000, 131_072), (4_095, 131_072), (4_096, 131_072), (4_097, 131_072),
                                        (40_000, 600_000), (200_000, 200_000)])
@pytest.mark.parametrize("J", [1, 500, 4_000])
def test_ids_listed_by_their_bits(cv, n, capacity, J):
    """Tables of 2^18 slots and more, whose occupied slots are listed by their
    bits, with the records that give the bits room (slots / 64) and fewer."""
    print(f"[dictionary] n={n} capacity={capacity} J={J}", flush=True)
    cols = _columns(n, J, n - J)
    perm, srt, r = cv.cv_sort_records(cv.to_device(tuple(cols)), max_journeys=capacity)
    assert r["count"] == J
    assert_exact("perm", u32(host(perm)), np.lexsort((cols[1], cols[0])).astype(np.uint32))
    off = cv.shard_offsets([n // 2, n - n // 2])[1]
    perm, srt, _, r = cv.cv_sort_records_features(cv.to_device(tuple(cols)), capacity, shard_offsets=off)
    a = n // 2
    exp = np.concatenate([np.lexsort((cols[1][:a], cols[0][:a])), np.lexsort((cols[1][a:], cols[0][a:]))])
    assert_exact("perm", u32(host(perm)), exp.astype(np.uint32))
