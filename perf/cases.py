"""The work that programs give this package, as cases that can be timed.

Each case goes through the package's public entry points as its users call
them: the preallocated pipelines (one batch of journeys, many shards), the
four calls that allocate and read their results, the lattice with
directions, the dense lattice with its normalisation and filter, record
hygiene, text extraction, and a serving session.  Inputs have the shape of
`paper_2305_07454_amd.gen` (Missouri box, 1 Hz random walks, lognormal journey
lengths, a 5 % share of duplicated and 2 % of swapped time stamps, feeds in
time order), drawn on the GPU; positions are whole multiples of 2^-40 degrees,
so that every sum below is exact and a seed gives the same bits each time.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2305_07454_amd import cvetl, gen, tune

DEV = "cuda"
UNIT = 2.0 ** -40           # degrees per position step
MEAN_JOURNEY = 2470         # records of a journey: lognormal, median 1 500, sigma 1
EARTH_R_M = 6371008.8
RECORD, FEATURES, JOURNEY, GROUP = 36, 49, 100, 32  # bytes per row


def listed():
    """The cases, smallest calls first."""
    return [
        # one vehicle fleet's files through the four calls, which allocate and read back: launches and latency
        dict(name="oneshot_small", kind="oneshot", records=33_265, mean=1386, layout="files", grid="c1"),
        # 2 000 short journeys, every row shuffled, 0.01 deg x 15 min
        dict(name="plain_shuffled", kind="plain", records=1_000_000, mean=500, layout="shuffled", grid="c0"),
        # a tenth of a state's day, journey files in random order, 0.005 deg x 5 min
        dict(name="plain_tenth", kind="plain", records=12_345_679, mean=MEAN_JOURNEY, layout="files", grid="c1"),
        # a state's full day: 50 000 journeys
        dict(name="plain_day", kind="plain", records=123_456_789, mean=MEAN_JOURNEY, layout="files", grid="c1"),
        # an hour of counties: few records in many uneven shards, 0.001 deg x 1 min
        dict(name="batch_hour", kind="batch", records=2_000_003, shards=40, grid="c2"),
        # county-day files of a state in one batch: 115 shards, half of the 400 M record workload
        dict(name="batch_days", kind="batch", records=200_000_000, shards=115, grid="c2"),
        # the lattice per cardinal direction from a sensor heading
        dict(name="directions", kind="directions", records=24_000_001, n_dir=4, source="heading", grid="c1"),
        # a day's groups as a dense tensor, normalised per channel, and filtered
        dict(name="lattice_day", kind="lattice", groups=1_550_000, n_t=288, n_dir=0, grid="c1"),
        # duplicate rows dropped and trips split at one-minute gaps
        dict(name="hygiene", kind="hygiene", records=40_000_000),
        # a small upload of hand-made text: fields of uneven width, empty headings, read back at once
        dict(name="csv_ragged", kind="csv", rows=50_000, ragged=True),
        # fixed-width text, the extraction's bulk form
        dict(name="csv_bulk", kind="csv", rows=4_000_000, ragged=False),
        # a serving session: pushes of uneven chunks into resident state, then a flush
        dict(name="serve_session", kind="serve", records=4_000_000, pushes=8, heavy=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["oneshot", "plain", "plain", "plain", "batch", "batch", "directions", "lattice", "hygiene",
                       "csv", "serve"])
    if kind == "oneshot":
        return dict(kind=kind, records=_log(rng, 5_000, 2_000_000), mean=_log(rng, 300, 3000),
                    layout=rng.choice(["files", "shuffled", "feed"]), grid=rng.choice(["c0", "c1", "c2"]))
    if kind == "plain":
        return dict(kind=kind, records=_log(rng, 50_000, 100_000_000), mean=_log(rng, 300, 3000),
                    layout=rng.choice(["files", "files", "shuffled", "feed"]), grid=rng.choice(["c0", "c1", "c1"]))
    if kind == "batch":
        return dict(kind=kind, records=_log(rng, 200_000, 150_000_000), shards=rng.randint(2, 115), grid="c2")
    if kind == "directions":
        return dict(kind=kind, records=_log(rng, 100_000, 40_000_000), n_dir=rng.choice([4, 4, 8, 12]),
                    source=rng.choice(["heading", "bearing"]), grid=rng.choice(["c0", "c1"]))
    if kind == "lattice":
        n_dir = rng.choice([0, 0, 4])
        return dict(kind=kind, groups=_log(rng, 50_000, 2_000_000), n_t=rng.randint(24, 96 if n_dir else 288),
                    n_dir=n_dir, grid="c1")
    if kind == "hygiene":
        return dict(kind=kind, records=_log(rng, 50_000, 60_000_000))
    if kind == "csv":
        return dict(kind=kind, rows=_log(rng, 5_000, 6_000_000), ragged=rng.random() < 0.5)
    return dict(kind="serve", records=_log(rng, 200_000, 8_000_000), pushes=rng.randint(3, 16),
                heavy=rng.random() < 0.3)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _generator(seed, part):
    g = torch.Generator(DEV)
    g.manual_seed((seed * 1_000_003 + part) & 0x7FFF_FFFF_FFFF)
    return g


def _split(rng, n, count, weights, cap=None):
    """`count` lengths of at least 1 in proportion to the weights, summing to n."""
    length = np.maximum(1, np.floor(weights / weights.sum() * n).astype(np.int64))
    if cap:
        length = np.minimum(length, cap)
    for _ in range(64):
        left = n - int(length.sum())
        if left == 0:
            break
        at = rng.permutation(count)[:abs(left)]
        if left > 0:
            length[at] += max(1, left // count)
        else:
            length[at] -= (length[at] > 1)
    assert int(length.sum()) == n
    return length


def _lengths(rng, n, mean, layout):
    count = max(1, n // mean)
    if layout == "shuffled":
        return _split(rng, n, count, rng.integers(100, 901, count).astype(np.float64))
    return _split(rng, n, count, rng.lognormal(0.0, 1.0, count), 86_400 if mean < 40_000 else None)


def _ids(g, count):
    """Distinct random non-negative 63-bit ids."""
    ids = torch.randint(0, 2 ** 63 - 1, (count,), device=DEV, generator=g)
    assert torch.unique(ids).numel() == count
    return ids


def _fold(free, width):
    """Integer walk reflected into [0, width)."""
    m = torch.remainder(free, 2 * width)
    return (width - (m - width).abs()).clamp_(0, width - 1)


def _speeds(g, n):
    s = torch.rand(n, device=DEV, generator=g) * 40.0
    s.clamp_(max=float(np.nextafter(np.float32(40), np.float32(0))))
    s[torch.rand(n, device=DEV, generator=g) < 0.05] = 0.0
    return s


def _walks(g, lengths, ids, period=None, start=None):
    """Journeys one after the other, each a random walk in time order."""
    length = torch.as_tensor(lengths, device=DEV)
    end = length.cumsum(0)
    head = end - length
    n, count = int(end[-1]), length.numel()
    which = torch.repeat_interleave(torch.arange(count, device=DEV), length)
    pos = torch.arange(n, device=DEV) - head[which]
    step_ms = torch.full((count,), 1000, device=DEV) if period is None else period
    if start is None:
        slack = ((gen.DAY_MS - (length - 1) * step_ms) // 1000).clamp_(min=1)
        start = 1000 * (torch.rand(count, device=DEV, generator=g, dtype=torch.float64) * slack).long()
    ts = gen.T0_MS + start[which] + step_ms[which] * pos
    coords = []
    for lo, hi in ((gen.LAT_LO, gen.LAT_HI), (gen.LON_LO, gen.LON_HI)):
        width = int((hi - lo) / UNIT)
        d = (torch.randn(n, device=DEV, generator=g) * (gen.WALK_SIGMA_DEG / UNIT)).long()
        d[head] = (torch.rand(count, device=DEV, generator=g, dtype=torch.float64) * width).long()
        c = d.cumsum(0)
        free = c - (c[head] - d[head])[which]
        coords.append(lo + _fold(free, width).double() * UNIT)
    rec = dict(journey_id=ids[which], ts_ms=ts, lat_deg=coords[0], lon_deg=coords[1], speed_mps=_speeds(g, n))
    return rec, head, length, which


def _take(rec, order):
    return {k: v[order] for k, v in rec.items()}


def _block_order(g, head, length):
    """Row order that puts whole journeys in random order."""
    p = torch.rand(length.numel(), device=DEV, generator=g).argsort(stable=True)
    size = length[p]
    at = size.cumsum(0) - size
    return torch.repeat_interleave(head[p] - at, size) + torch.arange(int(size.sum()), device=DEV)


def _not_adjacent(g, n, share):
    m = torch.rand(n, device=DEV, generator=g) < share
    m[1:] &= ~m[:-1].clone()
    return m


def _pick(g, mask, count):
    """`count` of the mask's positions, at random (every seed then gives tables of one size)."""
    at = mask.nonzero()[:, 0]
    assert at.numel() >= count
    return at[torch.rand(at.numel(), device=DEV, generator=g).argsort(stable=True)[:count]]


def _feed_order(g, ts, shard=None):
    """By (shard,) time stamp, ties in random order."""
    key = ((ts - gen.T0_MS) << 24) | torch.randint(0, 1 << 24, ts.shape, device=DEV, generator=g)
    if shard is not None:
        key |= shard << 56
    return torch.sort(key, stable=True)[1]


def _plain_records(case, seed):
    g = _generator(seed, 1)
    lengths = _lengths(np.random.default_rng(seed), case["records"], case["mean"], case["layout"])
    rec, head, length, _ = _walks(g, lengths, _ids(g, len(lengths)))
    n = case["records"]
    if case["layout"] == "feed":
        return _take(rec, _feed_order(g, rec["ts_ms"])), len(lengths)
    if case["layout"] == "shuffled":
        return _take(rec, torch.rand(n, device=DEV, generator=g, dtype=torch.float64).argsort(stable=True)), len(lengths)
    first = torch.zeros(n, dtype=torch.bool, device=DEV)
    first[head] = True
    dup = ((torch.rand(n, device=DEV, generator=g) < 0.05) & ~first).nonzero()[:, 0]
    before = rec["ts_ms"][dup - 1]
    rec["ts_ms"][dup] = before
    swap = _not_adjacent(g, n, 0.02)
    swap[head + length - 1] = False
    a = swap.nonzero()[:, 0]
    order = torch.arange(n, device=DEV)
    order[a], order[a + 1] = a + 1, a
    return _take(rec, order[_block_order(g, head, length)]), len(lengths)


def _batch_records(case, seed):
    """County-day shards: Zipf(1.2) sizes, Poisson journey counts, each shard a feed in time order."""
    n, shards = case["records"], case["shards"]
    rng = np.random.default_rng(seed)
    w = np.minimum(np.arange(1, shards + 1) ** -1.2, 3.0 / shards ** 0.9)
    sizes = _split(rng, n, shards, w)[rng.permutation(shards)]
    parts, owner = [], []
    for s, size in enumerate(sizes):
        count = min(int(size), max(1, int(rng.poisson(size / 1200.0))))
        parts.append(_split(rng, int(size), count, rng.lognormal(0.0, 1.0, count)))
        owner.append(np.full(count, s))
    g = _generator(seed, 2)
    lengths = np.concatenate(parts)
    rec, _, _, which = _walks(g, lengths, _ids(g, len(lengths)))
    shard = torch.as_tensor(np.concatenate(owner), device=DEV)[which]
    return _take(rec, _feed_order(g, rec["ts_ms"], shard)), [int(x) for x in sizes], len(lengths)


def _sorted_records(case, seed, part, gaps=False):
    """Records already in (journey, time) order, with the order they came in as `perm`."""
    g = _generator(seed, part)
    n = case["records"]
    lengths = _lengths(np.random.default_rng(seed), n, min(MEAN_JOURNEY, n), "files")
    rec, head, length, which = _walks(g, lengths, torch.sort(_ids(g, len(lengths)))[0])
    first = torch.zeros(n, dtype=torch.bool, device=DEV)
    first[head] = True
    dup = ((torch.rand(n, device=DEV, generator=g) < 0.05) & ~first).nonzero()[:, 0]
    before = rec["ts_ms"][dup - 1]
    rec["ts_ms"][dup] = before
    if gaps:
        # pauses: of less than a minute (a trip goes on) and of more
        inside = _not_adjacent(g, n, 0.05) & ~first
        inside[head + length - 1] = False
        at = _pick(g, inside, 2 * (n // 1500))
        jump = torch.zeros(n, dtype=torch.long, device=DEV)
        jump[at[::2]] = torch.randint(30_000, 50_000, at[::2].shape, device=DEV, generator=g)
        jump[at[1::2]] = torch.randint(90_000, 1_800_000, at[1::2].shape, device=DEV, generator=g)
        c = jump.cumsum(0)
        rec["ts_ms"] += c - c[head][which]
        same = _pick(g, _not_adjacent(g, n, 0.05) & ~first, n // 100)
        for k in ("ts_ms", "lat_deg", "lon_deg", "speed_mps"):
            copied = rec[k][same - 1]
            rec[k][same] = copied
    perm = _block_order(g, head, length)
    inverse = torch.empty_like(perm)
    inverse[perm] = torch.arange(n, device=DEV)
    return rec, inverse.int(), head, which, g


def _serve_records(case, seed):
    """A feed of open journeys; `heavy`: one in a hundred sampled at 20 Hz with three tenths of the records."""
    n = case["records"]
    rng = np.random.default_rng(seed)
    count = max(8, n // MEAN_JOURNEY)
    w = rng.lognormal(0.0, 1.0, count)
    period = np.full(count, 1000)
    if case["heavy"]:
        hv = rng.permutation(count)[:max(1, count // 100)]
        w[hv] *= (0.3 / 0.7) * (w.sum() - w[hv].sum()) / w[hv].sum()
        period[hv] = 50
    lengths = _split(rng, n, count, w)
    g = _generator(seed, 4)
    start = torch.as_tensor(1000 * rng.integers(0, 1500, count), device=DEV)
    rec, _, _, _ = _walks(g, lengths, _ids(g, count), torch.as_tensor(period, device=DEV), start)
    cuts = np.sort(rng.permutation(n - 1)[:case["pushes"] - 1] + 1)
    return _take(rec, _feed_order(g, rec["ts_ms"])), [0, *map(int, cuts), n], count


def _digits(v, width):
    p = 10 ** torch.arange(width - 1, -1, -1, device=DEV)
    return ((v[:, None] // p) % 10 + 48).to(torch.uint8)


def _csv_values(case, seed):
    g = _generator(seed, 5)
    n = case["rows"]
    r = lambda lo, hi: torch.randint(lo, hi, (n,), device=DEV, generator=g)  # noqa: E731
    v = dict(journey=r(0, 67_600_000), ms=r(0, gen.DAY_MS), lat=r(36_000_000, 40_600_000),
             lon=r(89_100_000, 95_800_000), speed=r(0, 4000), heading=r(0, 360), postal=r(63_000, 66_000))
    if case["ragged"]:
        v["ms"] = v["ms"] // 1000 * 1000
    v["blank"] = r(0, 20) == 0 if case["ragged"] else torch.zeros(n, dtype=torch.bool, device=DEV)
    return v


def _csv_text(case, v):
    """Text rows of seven fields; ragged rows leave out signs, leading zeros, whole-second fractions and some headings."""
    n, ragged = case["rows"], case["ragged"]
    cols, keep = [], []

    def put(block, kept=None):
        cols.append(block)
        keep.append(torch.ones(block.shape, dtype=torch.bool, device=DEV) if kept is None else kept)

    def char(c, kept=None):
        put(torch.full((n, 1), ord(c), dtype=torch.uint8, device=DEV), None if kept is None else kept[:, None])

    def number(whole, width):
        d = _digits(whole, width)
        seen = (d != 48).cumsum(1) > 0
        seen[:, -1] = True
        put(d, seen if ragged else None)

    none = torch.zeros(n, dtype=torch.bool, device=DEV)
    put(_digits(v["journey"] % 100_000, 5))
    put((97 + torch.stack([v["journey"] // 100_000 % 26, v["journey"] // 2_600_000], 1)).to(torch.uint8))
    for c in ",2021-05-09 ":
        char(c)
    s = v["ms"] // 1000
    for i, part in enumerate((s // 3600, s // 60 % 60, s % 60)):
        if i:
            char(":")
        put(_digits(part, 2))
    char(".", none if ragged else None)
    put(_digits(v["ms"] % 1000, 3), none[:, None].expand(n, 3) if ragged else None)
    for sign, q in (("+", v["lat"]), ("-", v["lon"])):
        char(",")
        char(sign, none if ragged and sign == "+" else None)
        number(q // 1_000_000, 3)
        char(".")
        put(_digits(q % 1_000_000, 6))
    char(",")
    put(_digits(v["postal"], 5))
    char(",")
    number(v["speed"] // 100, 3)
    char(".")
    put(_digits(v["speed"] % 100, 2))
    char(",")
    d, m = _digits(v["heading"], 3), None
    if ragged:
        m = (d != 48).cumsum(1) > 0
        m[:, -1] = True
        m &= ~v["blank"][:, None]
    put(d, m)
    char("\n")
    header = torch.frombuffer(bytearray(gen.CSV_HEADER), dtype=torch.uint8).to(DEV)
    body = torch.cat(cols, 1)
    return torch.cat([header, body[torch.cat(keep, 1)] if ragged else body.reshape(-1)])


def _groups(case, seed):
    """A group table: cells in clusters, as vehicles visit them."""
    grid, g, count = gen.GRIDS[case["grid"]], _generator(seed, 6), case["groups"]
    D = case["n_dir"] + 1 if case["n_dir"] else 1
    m = 2 * count // 8 + 64
    r = lambda hi, k: torch.randint(0, hi, (k,), device=DEV, generator=g)  # noqa: E731
    t, d, la, lo = (r(hi, m).repeat_interleave(8) for hi in (case["n_t"], D, grid.n_lat - 8, grid.n_lon - 8))
    key = torch.unique((((t * D) + d) * grid.n_lat + la + r(8, 8 * m)) * grid.n_lon + lo + r(8, 8 * m))
    key = key[torch.rand(key.numel(), device=DEV, generator=g).argsort(stable=True)[:count]].sort()[0]
    n = key.numel()
    assert n == count
    # one cell in five is slow with two vehicles or more; of the others half have a single vehicle
    turn = torch.rand(n, device=DEV, generator=g).argsort(stable=True)
    slow, single = turn < n // 5, turn >= 3 * n // 5
    volume = 2 + (torch.rand(n, device=DEV, generator=g) ** 4 * 40).int()
    volume[single] = 1
    num = volume * (1 + r(60, n)).int()
    mean = torch.rand(n, device=DEV, generator=g)
    mean = torch.where(slow, mean * 9.9, torch.where(single, mean * 38, 10.1 + mean * 28))
    return dict(key=key, count=num, n_journeys=volume, sum_speed=num.double() * mean.double(),
                min_speed=mean * 0.5, max_speed=mean + 1)


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _capacity(n, grid):
    return 4096 + (n // 2 if grid == "c2" else n // 6)


def _journey_capacity(case):
    return case["records"] // 1000 + 40 * case["shards"] + 64


def _table(fields, rows):
    """A program's own table: rows that a pass does not fill stay zero."""
    return {k: torch.zeros(rows, dtype=dt, device=DEV) for k, dt in fields}


def _zeroed(*tables):
    for t in tables:
        for v in t.values():
            v.zero_()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "csv":
        text = _csv_text(case, _csv_values(case, seed))
        if case["ragged"]:
            return dict(kind=kind, text=text)
        n = case["rows"]
        out = _table(cvetl.RECORD_FIELDS, n)
        need = cvetl._size(cvetl.lib().cv_csv_workspace_size, text.numel(), n)
        return dict(kind=kind, text=text, out=out, heading=torch.zeros(n, device=DEV), rows=n,
                    ok=torch.zeros(n, dtype=torch.uint8, device=DEV), ws=cvetl.workspace(need))
    if kind == "lattice":
        grid, C = gen.GRIDS[case["grid"]], cvetl.lattice_channels(case["n_dir"])
        return dict(kind=kind, case=case, grid=grid, groups=_groups(case, seed),
                    tensor=torch.empty((case["n_t"], C, grid.n_lat, grid.n_lon), device=DEV),
                    minmax=torch.empty(2 * C, device=DEV))
    tune.apply(case["records"])
    if kind == "oneshot":
        rec, _ = _plain_records(case, seed)
        return dict(kind=kind, rec=rec, grid=gen.GRIDS[case["grid"]],
                    groups=_table(cvetl.GROUP_FIELDS, _capacity(case["records"], case["grid"])))
    if kind == "plain":
        rec, count = _plain_records(case, seed)
        pipe = cvetl.Pipeline(case["records"], gen.GRIDS[case["grid"]], count, count,
                              _capacity(case["records"], case["grid"]))
        _zeroed(pipe.journeys, pipe.groups)
        return dict(kind=kind, rec=rec, pipe=pipe)
    if kind == "batch":
        rec, sizes, _ = _batch_records(case, seed)
        cap = _journey_capacity(case)
        pipe = cvetl.BatchPipeline(case["records"], len(sizes), gen.GRIDS[case["grid"]], cap, cap,
                                   _capacity(case["records"], case["grid"]))
        _zeroed(pipe.journeys, pipe.groups)
        return dict(kind=kind, rec=rec, pipe=pipe, offsets=cvetl.shard_offsets(sizes)[1])
    if kind == "directions":
        rec, perm, head, which, g = _sorted_records(case, seed, 3)
        n, grid = case["records"], gen.GRIDS[case["grid"]]
        cap = _capacity(n, case["grid"])
        out = _table(cvetl.GROUP_FIELDS, cap)
        need = cvetl._size(cvetl.lib().cv_grid_workspace_size, n, ctypes.byref(cvetl._spec_struct(grid)), cap)
        state = dict(kind=kind, case=case, rec=rec, perm=perm, grid=grid, out=out, ws=cvetl.workspace(need))
        if case["source"] == "heading":
            turn = (torch.randn(n, device=DEV, generator=g) * 512).long()
            turn[head] = torch.randint(0, 360 * 256, (head.numel(),), device=DEV, generator=g)
            c = turn.cumsum(0)
            deg = torch.remainder(c - (c[head] - turn[head])[which], 360 * 256) // 256
            column = torch.empty(n, device=DEV)
            column[perm.long()] = deg.float()
            state.update(column=column, sorted_column=torch.empty_like(column))
        else:
            state["feat"] = cvetl.cv_journey_features(rec)
        return state
    if kind == "hygiene":
        rec, perm = _sorted_records(case, seed, 7, gaps=True)[:2]
        return dict(kind=kind, rec=rec, perm=perm)
    rec, cuts, count = _serve_records(case, seed)
    n = case["records"]
    feat = {k: torch.empty(n, dtype=dt, device=DEV) for k, dt in cvetl.FEATURE_FIELDS}
    part = lambda d, a, b: {k: v[a:b] for k, v in d.items()}  # noqa: E731
    results = torch.zeros(len(cuts) - 1, 64, dtype=torch.uint8, device=DEV)
    chunks = [(part(rec, a, b), part(feat, a, b), results[i]) for i, (a, b) in enumerate(zip(cuts, cuts[1:]))]
    return dict(kind=kind, grid=gen.GRIDS["c4" if case["heavy"] else "c3"], chunks=chunks, feat=feat, results=results,
                journeys=count, table=_table(cvetl.GROUP_FIELDS, n // 3 + 4096),
                largest=max(b - a for a, b in zip(cuts, cuts[1:])))


def run(state):
    kind = state["kind"]
    if kind == "oneshot":
        perm, rec, _ = cvetl.cv_sort_records(state["rec"])
        feat = cvetl.cv_journey_features(rec)
        summary, _ = cvetl.cv_journey_summary(rec, feat)
        groups = state["groups"]
        _, r = cvetl.cv_grid_aggregate(rec, state["grid"], capacity=groups["key"].numel(), out=groups,
                                       flags=feat["flags"])
        return dict(perm=perm, sorted=rec, features=feat, summary=summary, groups=groups, count=r["count"],
                    n_out=r["n_out_of_grid"])
    if kind == "plain":
        p = state["pipe"]
        p.run(state["rec"])
        return dict(perm=p.perm, sorted=p.sorted, features=p.feat, summary=p.journeys, groups=p.groups, results=p.res)
    if kind == "batch":
        p = state["pipe"]
        p.run(state["rec"], state["offsets"])
        return dict(perm=p.perm, sorted=p.sorted, features=p.feat, summary=p.journeys, groups=p.groups,
                    journey_offsets=p.journey_offsets, group_offsets=p.group_offsets, out=p.shard_n_out, results=p.res)
    if kind == "directions":
        n_dir, heading = state["case"]["n_dir"], None
        if "column" in state:
            heading = cvetl.cv_gather_column(state["column"], state["perm"], out=state["sorted_column"])
        groups, res = cvetl.cv_grid_aggregate_dir(
            state["rec"], state["grid"], n_dir, 180.0 / n_dir, heading=heading, feat=state.get("feat"),
            capacity=state["out"]["key"].numel(), sync=False, ws=state["ws"], out=state["out"])
        return dict(heading=heading, groups=groups, result=res)
    if kind == "lattice":
        c = state["case"]
        t = cvetl.cv_lattice_dense(state["groups"], state["grid"], c["n_dir"], 0, c["n_t"], out=state["tensor"])
        t, minmax = cvetl.cv_lattice_normalize(t, state["grid"], c["n_dir"], minmax=state["minmax"])
        kept, _ = cvetl.cv_groups_filter(state["groups"], 2, 0.0, 10.0)
        return dict(tensor=t, minmax=minmax, kept=kept)
    if kind == "hygiene":
        kept, perm, _ = cvetl.cv_drop_duplicates(state["rec"], state["perm"])
        trip, journey, _ = cvetl.cv_split_trips(kept, 60_000)
        return dict(kept=kept, perm=perm, trip=trip, journey=journey)
    if kind == "csv":
        if "out" not in state:
            rec, heading, ok, _ = cvetl.cv_csv_extract(state["text"])
            return dict(records=rec, heading=heading, ok=ok)
        rec, heading, ok, res = cvetl.cv_csv_extract(state["text"], capacity=state["rows"], out=state["out"],
                                                     heading=state["heading"], row_ok=state["ok"], ws=state["ws"],
                                                     sync=False)
        return dict(records=rec, heading=heading, ok=ok, result=res)
    table = state["table"]
    rows = table["key"].numel()
    st = cvetl.Stream(state["grid"], state["journeys"], rows, state["largest"])
    for rec, feat, res in state["chunks"]:
        st.push(rec, feat, res)
    journeys, groups, _, _ = st.flush(state["journeys"], rows)
    st.close()
    for k, v in groups.items():  # into the program's own table
        table[k][:v.numel()].copy_(v)
    return dict(features=state["feat"], summary=journeys, groups=table, results=state["results"])


def work(case):
    """Bytes of one pass: every input once, every output once (group counts as these inputs give them)."""
    kind = case["kind"]
    if kind == "csv":
        return dict(bytes=case["rows"] * ((62 if case["ragged"] else 73) + RECORD + 5), flops=0)
    if kind == "lattice":
        grid = gen.GRIDS[case["grid"]]
        tensor = case["n_t"] * cvetl.lattice_channels(case["n_dir"]) * grid.n_lat * grid.n_lon
        return dict(bytes=6 * tensor + 40 * case["groups"], flops=0)
    n = case["records"]
    if kind == "directions":
        return dict(bytes=n * (RECORD + (12 if case["source"] == "heading" else 9)) + n // 60 * GROUP, flops=0)
    if kind == "hygiene":
        return dict(bytes=n * (2 * (RECORD + 4) + 24), flops=0)
    groups = n // 8 if case.get("grid") == "c2" or case.get("heavy") else n // 60
    journeys = n // case.get("mean", 1200 if kind == "batch" else MEAN_JOURNEY)
    perm = 0 if kind == "serve" else 4 + RECORD
    return dict(bytes=n * (RECORD + perm + FEATURES) + groups * GROUP + journeys * JOURNEY, flops=0)


# ---------------------------------------------------------------------------
# the same values by plain torch in 64 bits
# ---------------------------------------------------------------------------

def _over(x, c):
    """x / c, divided (torch multiplies by the reciprocal of a number)."""
    return x / torch.full((), float(c), dtype=torch.float64, device=DEV)


def _order(jid, ts, shard=None):
    order = torch.sort(ts, stable=True)[1]
    for col in (jid, shard):
        if col is not None:
            order = order[torch.sort(col[order], stable=True)[1]]
    return order


def _kinematics(r, first):
    ts, rad = r["ts_ms"], math.pi / 180.0
    lat, lon = r["lat_deg"], r["lon_deg"]
    before = lambda x: torch.cat([x[:1], x[:-1]])  # noqa: E731
    on = ~first
    dt = torch.where(on, ts - before(ts), 0)
    phi, phi0 = lat * rad, before(lat) * rad
    half = 0.5 * rad * (lat - before(lat))
    sl, cl = torch.sin(0.5 * rad * (lon - before(lon))), torch.cos(0.5 * rad * (lon - before(lon)))
    a = torch.sin(half) ** 2 + torch.cos(phi) * torch.cos(phi0) * sl ** 2
    step = torch.where(on, 2 * EARTH_R_M * torch.asin(a.sqrt().clamp_(max=1.0)), 0.0)
    secs = _over(dt.double(), 1000)
    moving = on & (dt > 0)
    speed = torch.where(moving, step / secs, 0.0)
    y = 2 * sl * cl * torch.cos(phi)
    x = 2 * torch.sin(half) * torch.cos(half) + 2 * torch.sin(phi0) * torch.cos(phi) * sl ** 2
    turned = step > 0
    bearing = torch.where(turned, torch.remainder(torch.atan2(y, x) / rad, 360.0), 0.0)
    both = moving & before(moving)
    accel = torch.where(both, (speed - before(speed)) / secs, 0.0)
    d = bearing - before(bearing)
    d = torch.where(d > 180, d - 360, torch.where(d <= -180, d + 360, d))
    return dict(step_m=step, dt_s=secs, speed_mps=speed, accel_mps2=accel, bearing_deg=bearing,
                dheading_deg=torch.where(turned & before(turned), d, 0.0)), moving, turned


def _pad(v, size):
    return v if size is None else torch.cat([v, torch.zeros(size - v.numel(), dtype=v.dtype, device=DEV)])


def _journey_rows(r, f, moving, first, size):
    j = first.long().cumsum(0) - 1
    count = int(j[-1]) + 1
    tot = lambda v: torch.zeros(count, dtype=torch.float64, device=DEV).index_add_(0, j, v.double())  # noqa: E731
    red = lambda v, how, z: torch.full((count,), z, dtype=v.dtype, device=DEV).scatter_reduce_(0, j, v, how)  # noqa: E731
    inf = math.inf
    rows = dict(distance_m=tot(f["step_m"]), sum_speed=tot(r["speed_mps"]), max_speed=red(r["speed_mps"], "amax", -inf),
                max_derived_speed=red(torch.where(moving, f["speed_mps"], 0.0), "amax", 0.0),
                lat_min=red(r["lat_deg"], "amin", inf), lat_max=red(r["lat_deg"], "amax", -inf),
                lon_min=red(r["lon_deg"], "amin", inf), lon_max=red(r["lon_deg"], "amax", -inf))
    return {k: _pad(rows[k], size) if k in rows else None for k, _ in cvetl.JOURNEY_FIELDS}


def _group_rows(r, grid, size, shard=None, sector=None, sectors=1):
    key = torch.div(r["ts_ms"] - grid.t0_ms, grid.bin_ms, rounding_mode="floor")
    if sector is not None:
        key = key * sectors + sector
    key = key * grid.n_lat + torch.floor(_over(r["lat_deg"] - grid.lat0_deg, grid.dlat_deg)).long()
    key = key * grid.n_lon + torch.floor(_over(r["lon_deg"] - grid.lon0_deg, grid.dlon_deg)).long()
    if shard is not None:
        key = key + shard * (grid.n_t * grid.n_lat * grid.n_lon)
    uniq, at = torch.unique(key, return_inverse=True)
    count, spd = uniq.numel(), r["speed_mps"]
    rows = dict(sum_speed=torch.zeros(count, dtype=torch.float64, device=DEV).index_add_(0, at, spd.double()),
                min_speed=torch.full((count,), math.inf, device=DEV).scatter_reduce_(0, at, spd, "amin"),
                max_speed=torch.full((count,), -math.inf, device=DEV).scatter_reduce_(0, at, spd, "amax"))
    return {k: _pad(rows[k], size) if k in rows else None for k, _ in cvetl.GROUP_FIELDS}


def exact(case, seed):
    kind = case["kind"]
    if kind == "csv":
        v = _csv_values(case, seed)
        return dict(records=dict(lat_deg=_over(v["lat"].double(), 1e6), lon_deg=-_over(v["lon"].double(), 1e6),
                                 speed_mps=_over(v["speed"].double(), 100)),
                    heading=torch.where(v["blank"], math.nan, v["heading"].double()))
    if kind == "lattice":
        return _exact_lattice(case, _groups(case, seed))
    if kind == "hygiene":
        rec, perm = _sorted_records(case, seed, 7, gaps=True)[:2]
        same = torch.ones(case["records"] - 1, dtype=torch.bool, device=DEV)
        for v in rec.values():
            same &= v[1:] == v[:-1]
        keep = torch.cat([same.new_ones(1), ~same])
        return dict(kept={k: rec[k][keep] for k in ("lat_deg", "lon_deg", "speed_mps")})
    grid = gen.GRIDS[case["grid"]] if "grid" in case else gen.GRIDS["c4" if case["heavy"] else "c3"]
    shard, pad_j, pad_g = None, None, None
    if kind == "directions":
        if case["source"] == "bearing":
            return None  # a sector's edge may fall on either side of a rounding
        state = prepare(case, seed)
        r = state["rec"]
        n_dir, deg = case["n_dir"], state["column"][state["perm"].long()].double()
        sector = torch.floor(_over(deg + 180.0 / n_dir, 360.0 / n_dir)).long() % n_dir
        rows = _group_rows(r, grid, state["out"]["key"].numel(), None, sector, n_dir + 1)
        return dict(heading=deg, groups=rows)
    if kind == "batch":
        rec, sizes, _ = _batch_records(case, seed)
        pad_j = _journey_capacity(case)
        shard = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.as_tensor(sizes, device=DEV))
    elif kind == "serve":
        rec, _, _ = _serve_records(case, seed)
    else:
        rec, pad_j = _plain_records(case, seed)
    order = _order(rec["journey_id"], rec["ts_ms"], shard)
    r = _take(rec, order)
    del rec
    if kind == "oneshot":
        pad_j = None
    pad_g = case["records"] // 3 + 4096 if kind == "serve" else _capacity(case["records"], case["grid"])
    first = torch.cat([r["ts_ms"].new_ones(1).bool(), r["journey_id"][1:] != r["journey_id"][:-1]])
    f, moving, _ = _kinematics(r, first)
    sh = None if shard is None else shard[order]
    out = dict(summary=_journey_rows(r, f, moving, first, pad_j), groups=_group_rows(r, grid, pad_g, sh))
    if kind == "serve":
        back = torch.empty_like(order)
        back[order] = torch.arange(order.numel(), device=DEV)
        out["features"] = {k: v[back] for k, v in f.items()}
        return out
    out["features"] = f
    out["sorted"] = {k: r[k] for k in ("lat_deg", "lon_deg", "speed_mps")}
    return out


def _exact_lattice(case, groups):
    grid = gen.GRIDS[case["grid"]]
    C, cells = cvetl.lattice_channels(case["n_dir"]), grid.n_lat * grid.n_lon
    out = torch.zeros(case["n_t"] * C * cells, dtype=torch.float64, device=DEV)
    td, cell = groups["key"] // cells, groups["key"] % cells
    at = 2 * td * cells + cell
    mean, volume = groups["sum_speed"] / groups["count"].double(), groups["n_journeys"].double()
    minmax = torch.full((C, 2), math.nan, dtype=torch.float64, device=DEV)
    for d in range(C // 2):
        m = td % (C // 2) == d
        for c, v in ((2 * d, mean), (2 * d + 1, volume)):
            if m.any():
                lo, hi = v[m].min(), v[m].max()
                minmax[c, 0], minmax[c, 1] = lo, hi
                out[at[m] + (c % 2) * cells] = (v[m] - lo) / (hi - lo)
    return dict(tensor=out.view(case["n_t"], C, grid.n_lat, grid.n_lon), minmax=minmax)
