"""Autotuner for the library's tuning knobs.

Sweeps the compiled radix-pass tile shapes (threads x keys per thread) on a
workload and keeps the fastest per workload signature (record count, whether
the batch is many shards, grid cardinality) in a JSON cache next to this file.
The plain workloads, their records in the order of a time-ordered feed, are timed
by the record sort's scatter passes (the library's per-kernel HIP-event timing;
journey files in near order need no pass, and up to 2^21 records all passes share one
launch of its own shape: both are refused); the batched workload (many uneven
shards in one set of launches) by its whole step, since its shape choice also
moves the group-key sort of the grid merge.  ``apply(n, workload)`` installs the
cached choice of the same signature, nearest in n, or leaves the library
default.

    python -m paper_2305_07454_amd.tune --workload c1|c2 [--reps 5]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ONE_LAUNCH = 1 << 21  # records up to which a sort's passes share one launch of its own shape

CACHE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuning.json")


def _load(path=CACHE):
    if os.path.exists(path):
        with open(path) as f:
            return json.load(f)
    return {"arch": "gfx950", "entries": []}


def signature(workload: str, n: int) -> dict:
    """What a tuning choice depends on: the record count, whether the batch is
    many shards (one key prefix more, interleaved feeds) and the grid's
    cardinality (records per group set how many partial rows the grid merge
    sorts)."""
    from . import gen
    g = gen.GRIDS.get(workload)
    cells = int(g.n_lat) * int(g.n_lon) * max(1, int(g.n_t)) if g is not None else 0
    return {"workload": workload, "n": int(n), "sharded": workload == "c2", "cells": cells}


def apply(n: int, workload: str | None = None) -> dict | None:
    """Install the cached choices for a batch of n records: the entry of the
    same workload signature (sharded or not, same grid), nearest in n; without
    a workload, the nearest n of any entry.  Returns the entry used."""
    from . import cvetl
    c = _load()
    want = signature(workload, n) if workload else None
    best = None
    for e in c.get("entries", []):
        if want is not None:
            sig = e.get("signature") or signature(e.get("workload", "c1"), e["n"])
            if sig["sharded"] != want["sharded"] or sig["cells"] != want["cells"]:
                continue
        if best is None or abs(e["n"] - n) < abs(best["n"] - n):
            best = e
    if best is None:
        return None
    cvetl.cv_tuning_set("sort_shape", best["sort_shape"])
    return best


def sweep_sort_shapes(rec, grid, reps=5, log=print):
    """Time the record sort passes for every compiled shape on one batch.
    ValueError for a batch that says nothing of the shapes: one that no pass
    sorts, or of so few records that all passes share a launch."""
    import torch
    from . import cvetl
    n = int(rec["journey_id"].numel())
    if n <= ONE_LAUNCH:
        raise ValueError(f"{n} records: up to {ONE_LAUNCH} the passes share one launch, whatever the shape")
    mj = max(1, min(n, 1 << 20))
    ws = cvetl.workspace(cvetl._size(cvetl.lib().cv_sort_workspace_size, n, mj), rec["journey_id"].device)
    shapes = cvetl.cv_tuning_get("sort_shapes")
    results = []
    for sh in range(shapes):
        cvetl.cv_tuning_set("sort_shape", sh)
        tile = cvetl.cv_tuning_get("sort_tile")
        perm, srt, r = cvetl.cv_sort_records(rec, max_journeys=mj, ws=ws)  # warm-up and key width
        if cvetl.cv_sort_passes(ws) == 0:
            raise ValueError("whole journeys in near order: no pass sorts them")
        db = int(cvetl.cv_tuning_get("radix_bits"))
        w0 = int(r.get("flags") or db)  # bits of the first digit (9 where that saves a pass)
        kb = int(r["key_bits"])
        passes = 0 if kb <= 0 else (1 if kb <= w0 else 1 + (kb - w0 + db - 1) // db)
        torch.cuda.synchronize()
        cvetl.cv_timing_reset()
        cvetl.cv_timing_enable(True)
        for _ in range(reps):
            cvetl.cv_sort_records(rec, max_journeys=mj, ws=ws, sync=False)
        torch.cuda.synchronize()
        cvetl.cv_timing_enable(False)
        ms = [cvetl.cv_timing_read(f"sort_pass{p}") for p in range(passes)]
        per = sum(m for m, _ in ms) / max(1, sum(c for _, c in ms))
        # the passes of one sort: shapes of 512 threads or more may take a
        # 9-bit first digit and one pass fewer, so the sort's sum decides
        tot = sum(m for m, _ in ms) / reps
        results.append({"sort_shape": sh, "tile": tile, "pass_ms": round(per, 5), "passes": passes,
                        "first_digit_bits": w0, "sort_ms": round(tot, 5)})
        log(f"shape {sh} (tile {tile}): {per:.4f} ms per pass, {passes} passes, {tot:.4f} ms per sort")
    return results


def sweep_batched(rec, sizes, grid, reps=5, log=print):
    """Time the whole batched step (sort, kinematics, summaries, grid merge)
    for every compiled shape on one resident batch of shards."""
    import torch
    from . import cvetl
    n = int(rec["journey_id"].numel())
    dev = rec["journey_id"].device
    off_h, off_d = cvetl.shard_offsets(sizes, dev)
    bp0, res0 = cvetl.cv_batch_run(rec, sizes, grid)
    J, G, mj = res0[1]["count"], res0[2]["count"], bp0.max_journeys
    del bp0
    torch.cuda.empty_cache()
    bp = cvetl.BatchPipeline(n, len(sizes), grid, mj, J, max(4096, int(1.25 * G)), dev)
    stream = torch.cuda.current_stream()
    results = []
    for sh in range(cvetl.cv_tuning_get("sort_shapes")):
        cvetl.cv_tuning_set("sort_shape", sh)
        bp.run(rec, off_d)
        torch.cuda.synchronize()
        assert all(r["status"] == 0 for r in bp.results())
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(stream)
        for _ in range(reps):
            bp.run(rec, off_d)
        ev[1].record(stream)
        torch.cuda.synchronize()
        ms = ev[0].elapsed_time(ev[1]) / reps
        results.append({"sort_shape": sh, "tile": cvetl.cv_tuning_get("sort_tile"), "step_ms": round(ms, 4)})
        log(f"shape {sh} (tile {cvetl.cv_tuning_get('sort_tile')}): {ms:.3f} ms per batched step")
    del bp
    torch.cuda.empty_cache()
    return results


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="c1", choices=["c0", "c1", "c2"])
    ap.add_argument("--n-journeys", type=int, default=None)
    ap.add_argument("--reps", type=int, default=5)
    ap.add_argument("--out", default=CACHE)
    args = ap.parse_args()
    import torch
    from . import cvetl, gen
    t = time.time()
    say = lambda m: print(f"[tune] {m}", file=sys.stderr, flush=True)  # noqa: E731
    if args.workload == "c2":
        shards = gen.make_c2()
        sizes = [x.n for x in shards]
        r = gen.concat(shards)
        del shards
    elif args.workload == "c1":
        r = gen.make_c1(**({"n_journeys": args.n_journeys} if args.n_journeys else {}))
    else:
        r = gen.make_c0(**({"n_journeys": args.n_journeys} if args.n_journeys else {}))
    say(f"{args.workload}: {r.n} records ({time.time() - t:.1f}s)")
    n = r.n
    rec = cvetl.to_device(r)
    del r
    if args.workload != "c2":
        order = torch.sort(rec["ts_ms"], stable=True)[1]
        rec = {k: v[order] for k, v in rec.items()}
        del order
    grid = gen.GRIDS[args.workload]
    if args.workload == "c2":
        res = sweep_batched(rec, sizes, grid, args.reps, log=say)
        best = min(res, key=lambda x: x["step_ms"])
    else:
        res = sweep_sort_shapes(rec, grid, args.reps, log=say)
        best = min(res, key=lambda x: x.get("sort_ms", x["pass_ms"] * x["passes"]))
    c = _load(args.out if os.path.exists(args.out) else CACHE)
    sig = signature(args.workload, n)
    c["entries"] = [e for e in c.get("entries", []) if e.get("workload") != args.workload or e["n"] != n]
    entry = {"workload": args.workload, "n": n, "signature": sig, "sort_shape": best["sort_shape"],
             "tile": best["tile"], "sweep": res, "device": torch.cuda.get_device_name(0)}
    entry.update({k: best[k] for k in ("pass_ms", "sort_ms", "step_ms") if k in best})
    c["entries"].append(entry)
    with open(args.out, "w") as f:
        json.dump(c, f, indent=1)
    print(json.dumps({"best": best, "sweep": res}))


if __name__ == "__main__":
    main()
