"""Autotuner of the batched launch and of the per-frame path.

Batched launch: three tunables.  Waves per column (1, 2 or 4 wave64s share a
column's rows): more waves shorten each column and, with fewer columns in
flight, shrink the set of object prefix tables the caches have to hold, at
the price of one barrier per recurrence step.  Columns per wave (1, or 2
with one column per 32-lane half, which shares the per-step work between two
columns at the price of more registers).  Resident workgroups of the
persistent kernel: more hide more latency; fewer leave each SIMD less
contended and shorten the tail when the column tasks do not divide evenly
into the resident set.  For a job list the tuner captures the launch once
per candidate, times a few graph replays with HIP events, keeps the fastest,
and caches the choice on disk keyed by the device, the built library and the
job signature (the multiset of frame height, width, stixel width and d_range).

Per-frame path: waves per column and the placement of the object prefix
table (global memory, or an LDS copy per column where it fits), timed the
same way on one frame.

Results never depend on the choices: every candidate computes the same bits.
"""

from __future__ import annotations

import hashlib
import json
import os
import statistics

from . import binding

DEFAULT_CACHE = os.path.join(os.path.expanduser("~"), ".cache", "stixels_autotune.json")


def signature(items) -> str:
    shapes = {}
    for h, disp, _ in items:
        H, W = disp.shape
        key = f"{H}x{W}/s{h.s}/d{h.D}"
        shapes[key] = shapes.get(key, 0) + 1
    return ";".join(f"{k}*{n}" for k, n in sorted(shapes.items()))


def device_key() -> str:
    import torch
    p = torch.cuda.get_device_properties(torch.cuda.current_device())
    return f"{p.name}|{getattr(p, 'gcnArchName', '')}|cu{p.multi_processor_count}"


def library_key() -> str:
    """Identity of the built library: which layout is fastest changes with its
    kernels."""
    try:
        with open(binding.lib_path(), "rb") as f:
            return hashlib.sha256(f.read()).hexdigest()[:16]
    except OSError:
        return "none"


def _load(path):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _store(path, data):
    os.makedirs(os.path.dirname(path), exist_ok=True)
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        json.dump(data, f, indent=1, sort_keys=True)
    os.replace(tmp, path)


def candidates(max_workgroups: int, ntasks: int):
    """Grid sizes to try: the resident maximum, fractions of it, and the
    sizes that split the tasks into whole rounds."""
    out = set()
    for frac in (1.0, 0.875, 0.75, 0.625, 0.5):
        out.add(max(1, int(max_workgroups * frac)))
    rounds = -(-ntasks // max_workgroups)
    for r in (rounds, rounds + 1):
        out.add(max(1, -(-ntasks // r)))
    return sorted(g for g in out if g <= max_workgroups)


def _time_all(run, stream, replays):
    """Milliseconds of each of `replays` runs after one warm-up run (HIP
    events on the launch stream)."""
    import torch
    run()                                          # warm
    torch.cuda.synchronize()
    ms = []
    for _ in range(replays):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record(stream)
        run()
        b.record(stream)
        b.synchronize()
        ms.append(a.elapsed_time(b))
    return ms


def _time(run, stream, replays):
    return statistics.median(_time_all(run, stream, replays))


WAVES = (1, 2, 4)


def tune(batch, items, stream, replays: int = 9, cache_path: str | None = DEFAULT_CACHE,
         force: bool = False, waves=(0,) + WAVES) -> dict:
    """Pick and apply waves per column and the workgroup count for `items`
    on `batch`; returns the record (also cached).  Leaves the batch captured
    with the chosen configuration.  waves 0 stands for the automatic choice
    where that spreads a column over a workgroup (elsewhere it equals one of
    the others and is not timed)."""
    cache, key = {}, None
    if cache_path:
        cache = _load(cache_path)
        key = f"{device_key()}|{library_key()}||{signature(items)}"
    if not force and key in cache and "columns" in cache[key]:
        rec = cache[key]
        batch.set_columns(rec["columns"])
        batch.set_waves(rec["waves"])
        batch.set_workgroups(rec["workgroups"])
        batch.capture(items, stream)
        return dict(rec, cached=True)

    # layouts: (waves per column, columns per wave); two columns per wave
    # only pair with one wave per column
    layouts = [(w, 1) for w in waves] + ([(1, 2)] if 1 in waves else [])
    timings = {}
    ntasks = {}
    held = {}                                      # waves a column really has
    for w, c in layouts:
        batch.set_waves(w)
        batch.set_columns(c)
        batch.set_workgroups(0)
        batch.capture(items, stream)
        # not available for these rows, or automatic and not spread: one wave
        # (a spread column has at least four)
        if batch.columns() != c or (batch.waves() != w if w else batch.waves() == 1):
            continue
        gmax, nt = batch.info()
        for g in candidates(gmax, nt):
            batch.set_workgroups(g)
            batch.capture(items, stream)
            timings[(c, w, g)] = _time(lambda: batch.replay(stream), stream, replays)
            ntasks[(c, w, g)] = nt
            held[(c, w, g)] = batch.waves()
    # Candidates within 1.5 % of the fastest are timed again, in three
    # interleaved blocks of `replays` replays each (so that a drift of the
    # clock or of the memory system over the sweep does not pick for them),
    # and keep the median of all their replays.
    first = dict(timings)
    fastest = min(timings.values())
    close = sorted(k for k, v in timings.items() if v <= fastest * 1.015)
    if len(close) > 1:
        samples = {k: [] for k in close}
        for _ in range(3):
            for c, w, g in close:
                batch.set_columns(c)
                batch.set_waves(w)
                batch.set_workgroups(g)
                batch.capture(items, stream)
                samples[(c, w, g)] += _time_all(lambda: batch.replay(stream), stream, replays)
        for k in close:
            timings[k] = statistics.median(samples[k])
    # near-ties (within 0.25 %, about the replay-to-replay noise) go to one
    # column per wave, fewer waves per column (those it has: the automatic
    # setting, 0, spreads it over several), then fewer workgroups: the same
    # speed for less of the device.  (A 1 % margin picked grids that
    # the kernel trace then showed 2-3 % slower.)
    fastest = min(timings[k] for k in close) if len(close) > 1 else fastest
    timings = {k: v for k, v in timings.items() if len(close) <= 1 or k in close}
    best = min((k for k, v in timings.items() if v <= fastest * 1.0025),
               key=lambda k: (k[0], held[k], k[2]))
    batch.set_columns(best[0])
    batch.set_waves(best[1])
    batch.set_workgroups(best[2])
    batch.capture(items, stream)
    def name(k):
        c, w, g = k
        return (f"c{c}/" if c > 1 else "") + f"w{w}/g{g}"
    rec = {"columns": best[0], "waves": best[1], "workgroups": best[2], "ms": timings[best],
           "tasks": ntasks[best],
           "tried": {name(k): round(v, 4) for k, v in sorted(first.items())},
           "refined": {name(k): round(v, 4) for k, v in sorted(timings.items())}}
    if cache_path:
        cache[key] = rec
        _store(cache_path, cache)
    return dict(rec, cached=False)


def tune_frame(handle, disp, out, stream, replays: int = 5, waves=WAVES,
               placements=(1, 2)) -> dict:
    """Pick and apply the recurrence of the per-frame path for frames of this
    size: the automatic setting (0, 0: a column spread over a workgroup), or
    waves per column and the object prefix table placement (1 HBM, 2 LDS where
    it fits); returns the timings."""
    H, W = disp.shape
    handle.set_waves(0)
    handle.set_po_placement(0)
    timings = {(0, 0): _time(lambda: handle.compute(disp, out, stream), stream, replays)}
    for pl in placements:
        handle.set_po_placement(pl)
        for w in waves:
            handle.set_waves(w)
            if handle.waves(W, H) != w:
                continue
            timings[(w, pl)] = _time(lambda: handle.compute(disp, out, stream), stream, replays)
    best = min(timings, key=timings.get)
    handle.set_waves(best[0])
    handle.set_po_placement(best[1])
    return {"waves": best[0], "po_placement": best[1], "ms": timings[best],
            "tried": {f"w{w}/{'lds' if pl == 2 else 'hbm'}" if w else "auto": round(v, 4)
                      for (w, pl), v in sorted(timings.items())}}
