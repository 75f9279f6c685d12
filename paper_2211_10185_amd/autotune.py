"""Pass-schedule autotuner for the FFT kinetic terms.

For a lattice size N, a state precision and a state count, the solver can run a
step as
  * the plane schedule (x2-x3 plane pass + x1 column pass: 2 passes per step),
    available where an N^2 plane fits in LDS, or
  * the row/column schedule (x3 row pass + three column passes: 4 passes), or
  * the split-x2 schedule (slab pass + pencil pass: 2 passes), in one or two tile
    shapes, and in complex64 from N = 96 up also with the two factors of x2 swapped
    (a radix-plan choice) and at 128 and 256 with 8-row tiles of 8 columns,
and, with k >= 2 states, either carry all states through one stream or split
them into two (or, with k >= 3, three) groups pipelined on their own streams.  ``tune`` times every candidate
on the device with the solver's own kernels and records the fastest in a JSON
cache; ``schedule_for`` is what ``Solver`` consults at creation.

Cache: ``$QFDTD_TUNING`` if set, else ``tuning.json`` next to this file.
Entry key: "N/precision/states" with states clipped to {1, 2+}.  An entry with a "pinned" note
was chosen from another measurement (the note says which) and ``tune`` leaves it as it is.
A complex64 entry keeps its rounding (``rounding``) when it is tuned again.
"""
from __future__ import annotations

import json
import os
import time
from typing import Dict, Iterable, Optional

HERE = os.path.dirname(os.path.abspath(__file__))
PLANE_LIMIT = {0: 128, 1: 96}      # largest N whose plane fits LDS (complex64 / complex128)
# sizes with split-x2 (slab and pencil) kernels
SPLIT_SIZES = {0: (96, 100, 108, 120, 128, 144, 150, 160, 162, 180, 192, 200, 216, 240, 250, 256), 1: ()}
SPLIT_WIDE_SIZES = {0: (128, 256), 1: ()}    # ... and with the 8-row, 8-column variant
SPLIT_SWAPPED_SIZES = {0: (96, 108, 120, 128, 144, 150, 160, 162, 180, 192, 200, 216, 240, 250), 1: ()}
# complex128 split-x2 kernels: every size from 32 up, with a second tile shape (variant 1) at some
SPLIT_C128_SIZES = (32, 36, 40, 48, 50, 54, 60, 64, 72, 80, 90, 96, 100, 108, 120, 128, 144, 150, 160, 162, 180, 192,
                    200, 216, 240, 250, 256)
SPLIT_SMALL_SIZES = (32, 36, 40, 48, 50, 54, 60, 64, 72, 80, 90)     # complex64, one tile shape
SPLIT_C128_SECOND = (40, 48, 72, 80, 96, 108, 120, 150, 160, 162, 192, 216, 250)
SPLIT_C64_SECOND = (150, 162, 250)     # complex64: the second tile shape where 4 does not divide N
_cache: Optional[Dict[str, dict]] = None


def cache_path() -> str:
    return os.environ.get("QFDTD_TUNING", os.path.join(HERE, "tuning.json"))


def _load() -> Dict[str, dict]:
    global _cache
    if _cache is None:
        try:
            with open(cache_path()) as f:
                _cache = json.load(f).get("entries", {})
        except (OSError, ValueError):
            _cache = {}
    return _cache


def key(N: int, precision: int, k: int) -> str:
    return "%d/%d/%d" % (N, precision, 1 if k <= 1 else 2)


def default_schedule(N: int, kinetic: int, precision: int, k: int) -> dict:
    # without a measurement: two streams pay off only once a group's passes fill the GPU
    single = k < 2 or N < 96
    return {"rowcol": False, "single_stream": single, "groups": 1 if single else 2, "split": False}


def cache_sized(N: int, precision: int, k: int) -> bool:
    """Complex64 states that together are a little larger than the 256 MB Infinity Cache.  On one stream the
    passes then still find most of them there; groups on streams of their own, each at another place of its
    states, lose that.  us per step, the three groups that three states are tuned to against one stream, with
    a real / complex V: 160^3 x 8 states (262 MB) 283 / 300 -> 278 / 277, 162^3 x 8 (272 MB) 433 / 441 -> 402 /
    420, 180^3 x 6 (280 MB) 426 / 429 -> 394 / 391, 200^3 x 4 (256 MB) 352 / 380 -> 341 / 360.  Groups win below
    (162^3 x 6, 204 MB: 257 / 268 against 269 / 272) and are within 3% above (200^3 x 5, 320 MB: 466 / 476 against
    464 / 466).  In complex128 it goes either way (160^3 x 4, 262 MB: 310 / 322 -> 290 / 286; 162^3 x 4, 272 MB:
    394 / 438 -> 397 / 439), so the tuned groups stay there."""
    return precision == 0 and 256e6 <= k * N ** 3 * 8 <= 290e6


def schedule_for(N: int, kinetic: int, precision: int, k: int) -> dict:
    """Tuned schedule if the cache has one for (N, precision, k), else the default."""
    if kinetic == 0:
        return {"rowcol": False, "single_stream": True, "groups": 1, "split": False}
    e = _load().get(key(N, precision, k))
    if e is None:
        return default_schedule(N, kinetic, precision, k)
    single = bool(e["single_stream"]) or (bool(e.get("split", False)) and cache_sized(N, precision, k))
    return {"rowcol": bool(e["rowcol"]), "single_stream": single,
            "groups": 1 if single else int(e.get("groups", 2)), "split": bool(e.get("split", False)),
            "split_variant": int(e.get("split_variant", 0))}


def ab_schedule(N: int, precision: int, k: int) -> Optional[dict]:
    """Split-x2 schedule of the A/B update of an FFT kinetic term, None where the other schedules stay.

    Measured (sin^2 kinetic term, us per step).  The best plane or row/column schedule against split-x2, one
    state / three: complex64 32: 15.8 -> 10.9 / 16.1 -> 11.7, 64: 20.9 -> 15.7 / 25.7 -> 21.4, 90: 42.5 -> 30.0 /
    58.4 -> 44.7, 128: 44.9 -> 34.4 / 92.5 -> 67.6 (above 128 the row/column passes stay: the split-x2 factors
    would change the FP32 results); complex128 64: 24.7 -> 17.4 / 31.9 -> 29.9, 128: 71.2 -> 45.9 / 187 -> 108,
    160: 139 -> 105 / 417 -> 323, 240: 556 -> 478 / 1752 -> 1357, 256: 613 -> 510 / 1853 -> 1430, but 216: 368 ->
    390 and 250: 622 -> 642 with one state.
    The second tile shape against the first, complex128 (fewer plane groups and registers beside the psi that
    this update also reads): 120 one state 65 -> 52 (three 114 -> 123), 160 three states 357 -> 323 (one 105
    either way), 162 151 -> 121 / 474 -> 427, 192 250 -> 219 / 723 -> 640, 250 three states 2182 -> 1831; at the
    other sizes that have one it is within 7% (80, one state: 29.2 -> 27.2) or slower (150 three states 316 -> 344).
    Three groups of states against one stream, three states: complex64 80: 40.0 -> 34.3, 90: 49.6 -> 44.7, 96:
    46.1 -> 43.7, 100: 52.7 -> 46.7, 120: 86.4 -> 66.5, 128: 78.2 -> 67.6, but 108: 58.0 -> 56.8 (no more than runs
    differ) and below 80 slower (72: 30.4 -> 30.5, 64: 21.4 -> 27.8); complex128 90: 60.0 -> 52.6, 96: 61.9 -> 54.4,
    100: 78.7 -> 69.9, 108: 94.0 -> 82.5, 120: 163 -> 114, 128: 120 -> 108, 160: 350 -> 323, but 80: 38.1 -> 39.8, 144:
    230 -> 231, 150: 323 -> 335, 162: 427 -> 430, 192: 640 -> 652, 240: 1357 -> 1349."""
    if precision == 0:
        if N not in SPLIT_SMALL_SIZES + (96, 100, 108, 120, 128):
            return None
        groups = 1 if N < 80 or N == 108 else min(k, 3)
        variant = 0
    else:
        if N not in SPLIT_C128_SIZES or (k == 1 and N in (216, 250)):
            return None
        groups = min(k, 3) if N in (90, 96, 100, 108, 120, 128, 160) else 1
        variant = 1 if N in (160, 162, 192, 250) or (N == 120 and k == 1) else 0
    return {"rowcol": False, "single_stream": groups == 1, "groups": groups, "split": True, "split_variant": variant}


def ab_schedule_for(N: int, precision: int, k: int, tuned: dict) -> dict:
    """Schedule of the A/B update beside the cache's choice for the split step: its own rule where it has
    split-x2 kernels, else plane or row/column passes on one stream.  A cache that asks for row and column
    passes in complex64 gets them: they round in another order than the plane passes."""
    ab = None if precision == 0 and tuned["rowcol"] else ab_schedule(N, precision, k)
    return ab or dict(tuned, split=False)


def candidates(N: int, precision: int, k: int):
    out = []
    plane_ok = N <= PLANE_LIMIT[precision]
    for rowcol in ([False, True] if plane_ok else [True]):
        groups = [1] if rowcol or k < 2 else ([1, 2, 3] if k >= 3 else [1, 2])
        for g in groups:
            out.append({"rowcol": rowcol, "single_stream": g == 1, "groups": g, "split": False})
    if N in SPLIT_SIZES[precision]:
        # variant 1 where 4 does not divide N: more_candidates
        variants = ([0] + ([1] if N % 4 == 0 else []) + ([2] if N in SPLIT_WIDE_SIZES[precision] else [])
                    + ([3] if N in SPLIT_SWAPPED_SIZES[precision] else []))
        groups = [1, 2, 3] if k >= 3 else ([1, 2] if k >= 2 else [1])
        for v in variants:
            for g in groups:
                out.append({"rowcol": False, "single_stream": g == 1, "groups": g, "split": True,
                            "split_variant": v})
    return out


def single_shape_split(N: int, precision: int) -> bool:
    """Sizes whose split-x2 kernels come on top of ``candidates`` (see ``more_candidates``)."""
    return N in (SPLIT_C128_SIZES if precision == 1 else SPLIT_SMALL_SIZES)


def more_candidates(N: int, precision: int, k: int):
    """The split-x2 candidates that ``candidates`` leaves out: every one of the sizes without a choice of
    factors, and the second tile shape of complex64 where 4 does not divide N."""
    if precision == 1:
        variants = ([0] if N in SPLIT_C128_SIZES else []) + ([1] if N in SPLIT_C128_SECOND else [])
    else:
        variants = ([0] if N in SPLIT_SMALL_SIZES else []) + ([1] if N in SPLIT_C64_SECOND else [])
    groups = [1, 2, 3] if k >= 3 else ([1, 2] if k >= 2 else [1])
    return [{"rowcol": False, "single_stream": g == 1, "groups": g, "split": True, "split_variant": v}
            for v in variants for g in groups]


def schedule_name(c: dict) -> str:
    """The schedule as a word of its own: what ``tune`` files times under."""
    kind = "split/v%d" % c.get("split_variant", 0) if c.get("split") else ("rowcol" if c["rowcol"] else "plane")
    return "%s/%d" % (kind, c.get("groups", 1))


def rounding(c: dict, N: int, precision: int) -> Optional[str]:
    """What decides the roundings of a complex64 step under the schedule: the radix sequence of its line
    transforms and the factors of x2, not its tiles or groups.  The energies of complex64 solves (FP64 sums
    over FP32 states) keep their digits only as long as this stays: other factors move them by up to 1e-6.
    Complex128 results move within 1e-14, so there it decides nothing (None)."""
    if precision == 1:
        return None
    if not c.get("split"):
        return "rowcol" if c["rowcol"] else "plane"
    if N in SPLIT_SMALL_SIZES:
        return "plane"                      # the operations of the plane passes
    v = c.get("split_variant", 0)
    # the 8-row tiles are the default factors at 128 (16 x 8) and others at 256 (32 x 8)
    return "swapped" if v == 3 else "32 x 8" if v == 2 and N == 256 else "default"


def candidate_name(c: dict, N: int = 256) -> str:
    """A short description of one of ``candidates`` by its tile columns (complex64; not a key: variants of
    other sizes and precisions may share it)."""
    if c.get("split"):
        v = c.get("split_variant", 0)
        cols = 4 if N % 4 == 0 else 2
        name = {0: "split/%dcol" % cols, 1: "split/2col", 2: "split8row/8col", 3: "split-swapped"}[v]
        return name + ("" if c.get("groups", 1) == 1 else "/%dstreams" % c["groups"])
    return ("rowcol" if c["rowcol"] else "plane") + ("/1stream" if c["groups"] == 1 else "/%dstreams" % c["groups"])


def time_schedule(N: int, precision: int, k: int, sched: dict, steps: int = 400, kinetic: int = 2,
                  reps: int = 2) -> float:
    """Microseconds per imaginary-time step of a harmonic problem under `sched` (the best of
    `reps` timed runs of `steps` steps, after a warm-up chunk that also captures the graph)."""
    import torch
    import synthetic as S
    from .solver import Solver
    a = 8.0 / N
    s = Solver(N, a, 1.0, kinetic, S.V_HARMONIC, (1.0,), precision=precision, n_states=k,
               rowcol=sched["rowcol"], groups=sched.get("groups", 1 if sched["single_stream"] else 2),
               split=sched.get("split", False), split_variant=sched.get("split_variant", 0))
    s.set_states(S.initial_states(N, k, 7))
    dt = a * a / 8
    s.evolve(50, dt)
    s.energies()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(reps):
        t0 = time.perf_counter()
        s.evolve(steps, dt)
        s.energies()
        torch.cuda.synchronize()
        best = min(best, 1e6 * (time.perf_counter() - t0) / steps)
    s.close()
    return best


def tune(sizes: Iterable[int], precisions: Iterable[int] = (0,), states: Iterable[int] = (1, 3),
         steps: int = 400, path: Optional[str] = None, verbose: bool = True, keep: Optional[str] = None) -> Dict[str, dict]:
    """Time every candidate schedule and write the winners to the cache at `path`.

    Where the cache at `keep` (default: the one that is written) has a complex64 entry, only candidates
    with the roundings of that entry are timed (see ``rounding``)."""
    global _cache
    path = path or cache_path()
    try:
        with open(keep or path) as f:
            kept = json.load(f).get("entries", {})
    except (OSError, ValueError):
        kept = {}
    try:
        with open(path) as f:
            doc = json.load(f)
    except (OSError, ValueError):
        doc = {"entries": {}}
    entries = doc.setdefault("entries", {})
    for N in sizes:
        for prec in precisions:
            for k in states:
                if entries.get(key(N, prec, k), {}).get("pinned"):
                    # a choice made from a measurement other than this timing (the entry says which)
                    if verbose:
                        print("tune N=%d prec=%d k=%d: pinned, kept" % (N, prec, k), flush=True)
                    continue
                times, cands = {}, {}
                old = kept.get(key(N, prec, k))
                for c in candidates(N, prec, k) + more_candidates(N, prec, k):
                    if old and rounding(c, N, prec) != rounding(old, N, prec):
                        continue
                    name = schedule_name(c)
                    cands[name] = c
                    times[name] = time_schedule(N, prec, k, c, steps)
                best = min(times, key=times.get)
                c = cands[best]
                entries[key(N, prec, k)] = {"rowcol": c["rowcol"], "single_stream": c["groups"] == 1,
                                            "groups": c["groups"], "split": c["split"],
                                            "split_variant": c.get("split_variant", 0),
                                            "us_per_step": {n: round(v, 2) for n, v in times.items()}}
                if verbose:
                    print("tune N=%d prec=%d k=%d -> %s %s" % (N, prec, k, best, entries[key(N, prec, k)]["us_per_step"]),
                          flush=True)
    doc["device"] = _device_name()
    with open(path, "w") as f:
        json.dump(doc, f, indent=1, sort_keys=True)
    _cache = None
    return entries


def _device_name() -> str:
    try:
        import torch
        return torch.cuda.get_device_name(0)
    except Exception:
        return "unknown"


if __name__ == "__main__":
    import argparse
    import synthetic as S
    ap = argparse.ArgumentParser(description="time the candidate schedules of every FFT lattice size")
    ap.add_argument("out", nargs="?", default=None, help="cache file to write (default: tuning.json here)")
    ap.add_argument("--steps", type=int, default=400, help="timed imaginary-time steps per run")
    ap.add_argument("--sizes", type=int, nargs="*", default=None, help="lattice sizes (default: 32..256)")
    ap.add_argument("--precisions", type=int, nargs="*", default=[0, 1], help="0: complex64, 1: complex128")
    a = ap.parse_args()
    sizes = a.sizes or [n for n in S.smooth_even_sizes(32, 256)]
    tune(sizes, precisions=a.precisions, states=(1, 3), steps=a.steps, path=a.out, keep=cache_path())
