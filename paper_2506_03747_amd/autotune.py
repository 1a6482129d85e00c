"""Autotuner of the forward's launch plan.

For each class of problems (confocal or not, window length, number of
histograms) it forces every supported unit shape in turn through the tuning
table, two units to a workgroup, and times the forward operator on a seeded
synthetic scene of that class, alone and as a list of three (HIP events, median
of repeated launches): an entry governs both.  A unit becomes an entry if it
beats the library's own plans by more than 2% in one and is not more than 2%
slower in the other.  The result is written as a JSON table that the package
installs at import (``load_tuning``);
``python -m paper_2506_03747_amd.autotune [out.json]``.

Timing only chooses among shapes the library already supports; every shape
computes the same result (the GPU tests force each one and compare them
with the oracle).
"""
from __future__ import annotations

import json
import sys

import numpy as np

from . import Batcher, forward, forward_batched, get_plan, make_params, out_shape, patches_from_depth, reset_tuning, set_tuning

CONFOCAL_UNITS = [(1, 4, 4), (1, 4, 2), (1, 2, 2), (1, 2, 1)]
NONCONFOCAL_UNITS = [(2, 2, 2), (2, 1, 2), (1, 1, 2)]

# Classes: (confocal, t range, histogram range) and the problem each is timed
# on: window T, bin width, scan side, laser side (0: confocal).
CLASSES = []
for _t_min, _t_max, _T, _bin in [(1, 767, 512, 16.0), (768, 1535, 1024, 8.0), (1536, 4096, 2048, 4.0)]:
    for _h_min, _h_max, _ns in [(1, 2047, 32), (2048, 8191, 64), (8192, 1 << 40, 128)]:
        CLASSES.append(dict(confocal=1, t_min=_t_min, t_max=_t_max, h_min=_h_min, h_max=_h_max,
                            T=_T, bin_ps=_bin, scan=_ns, lasers=0))
    CLASSES.append(dict(confocal=0, t_min=_t_min, t_max=_t_max, h_min=1, h_max=1 << 40,
                        T=_T, bin_ps=_bin, scan=64, lasers=4))


def _scene(cls, n_patch, seed):
    """Seeded planar-ish hidden surface facing a 2 x 2 m wall, half the
    patches masked out, depths spread over the middle of the window."""
    import torch
    rng = np.random.default_rng(seed)
    reach = 299792458.0 * cls["T"] * cls["bin_ps"] * 1e-12 / 2.0      # one-way range of the window
    z = np.asarray(0.3 * reach + 0.15 * reach * rng.uniform(size=(n_patch, n_patch)), np.float32)
    mask = (rng.uniform(size=(n_patch, n_patch)) < 0.5).astype(np.uint8)
    alb = rng.uniform(0, 1, (n_patch, n_patch)).astype(np.float32)
    side = lambda n: dict(nx=n, ny=n, half_x=1.0, half_y=1.0, cx=0.0, cy=0.0)
    rec, n = patches_from_depth(torch.from_numpy(z).cuda(), side(n_patch), torch.from_numpy(alb).cuda(),
                                torch.from_numpy(mask).cuda())
    laser = side(cls["lasers"]) if cls["lasers"] else None
    prm = make_params(side(cls["scan"]), cls["T"], cls["bin_ps"], 50.0, laser=laser)
    return prm, rec, n


def _time(fn, reps=7):
    import torch
    fn()
    torch.cuda.synchronize()
    ts = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1))
    return float(np.median(ts))


def choose(own, timings):
    """The unit to enter, or None: ``own`` is the library's plans' (alone, list)
    times, ``timings`` {unit: (alone, list)}."""
    best = None
    for unit, got in timings.items():
        r = [g / o for g, o in zip(got, own)]
        if min(r) < 0.98 and max(r) <= 1.02 and (best is None or r[0] * r[1] < best[0]):
            best = (r[0] * r[1], unit)
    return best[1] if best else None


def tune(n_patch=192, classes=CLASSES, verbose=True):
    """Time every unit per class; returns (table entries, all timings)."""
    import torch
    entries, report = [], []
    batcher = Batcher()
    try:
        for k, cls in enumerate(classes):
            prm, rec, n = _scene(cls, n_patch, seed=1000 + k)
            outs = [torch.empty(out_shape(prm), dtype=torch.float32, device="cuda") for _ in range(3)]
            key = {f: cls[f] for f in ("confocal", "t_min", "t_max", "h_min", "h_max")}

            def both():
                return (_time(lambda: forward(prm, rec, n, out=outs[0])),
                        _time(lambda: forward_batched([(prm, rec, n, o) for o in outs], batcher)))

            set_tuning([])
            own, timings, rows = both(), {}, []
            for unit in (CONFOCAL_UNITS if cls["confocal"] else NONCONFOCAL_UNITS):
                set_tuning([dict(key, tl=unit[0], tx=unit[1], ty=unit[2])])
                plan = get_plan(prm, rec.shape[0])
                # (its plan is the library's own where two of the units do not fit in LDS)
                if (plan["tl"], plan["tx"], plan["ty"]) == unit:
                    timings[unit] = both()
                    rows.append((unit, plan, timings[unit]))
            # (the library's own plans at both ends: the first timings of a class run
            # 1 to 2% slow)
            set_tuning([])
            own = tuple(map(min, own, both()))
            rows.insert(0, (None, get_plan(prm, rec.shape[0]), own))
            for unit, plan, (ms, list_ms) in rows:
                report.append(dict(key, T=cls["T"], scan=cls["scan"], lasers=cls["lasers"],
                                   unit=None if unit is None else list(unit), ms=ms, list_ms=list_ms, plan=plan))
                if verbose:
                    print(f"class {k} T={cls['T']} scan={cls['scan']}^2 lasers={cls['lasers']}^2 "
                          f"unit={unit or 'own'}: {ms:.4f} ms, list of 3 {list_ms:.4f} ms  {plan}", flush=True)
            unit = choose(own, timings)
            if unit:
                entries.append(dict(key, tl=unit[0], tx=unit[1], ty=unit[2]))
            del outs
    finally:
        reset_tuning()
    return entries, report


def main(argv=None):
    import torch
    argv = sys.argv[1:] if argv is None else argv
    out = argv[0] if argv else "tuning.json"
    entries, report = tune()
    with open(out, "w") as f:
        json.dump({"device": torch.cuda.get_device_name(0), "entries": entries, "timings": report}, f, indent=1)
    print(json.dumps(entries))


if __name__ == "__main__":
    main()
