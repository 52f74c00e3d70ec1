"""FFT plan autotuner: times every plan of each segment length on this device,
over a grid of persistent work-group counts for the two passes, and writes the
fastest choice per length to tuning.json (applied by Context by default), every
measurement to tuning_measurements.json beside it.

    python -m paper_2002_02150_amd.autotune [--lengths 131072,262144] [--out PATH]

Timing: fitness batches of `batches` points spread over the search rectangle
(every point evaluated; 256 by default, between the 192 points a 320-particle
swarm keeps inside the rectangle early in a search and the 311 it keeps at the
end, and 16, a small call), HIP events around `reps` back-to-back calls, best
of three such runs; a choice is ranked by the geometric mean over the batches.
The data are random: the cost of an evaluation does not depend on the data
values.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import torch

from . import fcas

DEFAULT_LENGTHS = (2048, 4096, 8192, 16384, 24576, 32768, 49152, 65536, 98304, 131072, 196608, 262144, 460800,
                   3686400, 7372800)
# persistent work-groups of the first pass, and of the last (and middle) one
GRIDS1 = (512, 1024, 2048)
GRIDS2 = (2048, 4096, 16384)
# rectangle of component masses in [1, 3] Msun at f_low = 30 Hz
BOX_LO = (0.0, -math.pi / 2, 15.0336, 0.841913)
BOX_HI = (2.0 * math.pi, math.pi / 2, 93.8141, 1.75126)


def _network(n_det, device):
    """A generic network: detectors spread over the globe with crossed arms."""
    pos, ten = [], []
    for i in range(n_det):
        lat, lon = 0.7 * math.sin(1.3 * i + 0.2), 2.1 * i + 0.4
        r = 6.37e6
        p = (r * math.cos(lat) * math.cos(lon), r * math.cos(lat) * math.sin(lon), r * math.sin(lat))
        east = (-math.sin(lon), math.cos(lon), 0.0)
        north = (-math.sin(lat) * math.cos(lon), -math.sin(lat) * math.sin(lon), math.cos(lat))
        a = [(math.cos(0.3 * i) * e + math.sin(0.3 * i) * n) for e, n in zip(east, north)]
        b = [(-math.sin(0.3 * i) * e + math.cos(0.3 * i) * n) for e, n in zip(east, north)]
        pos.append(p)
        ten.append([[0.5 * (a[x] * a[y] - b[x] * b[y]) for y in range(3)] for x in range(3)])
    return pos, ten


def time_plan(ctx, plan, g1, g2, xf, psd, theta, seg, reps):
    """Mean device time (ms) of one fitness call, over `reps` back-to-back calls."""
    ctx.select_plan(plan, g1, g2)
    ctx.set_segment(0, xf, psd)
    f = torch.empty(theta.shape[0], dtype=torch.float64, device=ctx.device)
    j = torch.empty(theta.shape[0], dtype=torch.int32, device=ctx.device)
    for _ in range(3):
        ctx.eval(theta, seg, f, j)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    samples = []
    for _ in range(3):
        e0.record()
        for _ in range(reps):
            ctx.eval(theta, seg, f, j)
        e1.record()
        torch.cuda.synchronize(ctx.device)
        samples.append(e0.elapsed_time(e1) / reps)
    return min(samples)


def rank(plans, grids1, grids2, batches, time, log=lambda s: None):
    """The choice of least geometric mean over the batches, and every
    measurement, of `plans` ([(plan, its dict)]), time(plan, grid1, grid2, batch)
    in ms.  A batch that gives each pass-1 tile of every point a work-group of
    its own (up to 1024 of them) does not use grid1: it is timed once per plan
    and grid2, so that noise between equal calls ranks nothing."""
    best, results, legs = None, [], {}
    for p, d in plans:
        tiles1 = d["n2"] // d["cols"]
        uses = [m for m in batches if m * tiles1 > 1024]
        for g1 in grids1 if uses else (max(grids1),):
            for g2 in grids2:
                each = []
                for m in batches:
                    at = g1 if m in uses else max(grids1)
                    if (p, at, g2, m) not in legs:
                        legs[p, at, g2, m] = time(p, at, g2, m)
                    each.append(legs[p, at, g2, m])
                ms = math.exp(sum(math.log(t) for t in each) / len(each))
                results.append(dict(plan=p, grid1=g1, grid2=g2, ms=ms, each=each))
                if best is None or ms < best["ms"]:
                    best = dict(plan=p, grid1=g1, grid2=g2, ms=ms)
        log(f"plan {p}: best so far {best}")
    return best, results


def autotune(lengths=DEFAULT_LENGTHS, n_det=4, fs=2048.0, batch=None, reps=10, grids=None, out=fcas.TUNING_PATH,
             device=0, log=print, batches=(16, 256), grids1=GRIDS1, grids2=GRIDS2):
    """Times the plans of `lengths` and writes the choices to `out`.  `batch`: one
    batch in place of `batches`; `grids`: the work-group counts of both passes in
    place of `grids1` and `grids2`."""
    if batch is not None:
        batches = (batch,)
    if grids is not None:
        grids1 = grids2 = grids
    dev = torch.device("cuda", device)
    pos, ten = _network(n_det, dev)
    gen = torch.Generator(device="cpu").manual_seed(1234)
    results, choices = [], {}
    most = max(batches)
    for n in lengths:
        plans = [(p, d) for p, d in fcas.plans() if d["n"] == n]
        if not plans:
            continue
        half = n // 2 + 1
        xf = torch.complex(torch.randn(n_det, half, generator=gen, dtype=torch.float64),
                           torch.randn(n_det, half, generator=gen, dtype=torch.float64)).to(dev)
        psd = torch.ones(n_det, half, dtype=torch.float64, device=dev)
        u = torch.rand(most, 4, generator=gen, dtype=torch.float64)
        lo, hi = torch.tensor(BOX_LO, dtype=torch.float64), torch.tensor(BOX_HI, dtype=torch.float64)
        theta = (lo + u * (hi - lo)).to(dev)
        seg = torch.zeros(most, dtype=torch.int32, device=dev)
        # the long three-pass lengths are timed with the 4 GiB workspace their
        # searches use (36 hour-long points per launch, measured fastest)
        ws = min(4 << 30, most * 2 * n * 8) if n > 262144 else 0
        ctx = fcas.Context(pos, ten, fs=fs, f_low=30.0, f_high=1000.0, box_lo=BOX_LO, box_hi=BOX_HI,
                           max_batch=most, max_samples=n, device=device, tuning=None, workspace_bytes=ws)
        best, measured = rank(plans, grids1, grids2, batches,
                              lambda p, g1, g2, m: time_plan(ctx, p, g1, g2, xf, psd, theta[:m], seg[:m], reps),
                              lambda t: log(f"N={n} {t}"))
        results += [dict(n=n, **r) for r in measured]
        ctx.close()
        choices[str(n)] = best
        log(f"N={n}: chose {best}")
    doc = dict(device=torch.cuda.get_device_name(dev), n_det=n_det, batch=most, batches=list(batches), reps=reps,
               what="mean device time of one fitness call (set-up, passes, finalize), geometric mean over the batches",
               written=time.strftime("%Y-%m-%d %H:%M:%S"), choices=choices, measurements=results)
    if out:
        # every context reads `out` when it is created, so it holds the choices
        # alone; the measurements behind them go beside it
        for path, part in ((out, {k: v for k, v in doc.items() if k != "measurements"}),
                           (os.path.splitext(out)[0] + "_measurements.json", doc)):
            with open(path, "w") as fh:
                json.dump(part, fh, indent=1)
                fh.write("\n")
    return doc


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--lengths", default=",".join(str(n) for n in DEFAULT_LENGTHS))
    ap.add_argument("--out", default=fcas.TUNING_PATH)
    ap.add_argument("--reps", type=int, default=10)
    a = ap.parse_args(argv)
    autotune(tuple(int(x) for x in a.lengths.split(",")), reps=a.reps, out=a.out,
             log=lambda s: print(s, flush=True))


if __name__ == "__main__":
    sys.exit(main())
