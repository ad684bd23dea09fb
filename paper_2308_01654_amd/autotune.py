"""Autotuner of the iteration kernel's launch shape.

For every shape bucket -- K in powers of two, T buckets (<=16, <=32, <=64,
<=128, <=256, >256) and circle-count buckets (0, <=16, <=64, <=256, >256) -- it runs
a representative sine-lane instance with every lanes-per-sample shape
(1, 2, 4, 8, 16), each with the iteration kernel that the library launches
there: the split kernel by its own rule, elsewhere the faster of k_batch's two
compilations (the second, for five waves per SIMD, at 8 or 16 lanes).  Whole
iterations are timed with HIP events.  For the fastest number of lanes it then
times k_batch, which steps in a batch may get where a step alone gets the split
kernel: with and without the tiles' LDS copy of their perturbations, and both
compilations.  The choices are written as a line "k_log2 t_bucket c_bucket
lanes stage occupancy" of ``tuning.txt``.
The library reads that file at its first launch (next to libmppi.so, or the
file named by MPPI_TUNING_FILE).  A bucket's lanes depend only on the
instance's own shape, so an instance computes the same bits alone and inside
any batch.

Usage (on the GPU): python -m paper_2308_01654_amd.autotune [--out PATH] [--quick]
"""
from __future__ import annotations

import argparse
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

T_REPS = {0: 16, 1: 30, 2: 60, 3: 100, 4: 200, 5: 400}
C_REPS = {0: 0, 1: 12, 2: 60, 3: 200, 4: 512}
LANES = (1, 2, 4, 8, 16)


def shape_scene(K, T, n_c):
    from paper_2308_01654_amd import scenes
    rng = np.random.Generator(np.random.PCG64(K * 1000 + T * 7 + n_c))
    p = scenes.params(K=K, T=T, dt=0.05, v_max=15.0, seed=17)
    return dict(params=p, x0=scenes._sine_x0(), waypoints=scenes.sine_lane(v_ref=15.0),
                circles=scenes.sine_circles(rng, n_c))


SPLIT = 2  # Planner.kernel() of the split kernel


def time_shape(sc, lanes, reps, rounds=3, stage=1, occ=-1):
    """(ms, kernel): best of `rounds` HIP-event timings of `reps` back-to-back
    iterations (the best filters out the other work of a shared GPU), and the
    iteration kernel they ran.  occ: -1 the library's choice of the kernel, 0 or
    1 a compilation of k_batch."""
    from paper_2308_01654_amd import mppi
    from paper_2308_01654_amd.hip_events import time_steps
    pl = mppi.Planner(sc["params"], lanes=lanes)
    try:
        pl.set_staging(stage)
        pl.set_occupancy(occ)
        pl.set_scene(sc["x0"], sc["waypoints"], sc["circles"])
        pl.step_resident(sc["x0"])
        pl.sync()
        return min(time_steps(pl, sc["x0"], reps) for _ in range(rounds)), pl.kernel()
    finally:
        pl.close()


def tune_shape(sc, lanes, reps):
    """(times by lanes, lanes, stage, occupancy, times of k_batch by (stage,
    occupancy)) of one shape."""
    def compilations(g):
        return (0, 1) if g >= 8 else (0,)

    times = {}
    for g in lanes:
        ms, kernel = time_shape(sc, g, reps)
        if kernel != SPLIT:
            ms = min(time_shape(sc, g, reps, occ=o)[0] for o in compilations(g))
        times[g] = ms
    best = min(times, key=times.get)
    k_batch = {(s, 0): time_shape(sc, best, reps, stage=s, occ=0)[0] for s in (1, 0)}
    stage = min(k_batch, key=k_batch.get)[0]
    for o in compilations(best)[1:]:
        k_batch[(stage, o)] = time_shape(sc, best, reps, stage=stage, occ=o)[0]
    occ = min((o for s, o in k_batch if s == stage), key=lambda o: k_batch[(stage, o)])
    return times, best, stage, occ, k_batch


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--out", default=os.path.join(HERE, "tuning.txt"))
    ap.add_argument("--k-min", type=int, default=10)
    ap.add_argument("--k-max", type=int, default=18)
    ap.add_argument("--t-buckets", default="0,1,2,3,4,5")
    ap.add_argument("--c-buckets", default="0,1,2,3,4")
    args = ap.parse_args(argv)
    lines = ["# launch-shape tuning table of the MPPI iteration kernel",
             "# written by: python -m paper_2308_01654_amd.autotune (HIP-event iteration time, "
             "best of 3 rounds, fastest of lanes 1/2/4/8/16 with the kernel launched there, "
             "then of k_batch at that shape LDS staging of the perturbations on (1) or off "
             "(0), then at 8 or 16 lanes its compilation: default (0) or five waves per SIMD "
             "(1))",
             "# columns: k_log2 t_bucket c_bucket lanes stage occupancy   (t: <=16,<=32,<=64,"
             "<=128,<=256,>256; c: 0,<=16,<=64,<=256,>256)"]
    t0 = time.time()
    tmp = args.out + ".partial"
    with open(tmp, "w") as f:  # rows are appended as they are measured
        f.write("\n".join(lines) + "\n")
    for kb in range(args.k_min, args.k_max + 1):
        K = 1 << kb
        for tb in [int(v) for v in args.t_buckets.split(",")]:
            T = T_REPS[tb]
            for cb in [int(v) for v in args.c_buckets.split(",")]:
                sc = shape_scene(K, T, C_REPS[cb])
                reps = 20 if K * T < 2_000_000 else 3
                times, best, stage, occ, k_batch = tune_shape(sc, [g for g in LANES if g <= T], reps)
                lines.append("%d %d %d %d %d %d" % (kb, tb, cb, best, stage, occ))
                with open(tmp, "a") as f:
                    f.write(lines[-1] + "\n")
                print("K=%-7d T=%-4d circles=%-4d " % (K, T, C_REPS[cb]) +
                      " ".join("g%d=%.4fms" % (g, ms) for g, ms in times.items()) +
                      "".join(" k_batch-g%d-stage%d-occ%d=%.4fms" % ((best,) + so + (ms,))
                              for so, ms in k_batch.items()) +
                      "  -> %d %d %d  (%.0fs)" % (best, stage, occ, time.time() - t0), flush=True)
    os.replace(tmp, args.out)
    print("wrote", args.out, flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
