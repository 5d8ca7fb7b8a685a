"""Measure tile configurations on the current GPU and write the tuning table
the library loads at start-up.

    python -m paper_1306_6192_amd.tune [--out PATH] [--what exact,grid,grouped]

Kinds of entries (each chosen by the library's own timing):

* ``exact``: the configuration and split-K factor of each benchmark shape
  (``gemm_tune``: every legal configuration and split-K factor, timed with
  HIP events on non-zero operands; the near-ties are re-timed and the fastest
  kept), keyed by (mode, m, n, k);
* ``grid``: the fastest configuration and split-K factor at every combination
  of the points 32, 48, 64, 96, ... 8192 of m, n and k, for shapes of whole
  16-byte chunks and for ragged ones (FP32, BF16 -- which F16 shares -- E4M3
  and split-BF16x3), consulted for every shape without an exact or bucket
  entry; each candidate is timed as a graph of back-to-back launches;
* ``plain-buckets`` (not in the shipped table): the measurement of ``exact`` on
  one representative shape per log2 bucket of (m, n, k) (``gemm_tune_bucket``),
  consulted before the grid;
* ``grouped``: the plain tile (128x128 or 64x64) per bucket for a problem
  launched alone (``gemm_tune_grouped``), and per mode the grouped kernel
  variant (one tile at three workgroups per CU, or two tiles with a cost
  model) and the small-tile efficiency of that cost model, measured on a
  mixed batch of seeded synthetic problems (``gemm_tune_grouped_mix``): 512 problems with m, n, k
  log-uniform in [32, 1024] (the grouped workload's distribution, another
  seed) for FP32, BF16, F16 and split-BF16x3, and 48 problems with m, n, k
  log-uniform in [64, 4096] (a serving batch) for E4M3.

The grouped buckets cover the grouped workload (dims log-uniform in [32, 1024],
FP32 and BF16) and the serving workload (dims log-uniform in [64, 4096], FP32,
BF16 and E4M3).  The representative shape of bucket b is the geometric mean of
the part of [2^b, 2^(b+1)) the workloads cover.  The table is saved after
every mode, so an interrupted run keeps what it measured.
"""
from __future__ import annotations

import argparse
import itertools
import math
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT_TABLE = os.path.join(HERE, "tuning", "mi355x.jsonl")

PLAIN_F32 = [(2048, 2048, 2048), (4096, 4096, 4096), (8192, 8192, 8192), (8192, 1024, 4096), (128, 8192, 8192),
             (512, 512, 512)]
SQUARES = [(2048, 2048, 2048), (4096, 4096, 4096), (8192, 8192, 8192)]

# dimension ranges of the workloads whose shapes are tuned per bucket
GROUPED_RANGE = (32, 1024)
SERVING_RANGE = (64, 4096)


def exact_shapes(mg):
    out = [(mg.MODE_F32, s) for s in PLAIN_F32]
    for mode in (mg.MODE_BF16, mg.MODE_F16, mg.MODE_F8E4M3, mg.MODE_SPLIT_BF16X3):
        out += [(mode, s) for s in SQUARES]
    return out


def bucket_reps(lo: int, hi: int):
    """(bucket, representative dimension) of every log2 bucket meeting [lo, hi]."""
    out = []
    for b in range(int(math.log2(lo)), int(math.log2(hi)) + 1):
        a, z = max(lo, 1 << b), min(hi, (1 << (b + 1)) - 1)
        if a <= z:
            out.append((b, int(round(math.sqrt(a * z)))))
    return out


def bucket_shapes(mg):
    """{mode: [representative (m, n, k)]} over the grouped and serving ranges."""
    ranges = {mg.MODE_F32: [GROUPED_RANGE, SERVING_RANGE], mg.MODE_BF16: [GROUPED_RANGE, SERVING_RANGE],
              mg.MODE_F8E4M3: [SERVING_RANGE]}
    out = {}
    for mode, rs in ranges.items():
        reps = {}
        for lo, hi in rs:
            for b, d in bucket_reps(lo, hi):
                reps.setdefault(b, []).append(d)
        # one representative per bucket (the lower one where both ranges
        # cover it: the grouped range ends at 1024)
        dims = [(b, sorted(ds)[(len(ds) - 1) // 2]) for b, ds in sorted(reps.items())]
        out[mode] = [(m, n, k) for (_, m), (_, n), (_, k) in itertools.product(dims, dims, dims)]
    return out


# The points of the measured grid: 2^b and 1.5 2^b from 32 to 8192.
GRID_POINTS = [32, 48] + [p << s for s in range(1, 8) for p in (32, 48)] + [8192]


def grid_shape(mg, mode, whole, i, j, q):
    """The shape measured for grid point (i, j, q): the point itself for whole
    16-byte chunks, odd dimensions just below it for ragged shapes; 16 rows
    stand for the first point of m, which all smaller m take too."""
    m, n, k = GRID_POINTS[i], GRID_POINTS[j], GRID_POINTS[q]
    if i == 0:
        m = 16
    if not whole:
        m, n, k = (max(3, int(d * 0.96)) | 1 for d in (m, n, k))
    return m, n, k


def grid_operands(mg, torch, mode, m, n, k, sets):
    out = []
    for _ in range(sets):
        a, b = torch.rand((m, k), device="cuda") * 2 - 1, torch.rand((k, n), device="cuda") * 2 - 1
        if mode in (mg.MODE_BF16, mg.MODE_F16):
            a, b = mg.convert(a, mode), mg.convert(b, mode)
        elif mode == mg.MODE_F8E4M3:
            a, b = mg.quantize_e4m3(a)[0], mg.quantize_e4m3(b)[0]
        out.append((a, b))
    return out


def grid_time(torch, stream, launch, reps, rounds):
    """Microseconds of one launch: `reps` of them captured in a graph, the best
    of `rounds` replays (launches back to back, as a program enqueues them)."""
    launch(0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        for r in range(reps):
            launch(r)
    best = float("inf")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(rounds):
        e0.record(stream)
        g.replay()
        e1.record(stream)
        stream.synchronize()
        best = min(best, e0.elapsed_time(e1) / reps * 1e3)
    return best


def k_ranges(mg, mode, info, k, split):
    """The k ranges that a split-K factor gives at `k`: whole grains (32 k for
    FP32 and split-BF16x3, 64 for BF16 and F16, 128 for FP8) each.  A factor
    that the waves along k of a small tile take costs nothing and stands."""
    if split <= info["waves"] and (info["BM"] < 64 or info["BM"] * info["BN"] == 4096 and info["waves"] == 8):
        return split
    grain = {mg.MODE_F32: 32, mg.MODE_SPLIT_BF16X3: 32, mg.MODE_F8E4M3: 128}.get(mode, 64)
    grains = -(-k // grain)
    return -(-grains // -(-grains // min(split, grains)))


def grid_candidates(mg, mode, infos, m, n, k):
    """(configuration, split) pairs worth timing: no 256-wide tile on a
    dimension of at most half of it, no split into ranges below 32 k, slabs of
    at most 64 MB, large outputs without large splits.  The split is the number
    of ranges it makes at this k: a factor that has fewer grains to deal out
    here would make more at the point's larger k."""
    for c, info in enumerate(infos):
        if (info["BM"] >= 256 and m <= 128) or (info["BN"] >= 256 and n <= 128):
            continue
        if info["BM"] >= 128 and m <= 32 and n * k < 1 << 20:
            continue
        if info["BM"] * info["BN"] <= 4096 and m * n > 1 << 24:
            continue
        split, last = 1, 0
        while split <= 64 and (split == 1 or k // split >= 32):
            if split > 1 and split * m * n * 4 > 64e6 or split > 4 and m * n > 1 << 21:
                break
            if k_ranges(mg, mode, info, k, split) != last:
                last = k_ranges(mg, mode, info, k, split)
                yield c, last
            split *= 2


def measure_grid(mg, _lib, torch, mode, path, limit_s):
    """Measure the grid points of a mode that the table at `path` lacks, and
    append their lines to it; stops after `limit_s` seconds (run again to go
    on)."""
    infos = [mg.config_info(mode, c) for c in range(mg.num_configs(mode))]
    chunks = [mg.config_chunk(mode, c) for c in range(len(infos))]
    es = _lib.ELEM_SIZE[mode]
    have = set()
    if os.path.exists(path):
        with open(path) as f:
            have = {ln.split(', "choices"')[0] for ln in f if ln.startswith('{"grid": %d,' % mode)}
    t0 = time.time()
    stream = torch.cuda.Stream()
    for whole, i, j in itertools.product((1, 0), range(len(GRID_POINTS)), range(len(GRID_POINTS))):
        head = '{"grid": %d, "whole": %d, "m": %d, "n": %d' % (mode, whole, i, j)
        if head in have:
            continue
        if time.time() - t0 > limit_s:
            return False
        row = []
        for q in range(len(GRID_POINTS)):
            m, n, k = grid_shape(mg, mode, whole, i, j, q)
            sets = max(1, min(3, int(6e8 / ((m * k + k * n) * es))))
            with torch.cuda.stream(stream):
                ops = grid_operands(mg, torch, mode, m, n, k, sets)
                out = torch.empty((m, n), device="cuda")

                def launcher(c, sp):
                    return lambda r: mg.gemm(ops[r % sets][0], ops[r % sets][1], out=out, mode=mode, cfg=c, split_k=sp)

                large = 2.0 * m * n * k > 2e9
                first = sorted((grid_time(torch, stream, launcher(c, sp), 3, 1), c, sp)
                               for c, sp in grid_candidates(mg, mode, infos, m, n, k)
                               if whole or not chunks[c] or min(m, n) >= 157 and k >= 444)
                close = [(c, sp) for t, c, sp in first[:12] if t < 1.25 * first[0][0] + 1]
                fine = min((grid_time(torch, stream, launcher(c, sp), 4 if large else 8, 3), c, sp) for c, sp in close)
            row.append((fine[1], fine[2]))
            del ops, out
        with open(path, "a") as f:
            f.write(head + ', "choices": "' + " ".join("%d:%d" % cs for cs in row) + '"}\n')
        if j == len(GRID_POINTS) - 1:
            print(f"grid {mg.MODE_NAMES[mode]} {'whole' if whole else 'ragged'} m point {i}: {time.time() - t0:.0f} s",
                  flush=True)
    return True


def calibrate_mix(mg, _lib, lib, torch, mode, count, lo, hi, stream):
    """gemm_tune_grouped_mix on `count` seeded problems with dims log-uniform
    in [lo, hi] (seed 100, not the benchmark's), operands uniform[-1, 1]
    on the device in the mode's element type."""
    # the seeded input generators live beside the package, at the
    # repository root
    root = os.path.dirname(HERE)
    if root not in sys.path:
        sys.path.insert(0, root)
    import synth
    g = torch.Generator(device="cuda").manual_seed(100)
    ops = []
    for m, n, k in synth.loguniform_dims(count, lo, hi, seed=100).tolist():
        a = torch.rand((m, k), device="cuda", generator=g) * 2 - 1
        b = torch.rand((k, n), device="cuda", generator=g) * 2 - 1
        if mode in (mg.MODE_BF16, mg.MODE_F16):
            a, b = mg.convert(a, mode), mg.convert(b, mode)
        elif mode == mg.MODE_F8E4M3:
            a, _ = mg.quantize_e4m3(a)
            b, _ = mg.quantize_e4m3(b)
        ops.append((a, b, torch.empty((m, n), device="cuda")))
    probs = [mg.make_problem(a, b, c, mode) for a, b, c in ops]
    torch.cuda.synchronize()
    _lib.check(lib.gemm_tune_grouped_mix(_lib.problems_array(probs), len(probs), stream))


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--out", default=DEFAULT_TABLE)
    ap.add_argument("--what", default="exact,grid,grouped")
    ap.add_argument("--modes", default="", help="comma-separated mode names to tune (default: all)")
    ap.add_argument("--limit", type=float, default=3600.0, help="seconds for the grid; a later run goes on")
    args = ap.parse_args(argv)
    what = set(args.what.split(","))
    import torch

    import paper_1306_6192_amd as mg
    from paper_1306_6192_amd import _lib
    torch.cuda.set_device(0)
    lib = mg.load()
    stream = torch.cuda.current_stream().cuda_stream
    os.makedirs(os.path.dirname(os.path.abspath(args.out)), exist_ok=True)

    def save():
        _lib.check(lib.gemm_tuner_save(args.out.encode()))

    keep = {mode for mode, name in mg.MODE_NAMES.items() if not args.modes or name in args.modes.split(",")}
    if "exact" in what:
        for mode, (m, n, k) in exact_shapes(mg):
            if mode not in keep:
                continue
            cfg, split = mg.tune(mode, m, n, k)
            info = mg.config_info(mode, cfg)
            print(f"{mg.MODE_NAMES[mode]:>13} {m}x{n}x{k}: cfg {cfg} ({info['BM']}x{info['BN']}x{info['BK']}) "
                  f"split {split}", flush=True)
        save()
    if "grouped" in what:
        mixes = {mg.MODE_F32: (512, 32, 1024), mg.MODE_BF16: (512, 32, 1024), mg.MODE_F16: (512, 32, 1024),
                 mg.MODE_SPLIT_BF16X3: (512, 32, 1024), mg.MODE_F8E4M3: (48, 64, 4096)}
        for mode, (count, lo, hi) in mixes.items():
            if mode not in keep:
                continue
            calibrate_mix(mg, _lib, lib, torch, mode, count, lo, hi, stream)
            print(f"grouped mix {mg.MODE_NAMES[mode]}: kernel variant and small-tile efficiency measured", flush=True)
        save()
    if "grid" in what:
        save()   # what the library holds (the grid lines it loaded among it), to which new lines are appended
        for mode in (mg.MODE_F32, mg.MODE_BF16, mg.MODE_F8E4M3, mg.MODE_SPLIT_BF16X3):
            if mode in keep and not measure_grid(mg, _lib, torch, mode, args.out, args.limit):
                print("the grid is not complete: run again", flush=True)
                return 1
        _lib.check(lib.gemm_tuner_load(args.out.encode()))
    buckets = bucket_shapes(mg)
    for kind, entry in (("plain-buckets", lib.gemm_tune_bucket), ("grouped", lib.gemm_tune_grouped)):
        if kind not in what:
            continue
        for mode, shapes in buckets.items():
            if mode not in keep:
                continue
            t0 = time.time()
            for i, (m, n, k) in enumerate(shapes):
                _lib.check(entry(mode, m, n, k, stream))
                if i % 64 == 63:
                    print(f"{kind} {mg.MODE_NAMES[mode]}: {i + 1}/{len(shapes)} ({time.time() - t0:.0f} s)",
                          flush=True)
            save()
            print(f"{kind} {mg.MODE_NAMES[mode]}: {len(shapes)} buckets in {time.time() - t0:.0f} s", flush=True)
    print(f"wrote {args.out}")


if __name__ == "__main__":
    sys.exit(main())
