"""The measured grid of the tuning table, without a GPU: which point a shape
takes, its class (whole 16-byte chunks or ragged), what comes before it, and
its file form.  Each case loads its own table in a process of its own."""
import json
import math
import os
import subprocess
import sys

from paper_1306_6192_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
POINTS = [32, 48] + [p << s for s in range(1, 8) for p in (32, 48)] + [8192]

LOOKUP = """
import ctypes, json, sys
sys.path.insert(0, %r)
from paper_1306_6192_amd import _lib
lib = _lib.load()
def look(mode, m, n, k):
    c, s = ctypes.c_int32(), ctypes.c_int32()
    _lib.check(lib.gemm_tuner_lookup(mode, m, n, k, ctypes.byref(c), ctypes.byref(s)))
    return c.value, s.value
out = [look(*q) for q in json.loads(sys.argv[1])]
if len(sys.argv) > 2:
    _lib.check(lib.gemm_tuner_save(sys.argv[2].encode()))
print(json.dumps(out))
"""


def lookups(table, shapes, save=None):
    env = dict(os.environ, MI355GEMM_TUNE_FILE=str(table))
    cmd = [sys.executable, "-c", LOOKUP % ROOT, json.dumps(shapes)] + ([str(save)] if save else [])
    r = subprocess.run(cmd, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [tuple(x) for x in json.loads(r.stdout.strip().splitlines()[-1])]


def line(mode, whole, i, j, choices):
    return ('{"grid": %d, "whole": %d, "m": %d, "n": %d, "choices": "' % (mode, whole, i, j)
            + " ".join("%d:%d" % c for c in choices) + '"}\n')


def nearest(d):
    if d <= 32:
        return 0
    return min(range(len(POINTS)), key=lambda i: abs(math.log(d) - math.log(POINTS[i])))


def test_every_dimension_takes_the_nearest_point(tmp_path):
    """k alone decides here (one row of the grid): the split written at point q
    is q + 1, so the lookup tells the point; all k around every turn."""
    f = tmp_path / "t.jsonl"
    f.write_text("".join(line(_lib.MODE_F32, w, 0, 0, [(6, q + 1) for q in range(len(POINTS))]) for w in (0, 1)))
    ks = sorted({max(1, int(p * r) + d) for p in POINTS for r in (1, math.sqrt(1.5), math.sqrt(4 / 3)) for d in (-1, 0, 1, 2)}
                | {1, 2, 31, 100000, 1 << 29})
    got = lookups(f, [(_lib.MODE_F32, 20, 30, k) for k in ks])
    assert [g[0] for g in got] == [6] * len(ks)
    assert [g[1] - 1 for g in got] == [nearest(k) for k in ks]


def test_class_and_order_of_the_table(tmp_path):
    """Whole chunks and ragged shapes have choices of their own (split-BF16x3:
    by n alone); an exact entry, then a bucket entry, come before the grid;
    F16 takes BF16's grid until it has one; a point not measured, an unknown
    configuration and a mode without a grid fall to the cost model."""
    n17 = len(POINTS)
    f = tmp_path / "t.jsonl"
    rows = [line(_lib.MODE_BF16, 1, 2, 2, [(3, 2)] * n17), line(_lib.MODE_BF16, 0, 2, 2, [(4, 1)] * n17),
            line(_lib.MODE_SPLIT_BF16X3, 1, 2, 2, [(2, 2)] * n17), line(_lib.MODE_SPLIT_BF16X3, 0, 2, 2, [(1, 1)] * n17),
            line(_lib.MODE_F8E4M3, 1, 2, 2, [(-1, 1), (9999, 1)] + [(5, 4)] * (n17 - 2)),
            '{"grid": 1, "whole": 2, "m": 0, "n": 0, "choices": "1:1"}\n', '{"grid": 1, "whole": 1, "m": 17, "n": 0, "choices": "1:1"}\n',
            '{"mode": 1, "m": 64, "n": 64, "k": 1000, "cfg": 0, "split": 3}\n',
            '{"bucket": "plain", "mode": 1, "bm": 6, "bn": 6, "bk": 11, "cfg": 1, "split": 5}\n']
    f.write_text("".join(rows))
    B, H, S, Q = _lib.MODE_BF16, _lib.MODE_F16, _lib.MODE_SPLIT_BF16X3, _lib.MODE_F8E4M3
    got = lookups(f, [(B, 64, 64, 64), (B, 64, 68, 64), (B, 64, 64, 65), (H, 64, 64, 64), (H, 64, 66, 64), (S, 64, 64, 65),
                      (S, 64, 65, 64), (B, 64, 64, 1000), (B, 65, 64, 1000), (B, 64, 64, 2048), (Q, 64, 64, 64)])
    assert got == [(3, 2), (4, 1), (4, 1), (3, 2), (4, 1), (2, 2), (1, 1), (0, 3), (3, 2), (1, 5), (5, 4)]
    other = lookups(f, [(Q, 64, 64, 32), (Q, 64, 64, 48), (_lib.MODE_F32, 64, 64, 64)])
    empty = tmp_path / "e.jsonl"
    empty.write_text("")
    assert other == lookups(empty, [(Q, 64, 64, 32), (Q, 64, 64, 48), (_lib.MODE_F32, 64, 64, 64)])


def test_grid_survives_save_and_load(tmp_path):
    f, g = tmp_path / "t.jsonl", tmp_path / "saved.jsonl"
    text = line(_lib.MODE_F32, 1, 3, 16, [(q % 5, 1 << (q % 7)) for q in range(len(POINTS))])
    f.write_text(text)
    a = lookups(f, [(_lib.MODE_F32, 96, 8192, p) for p in POINTS], save=g)
    assert text in g.read_text()
    assert lookups(g, [(_lib.MODE_F32, 96, 8192, p) for p in POINTS]) == a


def test_shipped_grid_is_complete_and_slabs_are_bounded():
    """Every point of the shipped table has a choice, and no shape, however
    large, is given slabs above what gemm_plain_noalloc holds."""
    seen = {}
    with open(os.path.join(ROOT, "paper_1306_6192_amd", "tuning", "mi355x.jsonl")) as f:
        for ln in f:
            if ln.startswith('{"grid"'):
                d = json.loads(ln)
                seen[(d["grid"], d["whole"], d["m"], d["n"])] = [tuple(map(int, c.split(":"))) for c in d["choices"].split()]
    for mode in (_lib.MODE_F32, _lib.MODE_BF16, _lib.MODE_F8E4M3, _lib.MODE_SPLIT_BF16X3):
        for w in (0, 1):
            for i in range(len(POINTS)):
                for j in range(len(POINTS)):
                    assert len(seen[(mode, w, i, j)]) == len(POINTS) and min(c for c, _ in seen[(mode, w, i, j)]) >= 0
    lib = _lib.load()
    import ctypes
    info = (ctypes.c_int32 * 6)()
    for mode in (_lib.MODE_F32, _lib.MODE_BF16, _lib.MODE_F16, _lib.MODE_F8E4M3):
        for m, n, k in ((1 << 20, 33, 4096), (40, 1 << 22, 8192), (100000, 100000, 100), (16, 1 << 26, 512), (8192, 8192, 1 << 25)):
            c, s = ctypes.c_int32(), ctypes.c_int32()
            _lib.check(lib.gemm_tuner_lookup(mode, m, n, k, ctypes.byref(c), ctypes.byref(s)))
            _lib.check(lib.gemm_config_info(mode, c, info))
            assert s.value == 1 or s.value <= info[3] or s.value * m * n * 4 <= _lib.NOALLOC_SCRATCH_BYTES


def test_slabs_are_bounded_by_fewer_ranges(tmp_path):
    """A shape larger than its point takes as many ranges as 64 MB of slabs
    hold, down to the ranges that need none."""
    f = tmp_path / "t.jsonl"
    f.write_text(line(_lib.MODE_F32, 0, 4, 16, [(6, 16)] * len(POINTS)) + line(_lib.MODE_F32, 0, 16, 16, [(6, 16)] * len(POINTS)))
    shapes = [(_lib.MODE_F32, m, n, 8191) for m, n in ((128, 8191), (129, 8191), (147, 7867), (155, 9001), (8191, 8191))]
    for (_, m, n, _), (cfg, split) in zip(shapes, lookups(f, shapes)):
        slab = (m * n + 3) // 4 * 16
        assert cfg == 6 and split == min(16, max(1, (64 << 20) // slab)), (m, n, split)


WS = """
import ctypes, json, sys
sys.path.insert(0, %r)
from paper_1306_6192_amd import _lib
lib = _lib.load()
def ws(mode, m, n, k, off):     # the addresses are not touched
    w = ctypes.c_uint64()
    p = _lib.problem(mode, m, n, k, (1 << 40) + off, k, (1 << 41) + off, n, 1 << 42, n)
    _lib.check(lib.gemm_plain_workspace_bytes(ctypes.byref(p), ctypes.byref(w)))
    return w.value
print(json.dumps([ws(*q) for q in json.loads(sys.argv[1])]))
"""


def workspaces(table, queries):
    env = dict(os.environ, MI355GEMM_TUNE_FILE=str(table)) if table else None
    r = subprocess.run([sys.executable, "-c", WS % ROOT, json.dumps(queries)], env=env, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])


def test_misaligned_operands_keep_the_waves_along_k(tmp_path):
    """A chunked configuration with waves along k has an any-shape form with as
    many: the ranges of a split factor up to them need no slabs on operands off
    16-byte alignment either (the figure reported beyond what is used stops at
    64 MB, so slabs that are used show above it).  k is below what is packed."""
    import ctypes
    lib = _lib.load()
    info = (ctypes.c_int32 * 6)()
    f = tmp_path / "t.jsonl"
    m, n, k = 4096, 4096, 384
    for mode in (_lib.MODE_F32, _lib.MODE_BF16, _lib.MODE_F16, _lib.MODE_F8E4M3):
        for cfg in range(lib.gemm_num_configs(mode)):
            _lib.check(lib.gemm_config_info(mode, cfg, info))
            waves_along_k = info[0] == 32 or (info[0] == 64 and info[1] == 64 and info[3] == 8)
            if not lib.gemm_config_chunk(mode, cfg) or not waves_along_k:
                continue
            f.write_text('{"mode": %d, "m": %d, "n": %d, "k": %d, "cfg": %d, "split": %d}\n' % (mode, m, n, k, cfg, info[3]))
            size = _lib.ELEM_SIZE[mode]
            assert max(workspaces(f, [(mode, m, n, k, off) for off in (0, size)])) <= _lib.NOALLOC_SCRATCH_BYTES, (mode, cfg)


def test_misaligned_operands_need_no_more_slabs_than_the_array_holds():
    """The shipped table on large flat outputs (below what is packed), aligned
    and one element off: what the allocation-free entry point holds suffices."""
    qs = [(mode, m, n, k, off * _lib.ELEM_SIZE[mode]) for mode in (_lib.MODE_F32, _lib.MODE_BF16, _lib.MODE_F16, _lib.MODE_F8E4M3)
          for m in (1, 16, 40, 64, 96, 128, 156) for n in (8192, 32768, 131072, 1 << 20, 1 << 22)
          for k in (256, 1024, 4096, 16384) for off in (0, 1)]
    for q, w in zip(qs, workspaces(None, qs)):
        assert w <= _lib.NOALLOC_SCRATCH_BYTES, (q, w)


def test_a_mostly_empty_round_takes_the_next_points_tile(tmp_path):
    """Above the workgroups that are resident at once (256 CUs), where the point
    was not: the configuration of the next point along the dimension further
    above, with the same k ranges; otherwise the point's own."""
    f = tmp_path / "t.jsonl"
    n17 = len(POINTS)
    # E4M3, ragged: configuration 15 (32x64, one workgroup per CU) at n = 2048, m = 256; up in m 14 (two per CU)
    # with the same ranges, up in n 6 with one; at m = 384 (nearest 384), up in m, 14 with other ranges
    rows = [line(_lib.MODE_F8E4M3, 0, 6, 12, [(15, 2)] * n17), line(_lib.MODE_F8E4M3, 0, 7, 12, [(14, 2)] * n17),
            line(_lib.MODE_F8E4M3, 0, 6, 13, [(6, 1)] * n17), line(_lib.MODE_F8E4M3, 0, 8, 12, [(14, 1)] * n17),
            line(_lib.MODE_SPLIT_BF16X3, 0, 6, 12, [(19, 2)] * n17), line(_lib.MODE_SPLIT_BF16X3, 0, 7, 12, [(18, 2)] * n17)]
    f.write_text("".join(rows))
    Q, S = _lib.MODE_F8E4M3, _lib.MODE_SPLIT_BF16X3
    k = 255
    shapes = [(Q, 256, 2047, k), (Q, 250, 2051, k), (Q, 257, 2047, k), (Q, 300, 2049, k), (Q, 257, 2070, k), (Q, 240, 2241, k),
              (Q, 256, 2047, 100), (Q, 257, 2047, 100), (S, 300, 2049, k)]
    # in one round; below the point in m and above in n: up in n, other ranges; up in m; further above in n; k of one range
    # (its neighbour's factor gives one range too); split-BF16x3: none
    want = [(15, 2), (15, 2), (14, 2), (14, 2), (15, 2), (15, 2), (15, 2), (14, 2), (19, 2)]
    assert lookups(f, shapes) == want


def test_the_next_points_tile_keeps_the_k_ranges(tmp_path):
    """Over the shipped table: a drawn shape's split factor gives the k ranges of
    its own point's."""
    import random
    grid = {}
    with open(os.path.join(ROOT, "paper_1306_6192_amd", "tuning", "mi355x.jsonl")) as fh:
        for ln in fh:
            if ln.startswith('{"grid"'):
                d = json.loads(ln)
                grid[(d["grid"], d["whole"], d["m"], d["n"])] = [tuple(map(int, c.split(":"))) for c in d["choices"].split()]
    table = tmp_path / "grid_only.jsonl"
    table.write_text("".join(line(*key, row) for key, row in grid.items()))
    r = random.Random(4)
    shapes = [(r.choice((0, 1, 3)), *(int(math.exp(r.uniform(math.log(17), math.log(4096)))) for _ in range(3))) for _ in range(4000)]
    grain, moved = {0: 32, 1: 64, 3: 128}, 0

    def ranges(mode, k, split):
        g = -(-k // grain[mode])
        return -(-g // -(-g // min(split, g)))

    for (mode, m, n, k), (cfg, split) in zip(shapes, lookups(table, shapes)):
        c = 16 // _lib.ELEM_SIZE[mode]
        own = grid[(mode, int(n % c == 0 and k % c == 0), nearest(m), nearest(n))][nearest(k)]
        moved += cfg != own[0]
        if own[1] * m * n * 4 <= _lib.NOALLOC_SCRATCH_BYTES:
            assert ranges(mode, k, split) == ranges(mode, k, own[1]), (mode, m, n, k, cfg, split, own)
    assert 0 < moved < 200, moved


def test_any_shape_tiles_of_the_rule():
    """The configurations that stand in for one that cannot run (any_shape_cfg
    names them by index): any-shape, of the tiles that were measured."""
    import ctypes
    lib = _lib.load()
    info = (ctypes.c_int32 * 6)()
    half = {6: (64, 64, 64, 4), 13: (128, 128, 32, 4), 24: (32, 64, 32, 4), 4: (128, 64, 64, 4)}
    want = {_lib.MODE_F32: {24: (64, 64, 32, 4), 25: (128, 128, 16, 4)}, _lib.MODE_BF16: half, _lib.MODE_F16: half,
            _lib.MODE_F8E4M3: {6: (64, 64, 128, 4), 11: (128, 128, 64, 4), 14: (32, 64, 64, 4), 4: (128, 64, 128, 4)},
            _lib.MODE_SPLIT_BF16X3: {5: (64, 64, 32, 4), 2: (128, 128, 32, 4)}}
    for mode, tiles in want.items():
        for cfg, tile in tiles.items():
            _lib.check(lib.gemm_config_info(mode, cfg, info))
            assert lib.gemm_config_chunk(mode, cfg) == 0 and tuple(info[:4]) == tile, (mode, cfg, list(info))
