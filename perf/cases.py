"""Performance cases: the products that programs built on this package run.

Every case is one pass through public entry points of ``paper_1306_6192_amd``:

* ``gemm``: one plain product (``gemm``, ``gemm_f64``, ``gemm_c32``).  With
  ``prep`` the left operand arrives as float32, as an activation does, and is
  brought into the reduced precision inside the pass (``convert``,
  ``quantize_e4m3``); the right operand is a weight the program holds in that
  precision.
* ``grouped``: a list of independent products in one launch (``ProblemBatch``,
  built once and run again and again).
* ``serve``: a burst of mixed requests submitted to a running ``Server``, until
  the last has finished.

Sizes are those of the benchmark, the tests and the tuning ranges (squares of
512 and 8192, (128, 8192, 8192), 512 problems of 32..1024, 48 requests of
64..4096) or generic ones beside them.  Inputs are uniform[-1, 1] for the
full-precision forms and N(0, 1) for the reduced ones, as in the benchmark.
"""
import math
import random

import torch

import paper_1306_6192_amd as mg
from paper_1306_6192_amd import _lib

MODES = {"f32": mg.MODE_F32, "bf16": mg.MODE_BF16, "f16": mg.MODE_F16, "e4m3": mg.MODE_F8E4M3,
         "split": mg.MODE_SPLIT_BF16X3}
ELEM = {"f32": 4, "bf16": 2, "f16": 2, "e4m3": 1, "split": 4, "f64": 8, "c32": 8}
SERVE_MIX = (("f32", 0.50), ("bf16", 0.85), ("e4m3", 1.0))   # cumulative shares of the served requests
ALIGN = 256   # elements between the starts of two matrices of a pool (at least 256 bytes)


def _gemm(name, dtype, m, n, k, prep=False):
    return {"name": name, "kind": "gemm", "dtype": dtype, "m": m, "n": n, "k": k, "prep": prep}


def listed():
    return [
        # the smallest call: one 64-square block product, where launch latency is everything
        _gemm("f32_64", "f32", 64, 64, 64),
        # the correctness configuration: a small product that does not fill the chip by itself
        _gemm("f32_512", "f32", 512, 512, 512),
        # the benchmark's dominant product
        _gemm("f32_8192", "f32", 8192, 8192, 8192),
        # the benchmark's skinny product: a batch of 128 rows against a large weight
        _gemm("f32_rows128", "f32", 128, 8192, 8192),
        # a few rows against a large 16-bit weight, as a program that generates step by step calls it
        _gemm("bf16_rows16", "bf16", 16, 8192, 8192),
        # a large 16-bit product from float32 activations
        _gemm("bf16_8192_prep", "bf16", 8192, 8192, 8192, True),
        # a mid-size 16-bit product whose dimensions are multiples of nothing
        _gemm("f16_ragged", "f16", 2047, 1999, 2501),
        # an 8-bit product with per-tensor quantisation of its float32 activations
        _gemm("e4m3_4096_prep", "e4m3", 4096, 4096, 4096, True),
        # a float32 product through the compensated bfloat16 form
        _gemm("split_2048", "split", 2048, 2048, 2048),
        # the double column of the paper's comparison, at a size where the chip is not yet full
        _gemm("f64_1024", "f64", 1024, 1024, 1024),
        # the grouped workload: many small independent products in one launch
        {"name": "grouped_bf16_512", "kind": "grouped", "dtype": "bf16", "count": 512, "lo": 32, "hi": 1024,
         "dims_seed": 0},
        # a serving burst over the request sizes and types of the serving workload
        {"name": "serve_48", "kind": "serve", "count": 48, "lo": 64, "hi": 4096, "dims_seed": 0},
    ]


def _log(rng, lo, hi):
    """A whole number log-uniform in [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.random()
    if what < 0.2:
        return {"kind": "grouped", "dtype": rng.choice(["f32", "bf16", "f16", "split"]), "count": _log(rng, 16, 512),
                "lo": 32, "hi": 1024, "dims_seed": rng.randrange(1 << 20)}
    if what < 0.3:
        return {"kind": "serve", "count": _log(rng, 4, 48), "lo": 64, "hi": 4096, "dims_seed": rng.randrange(1 << 20)}
    dtype = rng.choice(["f32", "f32", "bf16", "bf16", "f16", "e4m3", "split", "f64", "c32"])
    if rng.random() < 0.35:      # a few rows against a large right operand
        m, n, k = _log(rng, 1, 256), _log(rng, 1024, 8192), _log(rng, 1024, 8192)
    else:
        m, n, k = _log(rng, 32, 4096), _log(rng, 32, 4096), _log(rng, 32, 4096)
    if rng.random() < 0.5:       # half of the products have the round sizes of a chosen width
        n, k = (max(64, v // 64 * 64) for v in (n, k))
    return {"kind": "gemm", "dtype": dtype, "m": m, "n": n, "k": k,
            "prep": dtype in ("bf16", "f16", "e4m3") and rng.random() < 0.5}


def problems(case):
    """(dtype, m, n, k) of every product of one pass."""
    if case["kind"] == "gemm":
        return [(case["dtype"], case["m"], case["n"], case["k"])]
    r = random.Random(case["dims_seed"])
    out = []
    for _ in range(case["count"]):
        m, n, k = (_log(r, case["lo"], case["hi"]) for _ in range(3))
        u = r.random()
        out.append((case.get("dtype") or next(d for d, share in SERVE_MIX if u < share), m, n, k))
    return out


# --------------------------------------------------------------------------
# Inputs, in plain torch: from the seed alone.

def _random(count, dtype, g):
    """`count` float32 (or wider) values of the dtype's distribution."""
    if dtype == "f64":
        return torch.rand(count, dtype=torch.float64, device="cuda", generator=g) * 2 - 1
    if dtype == "c32":
        return torch.view_as_complex(torch.rand((count, 2), device="cuda", generator=g) * 2 - 1)
    if dtype in ("f32", "split"):
        return torch.rand(count, device="cuda", generator=g) * 2 - 1
    return torch.randn(count, device="cuda", generator=g)


def _quantise(x):
    """Per-tensor E4M3: codes and scale = amax / 448 in float32."""
    s = x.abs().max() / 448.0
    return (x / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8), s


def _reduce(x, dtype):
    """`x` in the product's element type, and its scale (1 but for e4m3)."""
    if dtype == "bf16":
        return x.to(torch.bfloat16), 1.0
    if dtype == "f16":
        return x.to(torch.float16), 1.0
    if dtype == "e4m3":
        q, s = _quantise(x)
        return q, float(s)
    return x, 1.0


def _pair(case, seed):
    """(A, B, scale_a, scale_b) of a plain product; A is float32 with `prep`."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    d, m, n, k = case["dtype"], case["m"], case["n"], case["k"]
    a = _random(m * k, d, g).view(m, k)
    b, sb = _reduce(_random(k * n, d, g).view(k, n), d)
    sa = 1.0
    if not case["prep"]:
        a, sa = _reduce(a, d)
    return a, b, sa, sb


def _pool(sizes, dtype, g):
    """Matrices of the given (rows, columns) as views of one pool, each start aligned, and the pool's scale."""
    starts, at = [], 0
    for r, c in sizes:
        starts.append(at)
        at += (r * c + ALIGN - 1) // ALIGN * ALIGN
    pool, s = _reduce(_random(max(at, 1), dtype, g), dtype)
    return [pool[o:o + r * c].view(r, c) for o, (r, c) in zip(starts, sizes)], s


def _many(case, seed):
    """[(A, B, C, mode, scale_a, scale_b)] of a grouped or served list in its order, and the buffer that holds every C, one after the other."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    ps = problems(case)
    out = torch.zeros(sum(m * n for _, m, n, _ in ps), device="cuda")
    done, at = [None] * len(ps), 0
    cs = []
    for _, m, n, _ in ps:
        cs.append(out[at:at + m * n].view(m, n))
        at += m * n
    for d in sorted({p[0] for p in ps}):
        idx = [i for i, p in enumerate(ps) if p[0] == d]
        a, sa = _pool([(ps[i][1], ps[i][3]) for i in idx], d, g)
        b, sb = _pool([(ps[i][3], ps[i][2]) for i in idx], d, g)
        for j, i in enumerate(idx):
            done[i] = (a[j], b[j], cs[i], MODES[d], sa, sb)
    return done, out


# --------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "gemm":
        a, b, sa, sb = _pair(case, seed)
        return {"kind": "gemm", "dtype": case["dtype"], "prep": case["prep"], "a": a, "b": b, "sa": sa, "sb": sb}
    ps, out = _many(case, seed)
    if case["kind"] == "grouped":
        batch = mg.ProblemBatch([(a, b, c) for a, b, c, _, _, _ in ps], MODES[case["dtype"]])
        return {"kind": "grouped", "batch": batch, "out": out}
    probs = [mg.make_problem(a, b, c, mode, sa, sb) for a, b, c, mode, sa, sb in ps]
    return {"kind": "serve", "server": mg.Server(), "probs": probs, "keep": ps, "out": out}


def run(state):
    if state["kind"] == "grouped":
        mg.grouped(state["batch"])
        return state["out"]
    if state["kind"] == "serve":
        server = state["server"]
        for p in state["probs"]:
            _lib.check(server.submit(p)[0])
        server.drain()
        return state["out"]
    d, a, b = state["dtype"], state["a"], state["b"]
    if d == "f64":
        return mg.gemm_f64(a, b)
    if d == "c32":
        return mg.gemm_c32(a, b)
    if not state["prep"]:
        return mg.gemm(a, b, mode=MODES[d], scale_a=state["sa"], scale_b=state["sb"])
    if d == "e4m3":
        q, s = mg.quantize_e4m3(a)
        # the product takes its scales as numbers, so the program reads the scale back
        return mg.gemm(q, b, mode=MODES[d], scale_a=float(s), scale_b=state["sb"]), q, s
    q = mg.convert(a, MODES[d])
    return mg.gemm(q, b, mode=MODES[d]), q


def work(case):
    nbytes = flops = 0
    for d, m, n, k in problems(case):
        es = ELEM[d]
        nbytes += es * (m * k + k * n) + (es if d in ("f64", "c32") else 4) * m * n
        flops += (8 if d == "c32" else 2) * m * n * k
        if case.get("prep"):
            # the float32 activations are what comes in; their codes go out besides
            nbytes += 4 * m * k
    return {"bytes": nbytes, "flops": flops}


def _codes64(x, dtype):
    """A product operand's values in binary64."""
    return x.view(torch.float8_e4m3fn).double() if dtype == "e4m3" else x.double()


def exact(case, seed):
    if case["kind"] != "gemm":
        names = {v: k for k, v in MODES.items()}
        ps, _ = _many(case, seed)
        return torch.cat([((_codes64(a, names[mode]) @ _codes64(b, names[mode])) * (sa * sb)).reshape(-1)
                          for a, b, _, mode, sa, sb in ps])
    d = case["dtype"]
    a, b, sa, sb = _pair(case, seed)
    if d == "c32":
        return a.to(torch.complex128) @ b.to(torch.complex128)
    if case["prep"]:
        q, sa = _reduce(a, d)
        c = (_codes64(q, d) @ _codes64(b, d)) * (sa * sb)
        return (c, None, None) if d == "e4m3" else (c, q.double())
    return (_codes64(a, d) @ _codes64(b, d)) * (sa * sb)
