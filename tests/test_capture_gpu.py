"""Products captured into graphs: a graph's workspace is its own.

Replays are compared bit by bit with the eager results, with eager work of the
same entry points on the captured stream in between (larger, so that the
stream's workspace grows after the capture) and beside them (unordered with the
replay), and the memory goes back once the graph is destroyed."""
import ctypes
import gc

import numpy as np
import pytest

import synth
from paper_1306_6192_amd import _lib
from tests._gpu import dev, host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402


def operands(mode, m, n, k, seed):
    A, B = synth.pair(m, n, k, seed=seed)
    a, b = dev(A), dev(B)
    if mode in (mg.MODE_BF16, mg.MODE_F16):
        a, b = mg.convert(a, mode), mg.convert(b, mode)
    elif mode == mg.MODE_F8E4M3:
        a, b = mg.quantize_e4m3(a)[0], mg.quantize_e4m3(b)[0]
    return a, b


def copies_config(mode):
    """A configuration that runs a ragged product on operand copies."""
    return next(c for c in range(mg.num_configs(mode)) if mg.config_chunk(mode, c))


# (mode, configuration, k ranges): operand copies, pre-split copies (split-BF16x3
# configuration 6), split-K slabs, and copies behind slabs
FORMS = [("copies", mg.MODE_BF16, None, 1), ("presplit", mg.MODE_SPLIT_BF16X3, 6, 1), ("slabs", mg.MODE_F32, 0, 3),
         ("copies behind slabs", mg.MODE_F8E4M3, None, 2)]


@pytest.mark.parametrize("name,mode,cfg,split", FORMS, ids=[f[0] for f in FORMS])
def test_replays_beside_eager_work_on_the_captured_stream(name, mode, cfg, split):
    log(f"capture {name}")
    cfg = copies_config(mode) if cfg is None else cfg
    kw = dict(mode=mode, cfg=cfg, split_k=split)
    # the second product needs a larger workspace than the first, the eager one a larger one still
    sizes = [(200, 301, 451), (333, 463, 601), (777, 1001, 901)]
    ops = [operands(mode, *s, seed=i) for i, s in enumerate(sizes)]
    want = [host(mg.gemm(a, b, **kw)) for a, b in ops]
    outs = [torch.empty(s[:2], device="cuda") for s in sizes]
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):        # the stream's workspace holds the first product before the capture
        mg.gemm(*ops[0], out=outs[0], **kw)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        for i in range(2):
            mg.gemm(*ops[i], out=outs[i], **kw)
    for _ in range(4):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(3):
                mg.gemm(*ops[2], out=outs[2], **kw)
        with torch.cuda.stream(other):
            g.replay()
        with torch.cuda.stream(side):
            mg.gemm(*ops[2], out=outs[2], **kw)
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert np.array_equal(host(o), w)


def test_grouped_and_quantise_captured():
    """A captured grouped launch keeps its own plan while later calls on the
    stream upload theirs; a captured quantisation its own partial maxima."""
    log("capture grouped, quantise")
    lists = []
    for seed, shapes in ((1, [(70, 90, 110), (130, 33, 64), (5, 200, 77)]), (2, [(64 + i, 40, 50 + i) for i in range(300)])):
        ps = [operands(mg.MODE_BF16, *s, seed=seed) + (torch.empty(s[:2], device="cuda"),) for s in shapes]
        lists.append((ps, mg.ProblemBatch(ps, mg.MODE_BF16)))
    x, y = (dev(synth.draw(synth.rng(i), s)) for i, s in ((3, (300, 500)), (4, (700, 900))))
    want = [[host(mg.gemm(a, b, mode=mg.MODE_BF16, cfg=0, split_k=1)) for a, b, _ in ps] for ps, _ in lists]
    want_q = [host(t) for t in mg.quantize_e4m3(x)]
    lib = _lib.load()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    q, sc = torch.empty((300, 500), dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        mg.grouped(lists[0][1])
        _lib.check(lib.gemm_quantize_e4m3(x.data_ptr(), x.numel(), q.data_ptr(), sc.data_ptr(),
                                          ctypes.c_void_p(side.cuda_stream)))
    for _ in range(4):
        for ps, _ in lists:
            for _, _, c in ps:
                c.fill_(float("nan"))
        q.zero_()
        sc.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):    # as many uploads as the stream's staging ring holds, and one more
            for _ in range(5):
                mg.grouped(lists[1][1])
                mg.quantize_e4m3(y)
        with torch.cuda.stream(other):
            g.replay()
        with torch.cuda.stream(side):
            mg.grouped(lists[1][1])
        torch.cuda.synchronize()
        for (ps, _), w in zip(lists, want):
            for (_, _, c), v in zip(ps, w):
                assert np.array_equal(host(c), v)
        assert np.array_equal(host(q), want_q[0]) and np.array_equal(host(sc), want_q[1])


def test_a_destroyed_graph_gives_its_workspace_back():
    log("capture memory")
    mode, n = mg.MODE_BF16, 4095         # 64 MB of operand copies
    cfg = copies_config(mode)
    a, b = (torch.randn((n, n), device="cuda").to(torch.bfloat16) for _ in range(2))
    out = torch.empty((n, n), device="cuda")
    mg.gemm(a, b, out=out, mode=mode, cfg=cfg, split_k=1)
    want = host(out)
    free = []
    for i in range(10):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            mg.gemm(a, b, out=out, mode=mode, cfg=cfg, split_k=1)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        if i in (0, 9):
            assert np.array_equal(host(out), want)
        del g
        gc.collect()
        mg.gemm(a, b, out=out, mode=mode, cfg=cfg, split_k=1)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    # ten graphs held 640 MB: less than two of them may be missing at the end
    assert free[1] - free[9] < 128 << 20, free


def test_forked_streams_of_one_capture():
    """Products on two streams of one capture, unordered with one another, have a
    workspace each."""
    log("capture, forked")
    mode, sizes = mg.MODE_BF16, [(333, 463, 601), (401, 517, 777)]
    cfg = copies_config(mode)
    ops = [operands(mode, *s, seed=i) for i, s in enumerate(sizes)]
    want = [host(mg.gemm(a, b, mode=mode, cfg=cfg, split_k=3)) for a, b in ops]
    outs = [torch.empty(s[:2], device="cuda") for s in sizes]
    side, fork = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        fork.wait_stream(side)
        for _ in range(3):
            mg.gemm(*ops[0], out=outs[0], mode=mode, cfg=cfg, split_k=3)
            with torch.cuda.stream(fork):
                mg.gemm(*ops[1], out=outs[1], mode=mode, cfg=cfg, split_k=3)
        side.wait_stream(fork)
    for _ in range(4):
        for o in outs:
            o.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert np.array_equal(host(o), w)
