"""Products whose tuned configuration cannot run on their operands (off 16-byte
alignment, or ragged with no room for packed copies): the any-shape
configuration that takes its place gives the bits of the same split-K factor,
through every entry point, on both sides of the rule that picks it; and it is
not far behind the best any-shape one."""
import ctypes

import numpy as np
import pytest

import synth
from paper_1306_6192_amd import _lib
from tests._gpu import dev, host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402

MODES = [mg.MODE_F32, mg.MODE_BF16, mg.MODE_F16, mg.MODE_F8E4M3, mg.MODE_SPLIT_BF16X3]
IDS = [_lib.MODE_NAMES[m] for m in MODES]


def operands(mode, m, n, k, off, seed):
    """Contiguous matrices that start `off` elements behind 16-byte alignment."""
    out = []
    for x in map(dev, synth.pair(m, n, k, seed=seed)):
        if mode in (mg.MODE_BF16, mg.MODE_F16):
            x = mg.convert(x, mode)
        elif mode == mg.MODE_F8E4M3:
            x = mg.quantize_e4m3(x)[0]
        buf = torch.empty(x.numel() + off, dtype=x.dtype, device="cuda")
        out.append(buf[off:].view(x.shape).copy_(x))
    return out


def expected(a, b, mode, m, n, k):
    return host(mg.gemm(a, b, mode=mode, cfg=0, split_k=mg.tuner_lookup(mode, m, n, k)[1])).view(np.uint32)


# tiles with waves along k: short k, long k on few tiles, long k on many; larger
# tiles; few and many 64x64 tiles per CU, with and without packed copies
MISALIGNED = [(20, 640, 256), (18, 320, 2560), (375, 320, 7552), (100, 4096, 1024), (128, 4096, 4096), (64, 16384, 256),
              (300, 300, 384), (3000, 1536, 256)]


@pytest.mark.parametrize("m,n,k", MISALIGNED)
@pytest.mark.parametrize("mode", MODES, ids=IDS)
def test_misaligned_operands(mode, m, n, k):
    log(f"any shape, misaligned {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    a, b = operands(mode, m, n, k, 1, seed=m + k)
    want = expected(a, b, mode, m, n, k)
    assert np.array_equal(host(mg.gemm(a, b, mode=mode)).view(np.uint32), want)
    out = torch.full((m, n), float("nan"), device="cuda")
    p = mg.make_problem(a, b, out, mode)
    ws = ctypes.c_uint64()
    _lib.check(_lib.load().gemm_plain_workspace_bytes(ctypes.byref(p), ctypes.byref(ws)))
    if mode != mg.MODE_SPLIT_BF16X3 or ws.value <= _lib.NOALLOC_SCRATCH_BYTES:
        _lib.check(_lib.load().gemm_plain_noalloc(ctypes.byref(p), torch.cuda.current_stream().cuda_stream))
        assert np.array_equal(host(out).view(np.uint32), want)


# few and many 64x64 tiles per CU; a choice with waves along k
RAGGED = [(201, 203, 1027), (261, 1025, 4099), (1501, 1503, 517), (3001, 1779, 449), (2047, 2049, 1023)]


@pytest.mark.parametrize("mode", MODES, ids=IDS)
def test_the_server_without_packed_copies(mode):
    """The plain-launch executor makes no packed copies."""
    server = mg.Server(executor=2)
    cases = []
    for m, n, k in RAGGED:
        log(f"any shape, served {_lib.MODE_NAMES[mode]} {(m, n, k)}")
        a, b = operands(mode, m, n, k, 0, seed=m)
        out = torch.full((m, n), float("nan"), device="cuda")
        cases.append((a, b, out, expected(a, b, mode, m, n, k)))
        torch.cuda.synchronize()
        _lib.check(server.submit(mg.make_problem(a, b, out, mode))[0])
    server.drain()
    for a, b, out, want in cases:
        assert np.array_equal(host(out).view(np.uint32), want)


@pytest.mark.parametrize("mode,m,n,k", [(mg.MODE_F8E4M3, 700, 8191, 8191), (mg.MODE_BF16, 8191, 600, 8001)])
def test_not_far_behind_the_best_any_shape_configuration(mode, m, n, k):
    """Packed copies above what the allocation-free entry point holds: the tile
    of the tuned configuration's own size was 2.5 to 3 times behind here."""
    log(f"any shape, timed {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    a, b = operands(mode, m, n, k, 0, seed=1)
    out = torch.empty((m, n), device="cuda")
    p = mg.make_problem(a, b, out, mode)
    split = mg.tuner_lookup(mode, m, n, k)[1]
    stream = torch.cuda.current_stream().cuda_stream

    def timed(run):
        run()
        best = float("inf")
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(4):
                run()
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    t = timed(lambda: _lib.check(_lib.load().gemm_plain_noalloc(ctypes.byref(p), stream)))
    best = min(timed(lambda: mg.gemm(a, b, out=out, mode=mode, cfg=c, split_k=split))
               for c in range(7) if not mg.config_chunk(mode, c))
    assert t < 1.75 * best, (t, best)
