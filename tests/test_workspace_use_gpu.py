"""The workspace that a product really uses: the plain-launch executor charges
that and no more, and the allocation-free entry point's array holds it (slabs,
pre-split copies, both)."""
import ctypes

import numpy as np
import pytest

import oracle
import synth
from paper_1306_6192_amd import _lib
from tests._gpu import dev, host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402


def operands(mode, m, n, k, seed):
    A, B = synth.pair(m, n, k, seed=seed)
    a, b = dev(A), dev(B)
    if mode == mg.MODE_BF16:
        a, b = mg.convert(a, mode), mg.convert(b, mode)
    elif mode == mg.MODE_F8E4M3:
        a, b = mg.quantize_e4m3(a)[0], mg.quantize_e4m3(b)[0]
    return A, B, a, b


def waves_along_k(mode, cfg):
    """k ranges that a workgroup of the configuration adds up (0: none)."""
    i = mg.config_info(mode, cfg)
    return i["waves"] if i["BM"] == 32 or (i["BM"] == 64 and i["BN"] == 64 and i["waves"] == 8) else 0


@pytest.mark.parametrize("mode,m,n,k", [(mg.MODE_F32, 512, 512, 512), (mg.MODE_BF16, 100, 3000, 5000),
                                        (mg.MODE_SPLIT_BF16X3, 512, 512, 512)])
def test_the_plain_executor_charges_no_unused_slabs(mode, m, n, k):
    """These split k within the workgroup: operands and output are all that a
    request holds."""
    log(f"workspace charged {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    cfg, split = mg.tuner_lookup(mode, m, n, k)
    assert 1 < split <= waves_along_k(mode, cfg)
    _, _, a, b = operands(mode, m, n, k, seed=k)
    c = torch.full((m, n), float("nan"), device="cuda")
    torch.cuda.synchronize()
    p = mg.make_problem(a, b, c, mode)
    base = ctypes.c_uint64()
    _lib.check(_lib.load().gemm_serve_footprint(ctypes.byref(p), ctypes.byref(base)))
    for budget, rc in ((base.value - 1, _lib.GEMM_ENOMEM), (base.value, _lib.GEMM_OK)):
        server = mg.Server(hbm_budget_bytes=budget, max_inflight=4, num_streams=1, max_batch=1, executor=2)
        assert server.submit(p)[0] == rc
        server.drain()
    assert np.array_equal(host(c), host(mg.gemm(a, b, mode=mode)))


PRESPLIT = range(6, 15)   # split-BF16x3 configurations on operand copies, whole k range per workgroup
# slabs; copies; copies and slabs; slabs of more ranges than a workgroup's waves
USES = [(mg.MODE_F8E4M3, 64, 4096, 8192), (mg.MODE_SPLIT_BF16X3, 1536, 1536, 1536),
        (mg.MODE_SPLIT_BF16X3, 2000, 1024, 2048), (mg.MODE_BF16, 300, 512, 8192)]


@pytest.mark.parametrize("mode,m,n,k", USES)
def test_the_array_holds_what_is_used(mode, m, n, k):
    log(f"workspace used {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    lib = _lib.load()
    cfg, split = mg.tuner_lookup(mode, m, n, k)
    presplit = mode == mg.MODE_SPLIT_BF16X3 and cfg in PRESPLIT
    assert presplit or split > max(1, waves_along_k(mode, cfg))
    need = (split * ((m * n + 3) // 4 * 16) if split > 1 else 0) + (4 * ((k + 15) // 16 * 16) * (m + n) if presplit else 0)
    A, B, a, b = operands(mode, m, n, k, seed=3)
    out = torch.full((m, n), float("nan"), device="cuda")
    p = mg.make_problem(a, b, out, mode)
    ws = ctypes.c_uint64()
    _lib.check(lib.gemm_plain_workspace_bytes(ctypes.byref(p), ctypes.byref(ws)))
    assert need <= ws.value <= _lib.NOALLOC_SCRATCH_BYTES
    want = host(mg.gemm(a, b, mode=mode))
    for _ in range(2):
        out.fill_(float("nan"))
        _lib.check(lib.gemm_plain_noalloc(ctypes.byref(p), torch.cuda.current_stream().cuda_stream))
        assert np.array_equal(host(out), want)
    if mode == mg.MODE_SPLIT_BF16X3:
        assert oracle.relerr(want, oracle.gemm(A, B)) <= 1e-5


def test_growing_products_replace_the_workspace_seldom():
    """Twenty ever larger ragged products (copies of 4 to 34 MB) on a stream
    that has no workspace yet: the buffer is replaced at every doubling, not at
    every product."""
    log("workspace growth")
    hip = ctypes.CDLL("libamdhip64.so")
    handle = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0
    stream = torch.cuda.ExternalStream(handle.value)
    mode = mg.MODE_BF16
    cfg = next(c for c in range(mg.num_configs(mode)) if mg.config_chunk(mode, c))
    sizes = range(1001, 3001, 100)
    x = torch.randn((3001, 3001), device="cuda").to(torch.bfloat16)
    out = torch.empty((3001, 3001), device="cuda")
    ops = [(x.view(-1)[:n * n].view(n, n), out.view(-1)[:n * n].view(n, n)) for n in sizes]
    torch.cuda.synchronize()
    free = [torch.cuda.mem_get_info()[0]]
    for a, c in ops:
        mg.gemm(a, a, out=c, mode=mode, cfg=cfg, split_k=1, stream=stream)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    replaced = sum(a != b for a, b in zip(free, free[1:]))
    assert replaced <= 6, free
    a, c = ops[-1]
    want = host(mg.gemm(a, a, mode=mode, cfg=cfg, split_k=1))
    assert np.array_equal(host(c), want)
