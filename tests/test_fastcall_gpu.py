"""The native call path of the Python layer against the layer's own path (taken
here by naming the current stream): the same results for everything the
native path accepts, and the layer's own behaviour for everything it leaves
alone."""
import numpy as np
import pytest

from paper_1306_6192_amd import _lib
from tests._gpu import host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402

# every element type a mode takes
TYPES = [(mg.MODE_F32, torch.float32), (mg.MODE_SPLIT_BF16X3, torch.float32), (mg.MODE_BF16, torch.bfloat16),
         (mg.MODE_BF16, torch.int16), (mg.MODE_BF16, torch.uint16), (mg.MODE_F16, torch.float16),
         (mg.MODE_F16, torch.int16), (mg.MODE_F16, torch.uint16), (mg.MODE_F8E4M3, torch.float8_e4m3fn),
         (mg.MODE_F8E4M3, torch.uint8), (mg.MODE_F8E4M3, torch.int8)]


def bits(t):
    return host(t.view(torch.int16) if t.dtype == torch.bfloat16 else t).view(np.uint8)


def values(mode, m, n):
    x = torch.rand((m, n), device="cuda") - 0.5
    if mode in (mg.MODE_BF16, mg.MODE_F16):
        return mg.convert(x, mode)
    return x.to(torch.float8_e4m3fn) if mode == mg.MODE_F8E4M3 else x


@pytest.mark.parametrize("mode,dtype", TYPES, ids=[f"{_lib.MODE_NAMES[m]}-{str(d)[6:]}" for m, d in TYPES])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (5, 7, 3), (1, 9, 4), (6, 1, 5), (64, 48, 80), (0, 3, 4), (3, 0, 4)])
def test_gemm_equals_the_general_path(mode, dtype, m, n, k):
    """Contiguous, row-strided, one-row and one-column operands, gradients
    required or not, an output given or not."""
    log(f"fastcall {mode} {dtype} {(m, n, k)}")
    fast = _lib.fastcall().gemm
    s = torch.cuda.current_stream()
    a, b = (values(mode, r, c + 3).view(dtype) for r, c in ((m, k), (k, n)))
    kw = dict(mode=mode, scale_a=1.5, scale_b=0.25)
    for x, y in ((a[:, :k].contiguous(), b[:, :n].contiguous()), (a[:, 1:k + 1], b[:, 2:n + 2]), (a[:, :k], b[:, :n].contiguous())):
        want = mg.gemm(x, y, stream=s, **kw)
        got = fast(x, y, None, mode, 1.5, 0.25)
        assert got is not None and got.dtype == torch.float32 and got.shape == (m, n) and not got.requires_grad
        assert np.array_equal(bits(got), bits(want))
        out = torch.full((m, n + 2), float("nan"), device="cuda")
        view = out[:, 1:n + 1]
        assert mg.gemm(x, y, out=view, **kw) is view
        assert np.array_equal(bits(view.contiguous()), bits(want))
        assert torch.isnan(out[:, [0, -1]]).all()
    if dtype == torch.float32 and m and n:
        x, y = a[:, :k].contiguous().requires_grad_(), b[:, :n].contiguous()
        got = mg.gemm(x, y, mode=mode)
        assert not got.requires_grad and np.array_equal(bits(got), bits(mg.gemm(x.detach(), y, mode=mode, stream=s)))


def test_other_entry_points_equal_the_general_path():
    log("fastcall f64, c32, convert, quantize")
    s = torch.cuda.current_stream()
    f = _lib.fastcall()
    for dtype, run in ((torch.float64, mg.gemm_f64), (torch.complex64, mg.gemm_c32)):
        for m, n, k in ((1, 1, 1), (33, 20, 50), (0, 2, 2), (4, 5, 0)):
            a, b = torch.randn((m, k), dtype=dtype, device="cuda"), torch.randn((k, n), dtype=dtype, device="cuda")
            got = f.gemm_same(a, b, None)
            assert got is not None and np.array_equal(bits(got), bits(run(a, b, stream=s)))
            out = torch.empty((m, n), dtype=dtype, device="cuda")
            assert run(a, b, out=out) is out and np.array_equal(bits(out), bits(got))
    for shape in ((7,), (3, 5), (2, 3, 4), (0, 4), ()):
        x = torch.randn(shape, device="cuda")
        for mode, dtype in ((mg.MODE_BF16, torch.bfloat16), (mg.MODE_F16, torch.float16)):
            got = f.convert(x, mode)
            assert got is not None and got.dtype == dtype and got.shape == x.shape
            assert np.array_equal(bits(got.reshape(-1)), bits(mg.convert(x, mode, stream=s).reshape(-1)))
        q, sc = f.quantize(x)
        q2, sc2 = mg.quantize_e4m3(x, stream=s)
        assert q.shape == x.shape and q.dtype == torch.uint8 and sc.shape == (1,)
        assert np.array_equal(bits(q.reshape(-1)), bits(q2.reshape(-1))) and np.array_equal(bits(sc), bits(sc2))


def test_what_is_not_plain_goes_to_the_general_path():
    """Left alone: subclasses, other layouts, types, shapes and devices, lazily
    conjugated or negated operands, functorch wrappers, active modes; the
    layer then raises, or runs, as it always did."""
    log("fastcall refusals")
    f = _lib.fastcall()
    a, b = torch.rand((4, 6), device="cuda"), torch.rand((6, 5), device="cuda")

    class Sub(torch.Tensor):
        pass

    sub = a.as_subclass(Sub)
    c = torch.zeros((4, 6), dtype=torch.complex64, device="cuda")
    for x, y, out in ((sub, b, None), (a.t(), b, None), (a, b.cpu(), None), (a.cpu(), b, None), (a, b[0], None), (a, b[:5], None),
                      (a.double(), b, None), (a, b, a), (a, b, torch.empty((4, 5), dtype=torch.float16, device="cuda")),
                      (a, b, torch.empty((5, 4), device="cuda").t()), (a.to_sparse(), b, None), (None, b, None), (a, 3.0, None)):
        assert f.gemm(x, y, out, mg.MODE_F32, 1.0, 1.0) is None
    assert f.gemm(a, b, None, 9, 1.0, 1.0) is None and f.gemm(a, b, None, mg.MODE_F32, 1, 1.0) is None
    assert f.gemm_same(c.conj(), c.t().contiguous(), None) is None and f.gemm_same(a, b, None) is None
    assert f.convert(a.t(), mg.MODE_BF16) is None and f.convert(a, mg.MODE_F32) is None and f.quantize(a.half()) is None
    with pytest.raises(ValueError, match="inner dimensions"):
        mg.gemm(a, b[:5])
    with pytest.raises(ValueError, match="device tensor"):
        mg.gemm(a.cpu(), b)
    with pytest.raises(ValueError, match="row-major"):
        mg.gemm(torch.rand((6, 4), device="cuda").t(), b)
    with pytest.raises(TypeError):
        mg.gemm(a.double(), b)
    with pytest.raises(ValueError):
        mg.convert(a.t(), mg.MODE_BF16)
    with pytest.raises(mg.GemmError) as e:      # C overlaps A: refused by the library, raised by the layer
        square = torch.rand((8, 8), device="cuda")
        mg.gemm(square, square.clone(), out=square)
    assert e.value.code == _lib.GEMM_EINVAL and "overlap" in str(e.value)
    assert np.array_equal(bits(mg.gemm(sub, b)), bits(mg.gemm(a, b)))

    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Fn(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    for mode in (Fn, Dispatch):
        with mode():
            assert f.gemm(a, b, None, mg.MODE_F32, 1.0, 1.0) is None
            assert mg.gemm(a, b).shape == (4, 5)
    seen = []

    def inner(x):
        seen.append(f.gemm(x, b, None, mg.MODE_F32, 1.0, 1.0))
        return x.sum()

    torch.func.vmap(inner)(torch.rand((2, 4, 6), device="cuda"))
    torch.func.grad(inner)(a)
    assert seen == [None, None]


def test_calls_run_on_the_current_stream():
    log("fastcall stream")
    a, b = torch.rand((300, 400), device="cuda"), torch.rand((400, 200), device="cuda")
    want = bits(mg.gemm(a, b))
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    out = torch.zeros((300, 200), device="cuda")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert np.array_equal(bits(mg.gemm(a, b)), want)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):        # captured only if it goes to the capturing stream
        mg.gemm(a, b, out=out)
    assert not out.any()
    g.replay()
    assert np.array_equal(bits(out), want)


@pytest.mark.parametrize("mode", [1 << 32, (1 << 32) + mg.MODE_BF16, 1 << 70, -1])
def test_a_mode_outside_32_bits_is_refused(mode):
    """By the layer itself, as a mode it does not know."""
    log(f"fastcall mode {mode}")
    a = torch.rand((4, 4), device="cuda")
    for x in (a, a.to(torch.bfloat16)):
        with pytest.raises(KeyError):
            mg.gemm(x, x.clone(), mode=mode)
    with pytest.raises(KeyError):
        mg.convert(a, mode)
