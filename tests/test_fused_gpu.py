"""Tiles with waves along k, and aligned operand copies, against the
register-staged tiles.

Every configuration of a mode sums an element in the same order for a given
split-K factor, so these are bitwise comparisons with configuration 0 (itself
held to the oracle's bound by the other GPU tests), which need no tolerance.
Operands lie in NaN-filled buffers, so a load past a row's or a matrix's end
that reaches a result shows; C lies in a NaN-filled buffer, so a store outside
shows."""
import numpy as np
import pytest

import synth
from paper_1306_6192_amd import _lib
from tests._gpu import dev, host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402

MODES = [mg.MODE_F32, mg.MODE_BF16, mg.MODE_F16, mg.MODE_F8E4M3, mg.MODE_SPLIT_BF16X3]
NAN_CODE = {mg.MODE_F8E4M3: 0x7F}


def operands(mode, m, n, k, seed):
    A, B = synth.pair(m, n, k, seed=seed)
    a, b = dev(A), dev(B)
    if mode in (mg.MODE_BF16, mg.MODE_F16):
        a, b = mg.convert(a, mode), mg.convert(b, mode)
    elif mode == mg.MODE_F8E4M3:
        a, b = mg.quantize_e4m3(a)[0], mg.quantize_e4m3(b)[0]
    return a, b


def in_nan(x, mode, lead, tail):
    """x inside a buffer of NaNs, `lead` elements from each row's start and
    `tail` after its end."""
    r, c = x.shape
    fill = NAN_CODE.get(mode, float("nan"))
    buf = torch.full((r, lead + c + tail), fill, dtype=x.dtype, device="cuda")
    view = buf[:, lead:lead + c]
    view.copy_(x)
    return view


def product(a, b, mode, m, n, **kw):
    big = torch.full((m + 2, n + 3), float("nan"), device="cuda")
    mg.gemm(a, b, out=big[1:m + 1, 1:n + 1], mode=mode, **kw)
    h = host(big)
    mask = np.ones(h.shape, dtype=bool)
    mask[1:m + 1, 1:n + 1] = False
    assert np.isnan(h[mask]).all(), "a store outside C"
    return h[1:m + 1, 1:n + 1].view(np.uint32)


# one element; a row and a column more or fewer than a tile of 32 or 64; k of
# one grain, one more than a k-tile, and enough for more ranges than waves;
# n below one tile of columns; whole and broken 16-byte chunks
SHAPES = [(1, 1, 1), (31, 65, 33), (33, 63, 127), (64, 64, 512), (5, 16, 1153), (40, 48, 2176), (97, 192, 640),
          (2, 130, 1100)]


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("mode", MODES, ids=[_lib.MODE_NAMES[m] for m in MODES])
def test_every_config_equals_the_first_on_nan_padded_operands(mode, m, n, k):
    """Splits of one range, fewer than the waves, as many, and more (slabs);
    contiguous operands, and odd strides on bases off 16-byte alignment."""
    log(f"fused {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    a, b = operands(mode, m, n, k, seed=m + 3 * n + 5 * k)
    ragged_a, ragged_b = in_nan(a, mode, 1, 2), in_nan(b, mode, 3, 2)
    whole_a, whole_b = in_nan(a, mode, 16, 32 - k % 16), in_nan(b, mode, 16, 32 - n % 16)
    for split in (1, 3, 8, 9):
        want = product(a, b, mode, m, n, cfg=0, split_k=split)
        for cfg in range(mg.num_configs(mode)):
            for x, y in ((a, b), (whole_a, whole_b), (ragged_a, ragged_b)):
                got = product(x, y, mode, m, n, cfg=cfg, split_k=split)
                assert np.array_equal(got, want), (cfg, split, x.stride(), y.stride())


# near the smallest sizes that are copied (157, FP32 1774; k 444), ragged in k,
# in n, in both; whole chunks on a misaligned base
PACKED = [(157, 445, 447), (500, 157, 444), (512, 513, 515), (600, 520, 513), (515, 1000, 520), (520, 528, 528)]


@pytest.mark.parametrize("m,n,k", PACKED)
@pytest.mark.parametrize("mode", MODES, ids=[_lib.MODE_NAMES[m] for m in MODES])
def test_copied_operands_give_the_same_bits(mode, m, n, k):
    """Configurations of whole chunks on ragged products: A, B or both are
    copied to aligned rows.  Also without an explicit configuration, and
    through the allocation-free entry point."""
    if mode == mg.MODE_F32:
        m, n, k = m + 1617, n + 1617, k
    log(f"packed {_lib.MODE_NAMES[mode]} {(m, n, k)}")
    a, b = operands(mode, m, n, k, seed=m + n + k)
    views = ((a, b), (in_nan(a, mode, 1, 2), b), (a, in_nan(b, mode, 3, 2)), (in_nan(a, mode, 5, 1), in_nan(b, mode, 1, 1)))
    want = product(a, b, mode, m, n, cfg=0, split_k=2)
    for cfg in range(mg.num_configs(mode)):
        if mg.config_chunk(mode, cfg) or mode == mg.MODE_SPLIT_BF16X3:
            for x, y in views:
                assert np.array_equal(product(x, y, mode, m, n, cfg=cfg, split_k=2), want), (cfg, x.stride(), y.stride())
    chosen = product(a, b, mode, m, n)
    for x, y in views:
        assert np.array_equal(product(x, y, mode, m, n), chosen), (x.stride(), y.stride())
    import ctypes
    out = torch.full((m, n), float("nan"), device="cuda")
    p = mg.make_problem(views[3][0], views[3][1], out, mode)
    _lib.check(_lib.load().gemm_plain_noalloc(ctypes.byref(p), torch.cuda.current_stream().cuda_stream))
    assert np.array_equal(host(out).view(np.uint32), chosen)


def test_capture_of_a_product_that_needs_a_workspace():
    """A ragged product (operand copies) and a split one captured on a stream
    that has no workspace yet: the graph's replays equal the eager results,
    also after eager work on other data in between."""
    log("capture with copies and slabs")
    cases = []
    for mode, m, n, k in ((mg.MODE_BF16, 600, 1029, 1031), (mg.MODE_F32, 100, 3000, 5000)):
        a, b = operands(mode, m, n, k, seed=m)
        cases.append((mode, a, b, torch.empty((m, n), device="cuda"), host(mg.gemm(a, b, mode=mode))))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        for mode, a, b, out, _ in cases:
            mg.gemm(a, b, out=out, mode=mode)
    for _ in range(3):
        for _, _, _, out, _ in cases:
            out.fill_(float("nan"))
        mg.gemm(torch.rand((700, 1031), device="cuda"), torch.rand((1031, 900), device="cuda"))
        g.replay()
        for _, _, _, out, want in cases:
            assert np.array_equal(host(out), want)
