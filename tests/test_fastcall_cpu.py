"""The native call path's refusals that need no GPU: whatever it does not take
it hands back as None, with no error left behind."""
import pytest

pytest.importorskip("torch")
from paper_1306_6192_amd import _lib


@pytest.mark.parametrize("mode", [-1, -(1 << 70), _lib.NUM_MODES, 1 << 32,
                                  (1 << 32) + 1, 1 << 63, 1 << 70, 1.0, None])
def test_modes_that_are_none(mode):
    f = _lib.fastcall()
    assert f.gemm(None, None, None, mode, 1.0, 1.0) is None
    assert f.convert(None, mode) is None
