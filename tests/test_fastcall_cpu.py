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


WITHOUT = """
import importlib.abc, sys
sys.path.insert(0, %r)
class Hide(importlib.abc.MetaPathFinder):
    def find_spec(self, name, path, target=None):
        if name.endswith("._fastcall"):
            raise ImportError(name)
sys.meta_path.insert(0, Hide())
import torch
import paper_1306_6192_amd as mg
from paper_1306_6192_amd import _lib
f = _lib.fastcall()
assert f.gemm(None, None, None, 0, 1.0, 1.0) is None and f.gemm_same(None, None, None) is None
assert f.convert(None, 1) is None and f.quantize(None) is None
for call in (lambda x: mg.gemm(x, x), lambda x: mg.gemm_f64(x.double(), x.double()), lambda x: mg.convert(x, mg.MODE_BF16),
             mg.quantize_e4m3):
    try:
        call(torch.zeros(2, 2))
    except ValueError as e:
        assert "device tensor" in str(e)
    else:
        raise AssertionError("a host tensor was accepted")
"""


def test_the_layer_works_without_the_native_path():
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", WITHOUT % root], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


def test_the_build_goes_on_without_a_host_compiler(monkeypatch, capsys):
    import importlib
    build = importlib.import_module("paper_1306_6192_amd.build")
    monkeypatch.setenv("CXX", "/nonexistent/compiler")
    build._build_fastcall(False)
    assert "not built" in capsys.readouterr().err
