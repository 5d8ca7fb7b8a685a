"""The tuning program's kinds of entries, without a GPU: which of the library's
measuring entry points each kind calls."""
import importlib.util
import os

import pytest

torch = pytest.importorskip("torch")
import paper_1306_6192_amd as mg  # noqa: E402

# (as a program is run: an import as the package's submodule would take the name
# of the package's function `tune`)
_spec = importlib.util.spec_from_file_location("tuning_program", os.path.join(os.path.dirname(mg.__file__), "tune.py"))
tune = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(tune)


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return 0
        return call


@pytest.mark.parametrize("kind,entry", [("plain-buckets", "gemm_tune_bucket"), ("grouped", "gemm_tune_grouped")])
def test_bucket_kinds(monkeypatch, tmp_path, kind, entry):
    lib = Recorder()
    monkeypatch.setattr(mg, "load", lambda: lib)
    monkeypatch.setattr(torch.cuda, "set_device", lambda d: None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("S", (), {"cuda_stream": 0}))
    monkeypatch.setattr(tune, "calibrate_mix", lambda *a: None)
    tune.main(["--what", kind, "--modes", "e4m3", "--out", str(tmp_path / "t.jsonl")])
    shapes = [args[1:4] for name, args in lib.calls if name == entry]
    assert shapes == tune.bucket_shapes(mg)[mg.MODE_F8E4M3]
    assert {name for name, _ in lib.calls} == {entry, "gemm_tuner_save"}
