"""The native marshalling and the Python one below it, on the host: without
_native.so the binding works on libdart.so alone."""

import os
import subprocess
import sys
import warnings

import pytest

import paper_2509_23866_amd as dart

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def without_native(monkeypatch):
    monkeypatch.setattr(dart, "_native", None)
    monkeypatch.setitem(sys.modules, dart.__name__ + "._native", None)  # its import fails


def test_calls_without_the_native_library_are_marshalled_in_python(without_native):
    """The Python path is reached, and complains as it does; what is missing is said
    once."""
    z, y = torch.zeros(2, 8), torch.zeros(2, dtype=torch.int32)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        with pytest.raises(ValueError):  # the tensors are not on a GPU
            dart.dart_tok_stats(z, y)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        with pytest.raises(ValueError):
            dart.dart_tok_stats(z, y)


def test_a_build_without_the_native_library_is_refused(without_native):
    with pytest.raises(RuntimeError, match="_native.so"):
        dart._nat(required=True)


def test_the_native_library_is_built():
    """What build() leaves is loaded, not the stand-in."""
    assert dart._nat(required=True).__name__.endswith("_native")


def test_one_hip_runtime_whatever_is_loaded_first():
    """torch brings its own HIP runtime; libdart.so opened before it must not bring a
    second one, whose streams and memory torch's would not be."""
    code = ("import paper_2509_23866_amd as dart\n"
            "assert dart.dart_kept_steps(10, 0.5) == 5\n"
            "import torch\n"
            "maps = open('/proc/self/maps').read().split('\\n')\n"
            "print(len({m.split()[-1] for m in maps if 'libamdhip64' in m}))\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    assert out.stdout.split() == ["1"]
