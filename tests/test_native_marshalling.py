"""The binding's libraries on the host: what they bring into the process."""

import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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
