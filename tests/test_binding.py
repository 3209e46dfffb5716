"""The binding's two marshalling paths: the native module and ctypes."""

import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_library_alone_is_enough():
    """Without the native module the binding loads, with a warning, and every call takes the ctypes path."""
    code = """
import sys, warnings
sys.modules["paper_2309_04909_amd._fastcall"] = None
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2309_04909_amd import bicop as B
assert any("_fastcall" in str(w.message) for w in seen), seen
import torch
x, prm, sd = torch.zeros(4, dtype=torch.int64), B.Params(64, 7, 11), B.Seeds(1, 2, 3)
for call in (lambda: B.drelu(x, x, prm, sd), lambda: B.trunc_det(x, x, 64, 13), lambda: B.drelu_send(0, x, prm, sd),
             lambda: B.rss_relu((x, x, x), prm, B.RssSeeds(1, 2, 3, 4, 5))):
    try:
        call()
    except TypeError:
        continue
    raise AssertionError("host tensors were not refused")
print("loaded", B.version())
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "loaded bicop" in r.stdout, r.stderr[-2000:]
