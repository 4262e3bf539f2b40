"""The race check of the library's own choices: tests/jitter_check_auto.py
against the jitter build in a process of its own."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu


def test_jitter_build_keeps_the_bits_of_the_automatic_choices():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = os.path.join(ROOT, "paper_0803_0048_amd", "libtpilu_jitter.so")
    assert os.path.exists(lib), "libtpilu_jitter.so is not built"
    print("[gpu] jitter check of the automatic choices in a child process", flush=True)
    r = subprocess.run([sys.executable, "-u", "-m", "tests.jitter_check_auto"], cwd=ROOT,
                       env=dict(os.environ, TPILU_LIBRARY="jitter"), capture_output=True, text=True, timeout=100)
    print(r.stdout[-4000:], flush=True)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "jitter build: all cases bitwise" in r.stdout
