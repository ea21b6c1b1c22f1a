"""CPU property test of the transforms' arithmetic (tests/host_mul_tw.cpp):
products by a root power in split Montgomery form, butterflies and reductions
against exact 128-bit arithmetic, optimised and under sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = ["-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("flags", [["-O2"], SAN], ids=["optimised", "sanitizers"])
def test_split_montgomery_arithmetic(tmp_path, flags):
    exe = str(tmp_path / "host_mul_tw")
    subprocess.check_call(["g++"] + flags + ["-std=c++17", "-o", exe, os.path.join(ROOT, "tests", "host_mul_tw.cpp")])
    r = subprocess.run([exe, "100000"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-2000:]
