"""CPU test of the context's host code (budgets, error returns), compiled with
the host compiler against a stand-in for the HIP runtime; no GPU, no device code."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("sanitize", [False, True], ids=["plain", "asan-ubsan"])
def test_context(sanitize):
    src = os.path.join(ROOT, "tests", "host", "context_test.cpp")
    inc = [os.path.join(ROOT, "tests", "host", "fake_hip"),
           os.path.join(ROOT, "paper_2309_10477_amd", "csrc")]
    flags = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all"] if sanitize else []
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "context_test")
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", *flags,
                               *(a for i in inc for a in ("-I", i)), src, "-o", exe])
        out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip() == "ok"
