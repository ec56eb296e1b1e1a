"""CPU accuracy test of the double-precision elementary functions of the path
kernels: csrc/fp64_math.hpp compiled by the host compiler, each function in ulps
against long double over its callers' arguments; no GPU, no device code."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_elementary_functions():
    src = os.path.join(ROOT, "tests", "host", "fp64_math_test.cpp")
    inc = [os.path.join(ROOT, "tests", "host", "fake_hip"),
           os.path.join(ROOT, "paper_2309_10477_amd", "csrc")]
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "fp64_math_test")
        subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall",
                               *(a for i in inc for a in ("-I", i)), src, "-o", exe])
        out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip() == "ok"
