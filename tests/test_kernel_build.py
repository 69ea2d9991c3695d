"""CPU checks of the compiled kernels: the layout of their LDS."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_wide_lds_accesses_are_aligned():
    from paper_1602_05716_amd import build
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    r = subprocess.run([build.HIPCC] + flags + ["-fsyntax-only", "--cuda-device-only",
                                                os.path.join(ROOT, "tests", "helpers", "lds_layout.hip")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
