"""CPU checks of the kernel sources, compiled and not run: the layout of their
LDS and the width of their counters."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _compiles(name):
    from paper_1602_05716_amd import build
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    return subprocess.run([build.HIPCC] + flags + ["-fsyntax-only", "--cuda-device-only",
                                                   os.path.join(ROOT, "tests", "helpers", name)],
                          capture_output=True, text=True)


@pytest.mark.parametrize("name", ["lds_layout.hip", "rdf_counters.hip"])
def test_static_checks(name):
    r = _compiles(name)
    assert r.returncode == 0, r.stderr
