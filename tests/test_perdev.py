"""Once-per-device initialisation (csrc/perdev.h), compiled for the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_once_per_device(tmp_path):
    exe = tmp_path / "perdev_host"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", os.path.join(HERE, "perdev_host.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "per device ok" in r.stdout, r.returncode


def test_no_process_wide_latch_on_function_attributes():
    """hipFuncSetAttribute is called from the per-device initialisers alone: no source keeps
    its status in a variable of the process."""
    import re
    csrc = os.path.join(os.path.dirname(HERE), "paper_2201_03509_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        s = open(os.path.join(csrc, f)).read() if f.endswith((".hip", ".h", ".cpp")) else ""
        assert not re.search(r"static\s+(const\s+)?hipError_t\s+\w+\s*=", s), f
