"""The helper that sets a kernel up once on every device (CPU only): a device
that has not had it gets it, and an error is not kept for later calls."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_once_per_device(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-pthread", "-fsanitize=thread",
                        "-I", os.path.join(ROOT, "paper_2209_10643_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "once_per_device_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_no_kernel_keeps_an_error():
    csrc = os.path.join(ROOT, "paper_2209_10643_amd", "csrc")
    for name in os.listdir(csrc):
        if name.endswith((".hip", ".h", ".cpp")):
            assert "static const hipError_t" not in open(os.path.join(csrc, name)).read(), name
