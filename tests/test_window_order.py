"""The window copies' order and launch sizes (csrc/window.h), without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_35065_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ missing")
def test_every_window_once_and_no_idle_groups(tmp_path):
    exe = tmp_path / "window_check"
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-o", str(exe), os.path.join(ROOT, "tests", "native", "window_check.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "window check ok" in r.stdout
