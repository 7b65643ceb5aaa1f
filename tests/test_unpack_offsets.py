"""The unpack's element offsets (host logic, no GPU): tests/c/unpack_offsets.cpp builds
against the library's own header and compares them with 64-bit ones up to o = 4096."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_unpack_offsets(tmp_path):
    exe = tmp_path / "unpack_offsets"
    cmd = ["hipcc", "-std=c++17", "-Wall", os.path.join(ROOT, "tests", "c", "unpack_offsets.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "unpack offsets ok" in run.stdout
