"""Contractions on whole tiles ask for no split-k scratch (host logic, no GPU):
tests/c/gemm_scratch.cpp builds against the library's own contraction source."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_gemm_scratch(tmp_path):
    exe = tmp_path / "gemm_scratch"
    src = os.path.join(ROOT, "paper_1810_08142_amd", "csrc", "gemm.hip")
    # host code only: no kernel is launched, so what the other sources define stays unresolved
    cmd = ["hipcc", "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-w", f'-DSOURCE="{src}"',
           os.path.join(ROOT, "tests", "c", "gemm_scratch.cpp"), "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "gemm scratch ok" in run.stdout
