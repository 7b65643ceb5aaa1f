"""A deep network's gradient where the device does not hold one delta per layer
(tests/c/mlp_memory.cpp refuses the larger allocation): it goes layer by layer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.gpu
@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_gradient_falls_back_to_two_deltas(tmp_path):
    from paper_1810_08142_amd import _lib
    so = _lib.lib()._name
    exe = tmp_path / "mlp_memory"
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
           "-I/opt/rocm/include", os.path.join(ROOT, "tests", "c", "mlp_memory.cpp"), so, "-L/opt/rocm/lib",
           "-lamdhip64", "-ldl", f"-Wl,-rpath,{os.path.dirname(so)}", "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "mlp memory ok" in run.stdout
