"""The partial sums of the ladder's contractions fit their buffers (host logic, no GPU):
tests/c/slab_splits.cpp builds against the library's own ladder source and walks the slabs
of the plain and of the exchange-symmetric form over v = 16..320 and o up to v/5."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source,flags", [("ppl.hip", []), ("ppl_bf16.hip", ["-DSPLIT_BF16"])])
def test_no_slab_needs_more_partial_sums_than_are_held(source, flags, tmp_path):
    exe = tmp_path / "slab_splits"
    src = os.path.join(ROOT, "paper_1810_08142_amd", "csrc", source)
    # host code only: no kernel is launched, so what the other sources define stays unresolved
    cmd = ["hipcc", "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-w", f'-DSOURCE="{src}"', *flags,
           os.path.join(ROOT, "tests", "c", "slab_splits.cpp"), "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "slab splits ok" in run.stdout
