"""A solver context when device memory runs out after rks_create: rks_api.cpp
compiled for the host alone and run against a HIP runtime of host memory with
a budget (sanitize/context_check.cpp).  What was allocated at first use before
must still fit, by giving back what the context can do without."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2508_05400_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_memory_that_runs_out_in_the_middle(tmp_path):
    objs = []
    for src in (os.path.join(CSRC, "rks_api.cpp"), os.path.join(HERE, "sanitize", "context_check.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        r = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1",
                            "-fPIC", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}", "-c", src, "-o", objs[-1]],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    exe = str(tmp_path / "context_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", *objs, os.path.join(CSRC, "dense.cpp"),
                        os.path.join(CSRC, "panels.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert run.stdout.strip().endswith("ok: 0 failures")
