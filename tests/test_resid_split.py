"""The split of a matrix's rows among the slots of the row-layout residual
kernel, on the host under UBSan: runs of empty rows, no nonzeros, more slots
than rows; and its batches of nonzeros up to entry 2^31 - 2."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2508_05400_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rows_are_shared_by_rows_and_nonzeros(tmp_path):
    exe = str(tmp_path / "resid_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", f"-I{CSRC}",
           os.path.join(HERE, "sanitize", "resid_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert run.stdout.strip().endswith("ok: 0 failures")
