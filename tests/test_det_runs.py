"""Bit-reproducible form (CPU): the slices and batches of a row's run of sorted
pairs, compiled for the host from the header the kernel uses, up to the largest
call of 2^32 - 1 pairs."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not found")
def test_slices_and_batches_of_runs(tmp_path):
    exe = tmp_path / "det_runs_check"
    src = os.path.join(HERE, "native", "det_runs_check.hip")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", src, "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-2000:]
    assert " 0 wrong" in r.stdout
