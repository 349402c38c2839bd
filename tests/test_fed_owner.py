"""Threads of the batched federated owner workgroups (CPU): the library's rule,
compiled for the host from the header that the launch uses."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not found")
def test_threads_by_the_fullest_row_block(tmp_path):
    exe = tmp_path / "fed_owner_check"
    src = os.path.join(HERE, "native", "fed_owner_check.hip")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", src, "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-2000:]
    assert " 0 wrong" in r.stdout
