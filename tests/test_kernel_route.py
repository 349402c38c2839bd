"""Choice of the sampled-gradient kernels (CPU): the library's rule on order,
key form and model size, compiled for the host from the header that the launch
uses."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not found")
def test_kernels_by_order_and_model_size(tmp_path):
    exe = tmp_path / "kernel_route_check"
    src = os.path.join(HERE, "native", "kernel_route_check.hip")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-I", os.path.join(ROOT, "include"), src,
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-2000:]
    assert " 0 wrong" in r.stdout
