"""Registers of the built kernels (CPU): spilled vector registers from the
metadata of the library's own code objects, for the kernels where spills have
crept in before."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2605_20353_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        count, p = int.from_bytes(data[p:p + 8], "little"), p + 8
        for _ in range(count):
            off, size, n = (int.from_bytes(data[p + 8 * i:p + 8 * i + 8], "little") for i in range(3))
            p += 24
            if build.ARCH.encode() in data[p:p + n]:
                yield data[at + off:at + off + size]
            p += n
        at = data.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def spills():
    """Kernel (mangled name) -> spilled vector registers."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    if not os.path.exists(build.LIB):
        build.build()
    out = {}
    for obj in code_objects(build.LIB):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("  - .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            out[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    assert len(out) > 100
    return out


# k_loss_grad<T, order, lanes, vec, scatter, wide, given>, k_bucket_accum<T, order, lanes, vec, wide>
LOSS_GRAD = "k_loss_gradI{t}Li{order}ELi{lanes}ELi{vec}ELb{scatter}ELb{wide}ELb0EE"

# double kernels that scatter in their loop, at one and two columns per lane:
# less than any shape spilled when row addresses were formed with the products
# (3, 15, 12 and 28)
DOUBLE_LIMITS = {(3, 1): 2, (3, 2): 14, (4, 1): 11, (4, 2): 27}


@pytest.mark.parametrize("order,vec", list(DOUBLE_LIMITS))
def test_double_scattering_kernels(spills, order, vec):
    for lanes in (4, 8, 16, 32, 64):
        if (lanes, vec) == (4, 1):
            continue
        key = LOSS_GRAD.format(t="d", order=order, lanes=lanes, vec=vec, scatter=1, wide=0)
        found = [n for name, n in spills.items() if key in name]
        assert len(found) == 1 and found[0] <= DOUBLE_LIMITS[order, vec], (key, found)


@pytest.mark.parametrize("order", [3, 4, 5])
def test_float_kernels_that_scatter_nothing(spills, order):
    # bounded to a number of wavefronts per SIMD that their registers fit
    for key in ("k_loss_gradIfLi%dELi\\d+ELi\\dELb0ELb0ELb0EE" % order, "k_bucket_accumIfLi%dELi\\d+ELi\\dELb0EE" % order):
        found = {name: n for name, n in spills.items() if re.search(key, name)}
        assert len(found) == 15 and max(found.values()) <= 2, found
