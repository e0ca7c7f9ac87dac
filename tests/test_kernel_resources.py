"""Registers of the compiled kernels (CPU only: read from the code objects in
the built library): kernels that run by default hold their values in
registers, with no scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1811_11558_amd", "libfvim.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"

pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="library not built"),
              pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")]


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{mangled kernel name: scratch bytes per lane} of every gfx950 kernel."""
    data = open(LIB, "rb").read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", {}
    at = data.find(magic)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + ln]
            p += 24 + ln
            if b"gfx950" not in target or size == 0:
                continue
            f = tmp_path_factory.mktemp("co") / "code.o"
            f.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                name = re.search(r"\.name:\s+(\S+)", part).group(1)
                out[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", part).group(1))
        at = data.find(magic, at + 1)
    return out


# the depth pass in the layout of 33 to 64 float64 nodes, every variant
# the row and column kernels of the contact iterations, up to 4096 points a side;
# the float64 row transforms, up to that length
KERNELS = [r"k_depth(_batch)?IdLi64ELi1E", r"k_x_(r2c|c2r)Id",
           r"k_(rows_fwd|rows_inv|columns|pk_\w+|f_rows_fwd|f_rows_inv|f_grad|f_momentum)ILi"]


@pytest.mark.parametrize("pattern", KERNELS)
def test_kernels_use_no_scratch(scratch, pattern):
    names = [k for k in scratch if re.search(pattern, k)]
    assert names
    assert {k: scratch[k] for k in names if scratch[k]} == {}
