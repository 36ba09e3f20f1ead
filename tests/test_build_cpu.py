"""What the compiler made of the kernels: the built library's own metadata, no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_05722_amd import _lib, buildlib

LLVM = "/opt/rocm/llvm/bin/"


def private_bytes(tmp_path):
    _lib.load()
    lib = shutil.copy(buildlib.LIB, tmp_path)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", os.path.basename(lib)], cwd=tmp_path, check=True,
                   capture_output=True)
    out = {}
    for name in os.listdir(tmp_path):
        if "gfx950" in name:
            text = subprocess.run([LLVM + "llvm-readelf", "--notes", name], cwd=tmp_path, check=True, capture_output=True,
                                  text=True).stdout
            for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", text):
                out[m.group(1)] = int(m.group(2))
    return out


def test_kernels_use_no_private_memory(tmp_path):
    """Private memory is traffic in the middle of a kernel."""
    if not os.path.exists(LLVM + "llvm-objdump"):
        pytest.skip("needs the ROCm LLVM tools")
    sizes = private_bytes(tmp_path)
    assert any("gemm_stream_kernel" in n for n in sizes) and any("attention_kernel" in n for n in sizes)
    bad = {n: b for n, b in sizes.items() if b}
    assert not bad, bad
