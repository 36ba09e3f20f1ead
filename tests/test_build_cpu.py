"""What the compiler made of the kernels: the built library's own metadata, no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_05722_amd import _lib, buildlib

LLVM = "/opt/rocm/llvm/bin/"

# Private memory is traffic in the middle of a kernel.  The LM head of up to 16 rows keeps its operand slice in
# registers; where the hidden size makes that slice 8 or 20 k-steps a wavefront, part of it does not fit.
SPILLS = {"gemm_norm_kernelILi8E", "gemm_norm_kernelILi20E"}


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
    if not os.path.exists(LLVM + "llvm-objdump"):
        pytest.skip("needs the ROCm LLVM tools")
    sizes = private_bytes(tmp_path)
    assert any("gemm_stream_kernel" in n for n in sizes) and any("attention_kernel" in n for n in sizes)
    bad = {n: b for n, b in sizes.items() if b and not any(s in n for s in SPILLS)}
    assert not bad, bad
