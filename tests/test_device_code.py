"""What the built library's kernels ask of the chip, read from the code objects built here."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_13485_amd import build as hip_build

LLVM = "/opt/rocm/llvm/bin"


def kernel_metadata(tmp_path):
    """name -> bytes of scratch memory per work item, of every kernel in libpropd.so"""
    if not os.path.exists(hip_build.LIB_PATH):
        hip_build.build()
    lib = shutil.copy(hip_build.LIB_PATH, tmp_path)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], check=True, cwd=tmp_path, capture_output=True)
    found = {}
    for name in os.listdir(tmp_path):
        if "gfx950" not in name:
            continue
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", name], check=True, cwd=tmp_path,
                               capture_output=True, text=True).stdout
        for block in notes.split("- .agpr_count")[1:]:
            kernel = re.search(r"\.name:\s+(\S+)", block[block.index(".language") if ".language" in block else 0:])
            found[kernel.group(1)] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1))
    return found


def test_no_kernel_uses_scratch_memory(tmp_path):
    """The attention and scoring kernels have loads and LDS reads in flight that the compiler
    does not track (they are waited for by hand).  A register spilled to scratch memory while such
    a load is on its way is saved before the value is there, and the load then lands in a
    register that holds something else by that time: a build that spills must not run."""
    if not os.path.exists(f"{LLVM}/llvm-objdump"):
        pytest.skip("no LLVM tools")
    scratch = kernel_metadata(tmp_path)
    assert any("tree_attn_bf16_kernel" in k for k in scratch) and any("early_head_bf16_kernel" in k for k in scratch)
    assert {k: v for k, v in scratch.items() if v} == {}
