"""What the built library's kernels ask of the chip, read from the code objects built here."""
import os
import re
import shutil
import subprocess
import sys

import pytest

from paper_2402_13485_amd import build as hip_build

LLVM = "/opt/rocm/llvm/bin"


def kernel_metadata(tmp_path):
    """name -> bytes of scratch memory per work item, of every kernel in libpropd.so as its sources are now"""
    if hip_build.stale():
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


SPILLING = """
#include <hip/hip_runtime.h>
// %d floats alive across the barrier, of 128 registers
extern "C" __global__ __launch_bounds__(1024) void tree_attn_bf16_kernel(float *p) {
  float v[%d];
#pragma unroll
  for (int i = 0; i < %d; ++i) v[i] = p[1024 * i + threadIdx.x];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < %d; ++i) p[1024 * i + (threadIdx.x ^ 1)] = v[i];
}
extern "C" __global__ void early_head_bf16_kernel(float *p) { p[threadIdx.x] = 0.f; }
"""


@pytest.mark.parametrize("live,spills", [(16, False), (200, True)])
def test_build_refuses_a_kernel_that_spills(tmp_path, monkeypatch, live, spills):
    """build() leaves the library alone when a kernel with hand-placed waits spills, with or without
    LLVM's tools at hand.  (The kernel here is compiled, never run.)"""
    (tmp_path / "one.hip").write_text(SPILLING % ((live,) * 4))
    lib = tmp_path / "lib.so"
    lib.write_text("the one before")
    monkeypatch.setattr(hip_build, "CSRC", str(tmp_path))
    monkeypatch.setattr(hip_build, "SOURCES", ["one.hip"])
    monkeypatch.setattr(hip_build, "LIB_PATH", str(lib))
    if spills:
        with pytest.raises(RuntimeError, match="tree_attn_bf16_kernel"):
            hip_build.build()
        assert lib.read_text() == "the one before" and sorted(os.listdir(tmp_path)) == ["lib.so", "one.hip"]
    else:
        hip_build.build()
        assert lib.read_bytes()[:4] == b"\x7fELF"


def test_library_older_than_a_source_is_stale(tmp_path, monkeypatch):
    for name in ("lib.so", "one.hip", "one.h"):
        (tmp_path / name).write_text("")
        os.utime(tmp_path / name, (1e9, 1e9))
    monkeypatch.setattr(hip_build, "CSRC", str(tmp_path))
    monkeypatch.setattr(hip_build, "LIB_PATH", str(tmp_path / "lib.so"))
    now = 2e9 if os.path.getmtime(hip_build.__file__) < 2e9 else 4e9
    os.utime(tmp_path / "lib.so", (now, now))
    assert not hip_build.stale()
    os.utime(tmp_path / "one.h", (now + 1, now + 1))
    assert hip_build.stale()
    os.remove(tmp_path / "lib.so")
    assert hip_build.stale()


@pytest.mark.parametrize("library,marshal", [(True, True), (True, False), (False, True)])
def test_library_and_marshalling_are_replaced_together(tmp_path, monkeypatch, capfd, library, marshal):
    """The library is built where the marshalling cannot be, which then goes: it was made for the library before.
    A library that is not replaced keeps the marshalling it came with."""
    (tmp_path / "one.hip").write_text(SPILLING % ((16 if library else 200,) * 4))
    (tmp_path / "marshal.cpp").write_text("int one() { return 1; }")
    for name in ("lib.so", "marshal.so"):
        (tmp_path / name).write_text("the one before")
    monkeypatch.setattr(hip_build, "CSRC", str(tmp_path))
    monkeypatch.setattr(hip_build, "SOURCES", ["one.hip"])
    monkeypatch.setattr(hip_build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(hip_build, "MARSHAL_PATH", str(tmp_path / "marshal.so"))
    if not marshal:
        monkeypatch.setattr(hip_build, "marshal_command", lambda out: ["/nowhere/g++", out])
    if library:
        hip_build.build()
    else:
        with pytest.raises(RuntimeError, match="tree_attn_bf16_kernel"):
            hip_build.build()
    left = {name: (tmp_path / name).read_bytes()[:4] for name in os.listdir(tmp_path) if ".so" in name}
    elf, before = b"\x7fELF", b"the "
    assert left == ({"lib.so": elf, "marshal.so": elf} if library and marshal else {"lib.so": elf} if library else
                    {"lib.so": before, "marshal.so": before})
    assert ("not built" in capfd.readouterr().err) == (not marshal)


def test_missing_or_old_marshalling_is_stale(tmp_path, monkeypatch):
    now = 2e9 if os.path.getmtime(hip_build.__file__) < 2e9 else 4e9
    for name, time in (("lib.so", now), ("marshal.so", now), ("marshal.cpp", 1e9)):
        (tmp_path / name).write_text("")
        os.utime(tmp_path / name, (time, time))
    monkeypatch.setattr(hip_build, "CSRC", str(tmp_path))
    monkeypatch.setattr(hip_build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(hip_build, "MARSHAL_PATH", str(tmp_path / "marshal.so"))
    assert not hip_build.stale()
    os.utime(tmp_path / "marshal.so", (1e9 - 1, 1e9 - 1))
    assert hip_build.stale()
    os.remove(tmp_path / "marshal.so")
    assert hip_build.stale()


def test_missing_marshalling_is_reported(tmp_path):
    """A copy of the package without it: the library loads, with a warning."""
    from paper_2402_13485_amd import binding
    shutil.copytree(os.path.dirname(binding.__file__), tmp_path / "pkg", ignore=shutil.ignore_patterns("_marshal.so", "csrc"))
    code = ("import warnings; warnings.simplefilter('error'); from pkg import binding\n"
            "try: binding.load_library()\nexcept RuntimeWarning as e: print(e)")
    done = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True)
    assert "marshalling is not there" in done.stdout, done
