"""Build the HIP library for gfx950 with hipcc (cross-compiles without a GPU), and the native argument
marshalling of the Python binding with the host compiler."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libpropd.so")
MARSHAL_PATH = os.path.join(HERE, "_marshal.so")
MARSHAL_SOURCE = "marshal.cpp"
HEADER = os.path.join(HERE, os.pardir, "include", "propd.h")
SOURCES = ["tree_mask.hip", "tree_attention.hip", "early_prune.hip", "accept_path.hip",
           "commit_path.hip", "tree_controller.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",  # no packed-fp32 codegen
    "-fvisibility=hidden", "-Wall",
]


# Kernels with loads or LDS reads in flight that the compiler does not track (they are waited for
# by hand).  A register that is saved to scratch memory or to an accumulation register while such a load
# is on its way is saved before the value is there, and the load then lands in a register that
# holds something else by that time, an address for instance.
HAND_WAITED = ("tree_attn_bf16_kernel", "early_head_bf16_kernel")


def unsafe_kernels(remarks: str) -> list:
    """Kernels of HAND_WAITED that spill, from the compiler's remarks on resource usage."""
    found, seen = [], set()
    for block in remarks.split("Function Name: ")[1:]:
        name = block.split()[0]
        used = {key: int(value) for key, value in
                re.findall(r"(AGPRs|ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", block)}
        for kernel in HAND_WAITED:
            if kernel in name:
                seen.add(kernel)
                if len(used) != 3 or any(used.values()):
                    found.append(f"{name}: {used}")
    return found + [f"{kernel}: no resource usage reported" for kernel in HAND_WAITED if kernel not in seen]


def has_marshal() -> bool:
    return os.path.exists(os.path.join(CSRC, MARSHAL_SOURCE))


def stale() -> bool:
    """Whether the library or the native marshalling is missing, or older than a source."""
    sources = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [HEADER, os.path.abspath(__file__)]
    newest = max(map(os.path.getmtime, sources))
    return any(not os.path.exists(made) or os.path.getmtime(made) < newest
               for made in [LIB_PATH] + [MARSHAL_PATH] * has_marshal())


def marshal_command(out: str) -> list:
    from torch.utils import cpp_extension
    includes = cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", *("-I" + i for i in includes),
            "-o", out, os.path.join(CSRC, MARSHAL_SOURCE), *("-L" + d for d in cpp_extension.library_paths()),
            "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_marshal(verbose: bool) -> bool:
    """The native marshalling as MARSHAL_PATH + ".new"; False if it cannot be built here (no host compiler, no
    PyTorch headers): the binding marshals in Python then, and says so."""
    try:
        cmd = marshal_command(MARSHAL_PATH + ".new")
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return True
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        print(f"the native marshalling is not built: {e}", file=sys.stderr, flush=True)
        return False


def build(verbose: bool = False) -> str:
    """Both are replaced only when the library is built: they share the structures of the header."""
    marshal = has_marshal() and build_marshal(verbose)
    try:
        build_library(verbose)
    except BaseException:
        if marshal:
            os.remove(MARSHAL_PATH + ".new")
        raise
    os.replace(LIB_PATH + ".new", LIB_PATH)
    if marshal:
        os.replace(MARSHAL_PATH + ".new", MARSHAL_PATH)
    elif has_marshal() and os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)  # made for the library before
    return LIB_PATH


def build_library(verbose: bool) -> None:
    """The library as LIB_PATH + ".new"."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    extra = os.environ.get("PROPD_EXTRA_HIPCC_FLAGS", "").split()  # tuning experiments only
    new = LIB_PATH + ".new"
    cmd = ["hipcc", *FLAGS, *extra, "-DPROPD_BUILD", "-Rpass-analysis=kernel-resource-usage",
           "-fno-caret-diagnostics", "-o", new, *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    done = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    context = []  # of the next line
    for line in done.stderr.splitlines():
        context.append(line)
        if line.startswith("In file included from"):
            continue
        if "[-Rpass-analysis=kernel-resource-usage]" not in line and "'-packed-fp32-ops' is not a recognized" not in line:
            print("\n".join(context), file=sys.stderr, flush=True)
        context = []
    if done.returncode != 0:
        raise subprocess.CalledProcessError(done.returncode, cmd)
    bad = unsafe_kernels(done.stderr)
    if bad:
        os.remove(new)
        raise RuntimeError("these kernels must not spill, the library is not replaced:\n" + "\n".join(bad))


if __name__ == "__main__":
    build(verbose=True)
    print(LIB_PATH)
