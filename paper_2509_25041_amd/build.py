"""Builds libgrace_moe.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's native calls with g++, in-tree."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig
from importlib import metadata, util

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgrace_moe.so")
SOURCES = ["table.cpp", "route.hip", "permute.hip", "combine.hip", "ffn.hip", "gemm_f32_split_up.hip", "gemm_f32_split_down.hip",
           "gemm_f32_split_shared.hip", "calibrate.hip", "sendlist.hip", "route_permute.hip", "ffn_tiny.hip", "ffn_tiny_mid.hip", "ffn_tiny_cols.hip", "ffn_tiny_down.hip"]

CALLS = os.path.join(HERE, "_torch_calls.so")              # the binding's calls that allocate (csrc/torch_calls.cpp)
STAMP = os.path.join(HERE, "libgrace_moe.stamp")   # digest of the sources the library was built from


def source_digest() -> str:
    """SHA-256 over the names and contents of every file the library is compiled from (content, not
    modification times: a copy of the tree to another machine keeps the answer)."""
    paths = sorted(os.path.join(CSRC, n) for n in os.listdir(CSRC) if n.endswith((".hip", ".h", ".cpp")))
    paths.append(os.path.join(ROOT, "include", "grace_moe.h"))
    h = hashlib.sha256(metadata.version("torch").encode())   # the calls are compiled against it
    for p in paths:
        h.update(os.path.basename(p).encode() + b"\0")
        with open(p, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def is_stale() -> bool:
    """True when the library is absent or was built from other sources than the ones in the tree."""
    if not all(os.path.exists(p) for p in (LIB, CALLS, STAMP)):
        return True
    with open(STAMP) as fh:
        return fh.read().strip() != source_digest()


def build(verbose: bool = False) -> str:
    """Compile every translation unit for gfx950 and link the shared library."""
    objs = []
    common = ["hipcc", "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-x", "hip",
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-Wno-unused-command-line-argument",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src + ".o")
        objs.append(obj)
        cmd = common + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    torch_dir = util.find_spec("torch").submodule_search_locations[0]
    inc = os.path.join(torch_dir, "include")
    procs.append(("torch_calls.cpp", subprocess.Popen(
        ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=1", "-I", os.path.join(ROOT, "include"), "-isystem", inc,
         "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
         os.path.join(CSRC, "torch_calls.cpp"), "-o", CALLS, "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"],
        stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            failed = True
            print(f"--- {src} failed ---\n{out}", file=sys.stderr)
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("compilation failed")
    digest = source_digest()
    link = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(link, check=True)
    with open(STAMP, "w") as fh:
        fh.write(digest + "\n")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
