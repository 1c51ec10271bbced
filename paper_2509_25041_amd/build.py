"""Builds libgrace_moe.so (HIP kernels + C ABI) for gfx950 with hipcc and the binding's native calls with g++, in-tree."""
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

STAMP = os.path.join(HERE, "libgrace_moe.stamp")   # digest of the sources the library was built from
# The binding's calls that allocate, a module of this interpreter; the library does not need it.
CALLS_SOURCE = "torch_calls.cpp"
CALLS = os.path.join(HERE, "_torch_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
CALLS_STAMP = os.path.join(HERE, "_torch_calls.stamp")


def source_digest() -> str:
    """SHA-256 over the names and contents of every file the library is compiled from (content, not
    modification times: a copy of the tree to another machine keeps the answer)."""
    return _digest(n for n in os.listdir(CSRC) if n.endswith((".hip", ".h", ".cpp")) and n != CALLS_SOURCE)


def calls_digest() -> str:
    """The same of the native calls, and what they are compiled against."""
    return _digest([CALLS_SOURCE], metadata.version("torch") + sysconfig.get_config_var("EXT_SUFFIX"))


def _digest(names, also: str = "") -> str:
    paths = sorted(os.path.join(CSRC, n) for n in names)
    paths.append(os.path.join(ROOT, "include", "grace_moe.h"))
    h = hashlib.sha256(also.encode())
    for p in paths:
        h.update(os.path.basename(p).encode() + b"\0")
        with open(p, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def is_stale() -> bool:
    """True when the library is absent or was built from other sources than the ones in the tree."""
    return _differs(LIB, STAMP, source_digest)


def calls_are_stale() -> bool:
    return _differs(CALLS, CALLS_STAMP, calls_digest)


def _differs(binary: str, stamp: str, digest) -> bool:
    if not os.path.exists(binary) or not os.path.exists(stamp):
        return True
    with open(stamp) as fh:
        return fh.read().strip() != digest()


def build(verbose: bool = False) -> str:
    """The library and the native calls, side by side."""
    try:
        calls = _compile_calls()
    finally:
        lib = build_library(verbose)   # (also where there is no g++)
    _finish_calls(calls)
    return lib


def build_calls() -> str:
    _finish_calls(_compile_calls())
    return CALLS


def _compile_calls() -> subprocess.Popen:
    torch_dir = util.find_spec("torch").submodule_search_locations[0]
    inc = os.path.join(torch_dir, "include")
    return subprocess.Popen(
        ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=1", "-I", os.path.join(ROOT, "include"), "-isystem", inc,
         "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
         os.path.join(CSRC, CALLS_SOURCE), "-o", CALLS, "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"],
        stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _finish_calls(process: subprocess.Popen) -> None:
    digest = calls_digest()
    out, _ = process.communicate()
    if process.returncode != 0:
        raise RuntimeError(f"compilation of {CALLS_SOURCE} failed\n{out}")
    with open(CALLS_STAMP, "w") as fh:
        fh.write(digest + "\n")


def build_library(verbose: bool = False) -> str:
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
