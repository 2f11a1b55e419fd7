"""Builds libpipad.so (HIP, gfx950 only) in-tree with hipcc, and the native half of the binding with g++.

    python -m paper_2301_00391_amd.build [-v] [-D NAME[=VALUE] ...] [-o PATH]

The native half is built for one interpreter and one torch, whose names its file bears (_host.*.so): another
interpreter or torch does not meet it.  With -o, or -D, the library alone is built.
-D passes a macro to every source: the measurement builds the profiles are taken with, e.g.
-D PIPAD_PARTS_MASK=1 (only the class parts of the hub rows run: results incomplete),
-D PIPAD_AGG_DEPTH=2, -D PIPAD_NO_ROW_ORDER.  -o writes the library somewhere else than in-tree;
the binding loads the file the environment variable PIPAD_LIBRARY names instead of the in-tree one.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpipad.so")
SOURCES = ["pipad_api.hip", "pipad_build.hip", "pipad_aggregate.hip", "pipad_transpose.hip",
           "pipad_ceilings.hip"]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: libpipad needs the ROCm toolchain")


def check_private_memory(remarks: str, limit: int = 64) -> None:
    """Fails the build when a kernel keeps more than a few spilled registers in private (scratch)
    memory.  The aggregation kernels take their arguments as one large struct; if the compiler
    cannot prove that it is only read at constant offsets it copies the whole struct (over 2 KB)
    into every lane's private memory, which costs an order of magnitude in run time and no test
    would notice."""
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "ScratchSize [bytes/lane]:" in line and name:
            size = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
            if size > limit and "5pipad" in name:  # this library's kernels (namespace pipad)
                raise RuntimeError(f"kernel {name} uses {size} bytes of private memory per lane "
                                   f"(limit {limit}): kernel arguments copied to scratch?")


def build(verbose: bool = False, defines=(), output: str = LIB) -> str:
    """Compiles every HIP source for gfx950 and links the shared library.  Always rebuilds."""
    flags = [*[f"-D{d}" for d in defines],
        "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
        # packed fp32 instructions are kept off on this target
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function",
    ]
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", f".{os.getpid()}.o"))
        cmd = [hipcc(), *flags, "-Rpass-analysis=kernel-resource-usage", "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stderr=subprocess.PIPE, text=True)))
        objs.append(obj)
    for cmd, p in procs:
        _, err = p.communicate()
        if p.returncode != 0:
            sys.stderr.write(err)
            raise RuntimeError("hipcc failed: " + " ".join(cmd))
        check_private_memory(err)
    link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", output, *objs]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.run(link, check=True)
    for o in objs:
        os.remove(o)
    return output


def host_path() -> str:
    """Where the native half of the binding for this interpreter and its torch lies."""
    import torch
    return os.path.join(HERE, f"_host.{sys.implementation.cache_tag}.torch-{re.sub('[^0-9A-Za-z.]', '_', torch.__version__)}.so")


def build_host(verbose: bool = False, output: str = "") -> str:
    """Compiles the native half of the binding against this interpreter and its torch.  Always rebuilds; the file is whole as soon as
    it is there (other processes may load it meanwhile)."""
    import sysconfig
    import torch
    output = output or host_path()
    root, part = os.path.dirname(torch.__file__), f"{output}.{os.getpid()}.part"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[a for d in (os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                         sysconfig.get_paths()["include"]) for a in ("-isystem", d)],
           "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "pipad_host.cpp"), "-o", part,
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, check=True)
        os.replace(part, output)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return output


def main(argv=None) -> None:
    import argparse
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("-v", action="store_true", help="print the compiler command lines")
    ap.add_argument("-D", action="append", default=[], metavar="NAME[=VALUE]")
    ap.add_argument("-o", default=LIB, metavar="PATH")
    a = ap.parse_args(argv)
    print(build(verbose=a.v, defines=a.D, output=a.o))
    if a.o == LIB and not a.D:
        print(build_host(verbose=a.v))


if __name__ == "__main__":
    main()
