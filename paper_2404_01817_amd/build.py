"""Build the HIP library ``libneat.so`` for gfx950 (MI355X) in-tree.

``csrc/node_loop_asm.h`` and ``csrc/node_loop_wide.h`` are regenerated by
``csrc/gen_node_loop.py`` and checked by ``csrc/check_node_loop.py`` (wait states, load completion,
GPR-index mode, clobbers), then every ``csrc/*.hip`` file is compiled by hipcc into an object under
``paper_2404_01817_amd/_build/`` (in parallel), then linked into
``paper_2404_01817_amd/libneat.so``.  Packed fp32 instructions are disabled
for device code (``-packed-fp32-ops``); hipcc's host pass warns that it does
not know that feature, which is harmless.

    python -m paper_2404_01817_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libneat.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

CFLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wall", "-Wno-unused-command-line-argument",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *CFLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False) -> str:
    """Regenerate the assembly node loop, compile every source and link
    libneat.so; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    r = subprocess.run([sys.executable, os.path.join(CSRC, "gen_node_loop.py")],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("gen_node_loop.py failed:\n" + r.stderr)
    # the generated assembly must pass its static hazard checks
    r = subprocess.run([sys.executable, os.path.join(CSRC, "check_node_loop.py")],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("the node loop fails its hazard checks:\n" + r.stdout)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
