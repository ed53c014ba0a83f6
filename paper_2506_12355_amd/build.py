"""Build the gfx950 attention library in place: ``libqm_attn.so`` beside this file.

Usage: ``python -m paper_2506_12355_amd.build`` (or call :func:`build`).  It
always recompiles.  hipcc cross-compiles for gfx950 without a GPU present.

It also builds ``libqm_attn_debug.so``, the same sources with
``-DQM_DEBUG_SYNC``: a barrier after every key block on top of the K/V ring
protocol's own.  The tests check that it gives the same bytes as the release
library; nothing else loads it.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_NAME = "libqm_attn.so"
LIB_PATH = os.path.join(PKG_DIR, LIB_NAME)
DEBUG_LIB_PATH = os.path.join(PKG_DIR, "libqm_attn_debug.so")

SOURCES = ["qm_attn.cpp", "attn_fwd_gfx950.hip", "attn_fwd_split_gfx950.hip",
           "attn_fwd_rows128_gfx950.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    # no packed fp32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # device code never sees a NaN in valid use: fmax needs no quieting of its inputs
    "-Xarch_device", "-fno-honor-nans",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = shutil.which("hipcc") or os.path.join(rocm, "bin", "hipcc")
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found; a ROCm toolchain is required to build")
    return path


def compile_command(source: str, out_path: str, debug_sync: bool = False) -> list:
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    return ([hipcc()] + flags + (["-DQM_DEBUG_SYNC"] if debug_sync else [])
            + ["-I", INCLUDE, "-I", CSRC, "-c", "-o", out_path, os.path.join(CSRC, source)])


def link_command(objects: list, out_path: str) -> list:
    return [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out_path] + objects


def _run_all(commands: list, verbose: bool) -> None:
    """Run the commands, as many at once as there are CPUs to keep busy."""
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        return cmd, subprocess.run(cmd, capture_output=True, text=True)

    failed = []
    with ThreadPoolExecutor(max_workers=min(len(commands), len(os.sched_getaffinity(0)), 16)) as ex:
        for cmd, res in ex.map(run, commands):
            if res.returncode != 0:
                failed.append(f"{' '.join(cmd)} failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")
            elif verbose and res.stderr.strip():
                print(res.stderr, file=sys.stderr)
    if failed:
        raise RuntimeError("\n".join(failed))


def build(verbose: bool = False) -> str:
    """Compile every source into ``libqm_attn.so`` and ``libqm_attn_debug.so``
    (sources compiled side by side; each library atomically replaced)."""
    with tempfile.TemporaryDirectory() as tmp:
        compiles, links = [], []
        for path, debug in ((LIB_PATH, False), (DEBUG_LIB_PATH, True)):
            objects = [os.path.join(tmp, f"{s}.{int(debug)}.o") for s in SOURCES]
            compiles += [compile_command(s, o, debug) for s, o in zip(SOURCES, objects)]
            links.append(link_command(objects, path + f".tmp{os.getpid()}"))
        _run_all(compiles, verbose)
        _run_all(links, verbose)
    for path in (LIB_PATH, DEBUG_LIB_PATH):
        os.replace(path + f".tmp{os.getpid()}", path)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
