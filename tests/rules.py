"""Which instance of the kernel a call runs (csrc/attn_fwd_rules.h), asked of the rules
themselves: compiled for the host, without the kernels."""
from __future__ import annotations

import ctypes
import os
import subprocess
import tempfile

from paper_2506_12355_amd import build as qbuild

WRAPPER = """
#include "attn_fwd_rules.h"
static qm::AttnArgs args(int dtype, int B, int H, int N, int d, int causal) {
  qm::AttnArgs a = {};
  a.B = B, a.H = H, a.Hkv = H, a.N = N, a.d = d, a.dv = d == 192 ? 128 : d;
  a.causal = causal, a.dtype = dtype;
  return a;
}
extern "C" int groups(int dtype, int B, int H, int N, int d, int causal, int cus) {
  return qm::key_groups(args(dtype, B, H, N, d, causal), cus);
}
extern "C" int waves(int dtype, int B, int H, int N, int d, int causal, int cus) {
  return qm::choose_waves(args(dtype, B, H, N, d, causal), cus);
}
extern "C" int grid(int total, int resident, int cus, int per_cu, int threads, int dtype, int N) {
  return qm::tile_grid(total, resident, cus, per_cu, threads, dtype, N);
}
"""
DTYPES = {"f16": 0, "bf16": 1, "e4m3": 2}
_lib = None


def library() -> ctypes.CDLL:
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "rules.hip"), os.path.join(d, "rules.so")
            with open(src, "w") as f:
                f.write(WRAPPER)
            subprocess.run([qbuild.hipcc(), "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950",
                            "-O1", "-std=c++17", "-fPIC", "-shared", "-I", qbuild.CSRC, "-o", so, src],
                           check=True, capture_output=True)
            _lib = ctypes.CDLL(so)
    return _lib


def key_groups(dtype: str, B: int, H: int, N: int, d: int, causal: bool, cus: int = 256) -> int:
    return library().groups(DTYPES[dtype], B, H, N, d, int(causal), cus)


def waves(dtype: str, B: int, H: int, N: int, d: int, causal: bool, cus: int = 256) -> int:
    return library().waves(DTYPES[dtype], B, H, N, d, int(causal), cus)
