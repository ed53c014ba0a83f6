"""The order in which causal query blocks that all run at once are dealt to the
CUs (csrc/tile_order.h), compiled for the host: every tile is taken once, from the
XCD's own stretch of heads, a long block beside a short one."""
from __future__ import annotations

import ctypes
import subprocess

import pytest

from paper_2506_12355_amd import build as qbuild

WRAPPER = """
#include "tile_order.h"
extern "C" void order(int total, int row, int nq, int heads, int* out) {
  for (int w = 0; w < total; ++w) out[w] = qm::balanced_tile(w, total, row, nq, heads);
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    try:
        cc = qbuild.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("order")
    (d / "order.hip").write_text(WRAPPER)
    subprocess.run([cc, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                    "-shared", "-I", qbuild.CSRC, "-o", str(d / "order.so"), str(d / "order.hip")],
                   check=True, capture_output=True)
    lib = ctypes.CDLL(str(d / "order.so"))

    def call(total, row, nq, heads):
        out = (ctypes.c_int * total)()
        lib.order(total, row, nq, heads, out)
        return list(out)

    return call


@pytest.mark.parametrize("cus,per_cu", [(256, 2), (256, 3), (32, 3), (304, 2)])
def test_every_tile_once_and_long_beside_short(order, cus, per_cu):
    """Every head count and block count that the rule for single blocks admits."""
    row = cus // 8
    for nq in range(1, 18):
        for heads in range(1, cus * per_cu // 8 * 8 // nq + 1):
            total = nq * heads
            if total <= cus:
                continue
            tiles = order(total, row, nq, 0 if heads % 8 else heads // 8)
            assert sorted(tiles) == list(range(total)), (nq, heads)
            p, left = divmod(total, 8)
            blocks = [t % 8 * p + t // 8 if t < 8 * p else t for t in tiles]   # as the kernel decodes
            first = 0
            for x in range(8):
                took = blocks[x::8]
                n = p + (x < left)
                assert sorted(took) == list(range(first, first + n)), (nq, heads, x)
                first += n
                # the lengths in rows over the XCD's CUs
                took = [nq - b % nq for b in took]
                second = min(row, n - row)
                if nq == 2 and heads % 8 == 0:
                    assert all(a + b == 3 for a, b in zip(took[:row], took[row:row + second]))
                else:
                    want = sorted(took, reverse=True)
                    want[row:row + second] = want[row:row + second][::-1]
                    assert took == want, (nq, heads, x)
