"""The choice of an instance per call (csrc/attn_fwd_rules.h) on 256 CUs (CPU only)."""
from __future__ import annotations

import pytest

from paper_2506_12355_amd import build as qbuild
from tests import rules


@pytest.fixture(autouse=True)
def _compiler():
    try:
        qbuild.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")


@pytest.mark.parametrize("dtype,H,N,d,causal,groups", [
    ("f16", 2, 384, 64, False, 4), ("f16", 2, 383, 64, False, 1), ("bf16", 30, 1000, 64, False, 2),
    ("bf16", 3, 1536, 128, False, 2), ("bf16", 3, 1535, 128, True, 1), ("e4m3", 3, 384, 128, True, 4),
    ("f16", 2, 8192, 192, True, 1), ("bf16", 8, 4096, 128, True, 2), ("bf16", 17, 4096, 128, True, 1),
])
def test_key_groups(dtype, H, N, d, causal, groups):
    assert rules.key_groups(dtype, 1, H, N, d, causal) == groups


@pytest.mark.parametrize("dtype,H,N,d,causal,waves", [
    ("bf16", 64, 8192, 128, False, 8), ("bf16", 512, 512, 128, True, 4), ("f16", 128, 4096, 64, False, 4),
    ("e4m3", 64, 8192, 128, True, 8), ("bf16", 16, 4096, 192, True, 4), ("bf16", 256, 8192, 192, True, 8),
    ("bf16", 24, 4096, 128, True, 8), ("bf16", 96, 3000, 128, False, 4),
    # past a whole round, heads' middle blocks only (else whole pairs)
    ("bf16", 8, 8256, 128, True, 4), ("f16", 8, 8256, 64, True, 4), ("e4m3", 8, 8193, 128, True, 4),
    ("bf16", 8, 8321, 128, True, 8), ("e4m3", 24, 5376, 128, True, 4), ("bf16", 8, 8193, 192, True, 8),
    ("bf16", 8, 16500, 128, True, 8), ("bf16", 8, 16500, 64, True, 4), ("e4m3", 8, 16500, 128, True, 8),
])
def test_waves(dtype, H, N, d, causal, waves):
    assert rules.waves(dtype, 1, H, N, d, causal) == waves


def test_grid():
    """One workgroup per tile for FP8 two to a CU and a last round of more than one tile
    to a CU, as far as a grid's 2^31 threads reach; else what is resident."""
    def grid(total, dtype="e4m3", per_cu=2, N=2048, cus=256):
        return rules.library().grid(total, cus * per_cu // 8 * 8, cus, per_cu, 256, rules.DTYPES[dtype], N)

    most = (2 ** 31 - 1) // 256
    assert [grid(t) for t in (1, 512, 513, 768, 769, 1024, 1025)] == [1, 512, 512, 512, 769, 1024, 512]
    assert grid(most // 512 * 512) == most // 512 * 512 and grid(2 ** 31 - 1) == 512
    assert grid(769, dtype="bf16") == 512 and grid(769, N=1000) == 512
    assert grid(300, per_cu=1) == 256 and grid(511, per_cu=1) == 256
    assert grid(5, cus=3) == 5   # too few CUs for a round of the XCDs
