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
])
def test_waves(dtype, H, N, d, causal, waves):
    assert rules.waves(dtype, 1, H, N, d, causal) == waves
