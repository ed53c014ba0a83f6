"""Grids too small to fill the device: causal query blocks run one per
workgroup instead of in pairs, in an order that depends on how the heads fall on
the XCDs.  Shapes on both sides of each rule, head counts that do and do not
divide over the XCDs, ragged lengths; every output against the oracle."""
from __future__ import annotations

import pytest

import seeded_inputs as si
from oracle import attention_fp64
from tests.gpu_util import check_close, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qa():
    import torch
    import paper_2506_12355_amd as qa
    assert torch.cuda.is_available()
    qa.load_library()
    return qa


@pytest.mark.parametrize("B,H,Hkv,N,d,dtype", [
    (1, 1, 1, 300, 128, "bf16"),      # fewer tiles than XCDs
    (1, 12, 3, 1300, 128, "f16"),     # heads straddle the XCDs' halves
    (2, 8, 8, 1025, 64, "bf16"),      # whole heads per half, a last block of one row
    (1, 64, 8, 1000, 128, "bf16"),    # two query blocks to a CU
    (5, 13, 13, 1000, 64, "f16"),     # just under three to a CU
    (3, 33, 33, 700, 128, "bf16"),    # past what is resident: pairs
])
def test_causal_small_grid_matches_oracle(qa, B, H, Hkv, N, d, dtype):
    print(f"case small grid B={B} H={H} Hkv={Hkv} N={N} d={d} {dtype}", flush=True)
    q, k, v = si.make_qkv(B, H, N, d, dtype, seed=310 + N + H, Hkv=Hkv)
    tq, tk, tv = (to_device(x, dtype) for x in (q, k, v))
    o, lse = qa.fwd(tq, tk, tv, causal=True)
    Or, lr = attention_fp64(q, k, v, si.default_scale(d), True, dtype)
    check_close(to_host64(o), to_host64(lse), Or, lr, dtype, f"small grid {B}x{H}x{N}")
