"""Grids too small to fill the device: causal query blocks run one per
workgroup instead of in pairs, in an order that depends on how the heads fall on
the XCDs, and the smallest grids split their keys over two or four groups of a
workgroup's wavefronts.  Shapes on both sides of each rule, head counts that do
and do not divide over the XCDs, ragged lengths; every output against the
oracle."""
from __future__ import annotations

import math

import numpy as np
import pytest

import seeded_inputs as si
from oracle import attention_fp64
from tests.gpu_util import check_close, half_ulp, to_device, to_host64

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
    (1, 40, 8, 1000, 128, "f16"),     # whole heads per XCD, some CUs with two blocks
    (1, 54, 18, 640, 64, "bf16"),     # heads shared between XCDs, blocks left over
    (2, 80, 80, 200, 128, "bf16"),    # heads of two blocks
    (3, 33, 33, 700, 128, "bf16"),    # past what is resident: pairs
])
def test_causal_small_grid_matches_oracle(qa, B, H, Hkv, N, d, dtype):
    print(f"case small grid B={B} H={H} Hkv={Hkv} N={N} d={d} {dtype}", flush=True)
    q, k, v = si.make_qkv(B, H, N, d, dtype, seed=310 + N + H, Hkv=Hkv)
    tq, tk, tv = (to_device(x, dtype) for x in (q, k, v))
    o, lse = qa.fwd(tq, tk, tv, causal=True)
    Or, lr = attention_fp64(q, k, v, si.default_scale(d), True, dtype)
    check_close(to_host64(o), to_host64(lse), Or, lr, dtype, f"small grid {B}x{H}x{N}")


# (B, H, Hkv, N, d, dtype, causal, scale multiplier): the lengths on both sides of
# the rules for two and four key groups on 256 CUs, one block past a whole number of
# group steps, query blocks in pairs, a negative and a negligible scale
SPLIT = [
    (1, 2, 2, 384, 64, "f16", False, 1.0), (1, 2, 2, 383, 64, "f16", False, 1.0),
    (1, 6, 2, 385, 64, "bf16", True, 1.0), (3, 5, 5, 1001, 64, "bf16", True, 1.0),
    (1, 4, 1, 4100, 64, "f16", True, 1.0), (1, 7, 7, 4223, 64, "bf16", True, 1.0),
    (1, 30, 10, 1000, 64, "f16", False, -1.0), (2, 16, 16, 768, 64, "bf16", True, 0.0),
    (1, 3, 3, 1536, 128, "bf16", False, 1.0), (1, 3, 3, 1535, 128, "bf16", False, 1.0),
    (1, 5, 5, 1600, 128, "f16", True, 1.0), (2, 3, 1, 1793, 128, "bf16", True, -1.0),
    (1, 12, 4, 4097, 128, "f16", True, 1.0), (1, 2, 2, 2111, 128, "bf16", False, 0.0),
]


@pytest.mark.parametrize("B,H,Hkv,N,d,dtype,causal,mult", SPLIT)
def test_key_groups_match_oracle_in_both_layouts(qa, B, H, Hkv, N, d, dtype, causal, mult):
    import torch
    print(f"case key groups {B}x{H}/{Hkv}x{N}x{d} {dtype} causal={causal} scale x{mult}", flush=True)
    q, k, v = si.make_qkv(B, H, N, d, dtype, seed=410 + N + H, Hkv=Hkv)
    scale = si.default_scale(d) * mult
    tq, tk, tv = (to_device(x, dtype) for x in (q, k, v))
    o, lse = qa.fwd(tq, tk, tv, causal=causal, scale=scale)
    Or, lr = attention_fp64(q, k, v, scale, causal, dtype)
    check_close(to_host64(o), to_host64(lse), Or, lr, dtype, f"key groups {B}x{H}x{N}x{d}")
    bn = [t.transpose(1, 2).contiguous() for t in (tq, tk, tv)]
    o2, lse2 = qa.fwd(*bn, causal=causal, scale=scale, layout="bnhd")
    assert torch.equal(o2.transpose(1, 2).contiguous().view(torch.int16), o.view(torch.int16))
    assert torch.equal(lse2.view(torch.int32), lse.view(torch.int32))


@pytest.mark.parametrize("B,H,Hkv,N", [(1, 3, 3, 384), (1, 4, 2, 1000), (2, 8, 8, 1000), (1, 5, 1, 4161)])
@pytest.mark.parametrize("causal", [False, True])
def test_fp8_key_groups_exact_weights(qa, B, H, Hkv, N, causal):
    """Weights that are exact in E4M3, so only fp32 sums and the bf16 store round:
    each of up to N + 128 sums moves a row by 2^-24 of sum P|v| twice over."""
    import torch
    print(f"case FP8 key groups {B}x{H}/{Hkv}x{N} causal={causal}", flush=True)
    codes8 = si.make_qkv_fp8_dyadic(B, H, N, 128, seed=510 + N, v_binade=True, Hkv=Hkv)
    codes = [torch.from_numpy(x).cuda().view(torch.float8_e4m3fn) for x in codes8]
    scales = (0.5, 2.0, 0.0123)
    o, lse = qa.fwd_fp8(*codes, scales, causal=causal, scale=math.log(2.0))
    q8, k8, v8 = codes8
    Or, lr = attention_fp64(q8, k8, v8, math.log(2.0), causal, "e4m3", descale=scales)
    PV, _ = attention_fp64(q8, k8, v8 & 0x7F, math.log(2.0), causal, "e4m3", descale=scales)
    bound = half_ulp(Or, "bf16") + (2 * (N + 128) * 2.0 ** -24 + 1e-5) * PV
    assert np.all(np.abs(to_host64(o) - Or) <= bound)
    assert np.max(np.abs(to_host64(lse) - lr)) <= 1e-3
    bn = [t.transpose(1, 2).contiguous() for t in codes]
    o2, lse2 = qa.fwd_fp8(*bn, scales, causal=causal, scale=math.log(2.0), layout="bnhd")
    assert torch.equal(o2.transpose(1, 2).contiguous().view(torch.int16), o.view(torch.int16))
    assert torch.equal(lse2.view(torch.int32), lse.view(torch.int32))


@pytest.mark.parametrize("B,H,N,d,dtype", [(2, 160, 500, 64, "bf16"), (2, 130, 700, 128, "f16")])
def test_tile_sizes_agree_on_full_grids(qa, B, H, N, d, dtype):
    """Grids past the key groups' rules, where a forced tile size does choose
    between 128- and 256-row workgroups: the same bytes."""
    import torch
    print(f"case full grid tiles {B}x{H}x{N}x{d} {dtype}", flush=True)
    tq, tk, tv = (to_device(x, dtype) for x in si.make_qkv(B, H, N, d, dtype, seed=610 + N))
    try:
        for causal in (False, True):
            res = []
            for rows in (128, 256, 0):
                qa.set_tile_rows(rows)
                res.append(qa.fwd(tq, tk, tv, causal=causal))
            for o, lse in res[1:]:
                assert torch.equal(o.view(torch.int16), res[0][0].view(torch.int16))
                assert torch.equal(lse.view(torch.int32), res[0][1].view(torch.int32))
    finally:
        qa.set_tile_rows(0)


@pytest.mark.parametrize("B,H,Hkv,N,d,dv,dtype,layout,rows", [
    (1, 3, 3, 1100, 64, 64, "bf16", 0, 0),     # four key groups
    (1, 3, 1, 2177, 128, 128, "f16", 1, 0),    # two key groups, two-block rings
    (1, 9, 9, 1300, 64, 64, "f16", 0, 0),      # two key groups, four-block rings
    (1, 48, 48, 900, 128, 128, "bf16", 1, 0),  # 128-row [B][N][H][d]
    (1, 5, 5, 900, 192, 128, "bf16", 0, 0),    # 128-row, 192-wide keys
    (2, 80, 80, 900, 64, 64, "bf16", 0, 256),  # eight waves, deferred second product
])
def test_checking_build_gives_the_same_bytes(qa, B, H, Hkv, N, d, dv, dtype, layout, rows):
    """The build with a barrier per key block agrees on the small grids' routes, whose
    groups share barriers and exchange results through the rings' LDS."""
    import torch
    print(f"case checking build {B}x{H}x{N}x{d} {dtype} layout={layout}", flush=True)
    libs = (qa.load_library(), qa.open_library(qa.DEBUG_LIB_PATH))
    tq, tk, tv = (to_device(x, dtype) for x in si.make_qkv(B, H, N, d, dtype, seed=710 + N, Hkv=Hkv, dv=dv))
    if layout:
        tq, tk, tv = (t.transpose(1, 2).contiguous() for t in (tq, tk, tv))
    try:
        for causal in (0, 1):
            res = []
            for lib in libs:
                assert lib.qm_attn_set_tile_rows(rows) == 0
                o = torch.full((B, N, H, dv) if layout else (B, H, N, dv), float("nan"),
                               dtype=tq.dtype, device="cuda")
                lse = torch.full((B, H, N), float("nan"), device="cuda")
                assert lib.qm_attn_fwd_layout(
                    tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), o.data_ptr(), lse.data_ptr(), B, H,
                    Hkv, N, d, dv, si.default_scale(d), causal,
                    torch.cuda.current_stream().cuda_stream, 0 if dtype == "f16" else 1, layout) == 0
                torch.cuda.synchronize()
                res.append((o.view(torch.int16), lse.view(torch.int32)))
            assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    finally:
        for lib in libs:
            lib.qm_attn_set_tile_rows(0)
