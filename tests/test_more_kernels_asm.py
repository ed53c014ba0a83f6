"""The compiled kernels outside attn_fwd_gfx950.hip (CPU only), under the rules
that file's kernels are held to: no SGPR hazard at a direct load, one s_nop before
each, no packed fp32 instruction, no spilled VGPR, no scratch, and at most 256
VGPRs."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2506_12355_amd import build as qbuild
from tests.asm_hazards import dma_sgpr_hazards_cfg, instructions, is_direct_load

SOURCES = [s for s in qbuild.SOURCES if s.endswith(".hip") and s != "attn_fwd_gfx950.hip"]


@pytest.mark.parametrize("debug", [False, True])
@pytest.mark.parametrize("source", SOURCES)
def test_compiled_kernels(tmp_path, source, debug):
    try:
        qbuild.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    out = str(tmp_path / "k.s")
    cmd = qbuild.compile_command(source, out, debug_sync=debug)
    cmd[cmd.index("-c")] = "-S"
    res = subprocess.run(cmd + ["--cuda-device-only"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    text = open(out).read()
    kernels = list(re.finditer(r"^(_Z\w*attn_fwd\w*_kernel\w*):\s*(?:;.*)?$", text, flags=re.M))
    assert kernels
    for m in kernels:
        body = text[m.end():text.index(".Lfunc_end", m.end())]
        insts = instructions(body)
        assert any(is_direct_load(i) for i in insts), m.group(1)
        bad = dma_sgpr_hazards_cfg(body)
        assert not bad, f"{m.group(1)}: {bad[:3]}"
        for i, inst in enumerate(insts):
            if is_direct_load(inst):
                assert i > 0 and insts[i - 1].startswith("s_nop"), (m.group(1), i, inst)
        packed = [i for i in insts if re.match(r"v_pk_(add|mul|fma|mov)_f32", i)]
        assert not packed, f"{m.group(1)}: {packed[:3]}"
    for key, most in (("vgpr_spill_count", 0), ("private_segment_fixed_size", 0), ("vgpr_count", 256)):
        values = [int(x) for x in re.findall(rf"\.{key}:\s+(\d+)", text)]
        assert len(values) == len(kernels) and max(values) <= most, (key, values)
