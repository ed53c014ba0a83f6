"""The calls whose speed this package is kept to: attention forward as programs
make it, through ``fwd`` and ``fwd_fp8``.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges.
A case is a dict of plain values: the storage type, batch, query heads,
key/value heads, tokens, head widths, mask, tensor layout and the factor on Q
and K (2 for sharper rows).  ``prepare`` makes the tensors a program has in
hand before the call, ``run`` is one forward call with its outputs allocated by
the call, ``exact`` the same in 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_2506_12355_amd as qa

E4M3_MAX = 448.0


def _case(name, dtype, B, H, N, d, causal, Hkv=None, dv=None, layout="bhnd", mult=1.0):
    return {"name": name, "dtype": dtype, "B": B, "H": H, "Hkv": Hkv or H, "N": N, "d": d,
            "dv": dv or d, "causal": causal, "layout": layout, "mult": mult}


def listed():
    return [
        # a single short sequence on two heads: the smallest call, all latency
        _case("tiny_f16_d64", "f16", 1, 2, 128, 64, False),
        # one prompt of an odd length with grouped heads (64 query, 8 key/value): a
        # request that is prefilled by itself
        _case("prompt_gqa_bf16", "bf16", 1, 64, 1000, 128, True, Hkv=8),
        # many short training sequences, causal, hidden size 2048
        _case("short_causal_bf16", "bf16", 32, 16, 512, 128, True),
        # an encoder's batch: narrow heads, no mask
        _case("encoder_f16_d64", "f16", 8, 16, 1024, 64, False),
        # tensors as the projections write them, [B][N][heads][d]
        _case("projected_bf16", "bf16", 16, 16, 1024, 128, False, layout="bnhd"),
        # a causal batch of middling length in fp16
        _case("batch_causal_f16", "f16", 4, 32, 2048, 128, True),
        # queries and keys wider than values (multi-head latent attention, 128 + 64)
        _case("latent_bf16", "bf16", 1, 16, 4096, 192, True, dv=128),
        # 8k tokens without and with the mask: the workload the package is quoted on
        _case("long_bf16", "bf16", 2, 32, 8192, 128, False),
        _case("long_causal_bf16", "bf16", 2, 32, 8192, 128, True),
        # the same in FP8 with per-tensor scales
        _case("long_causal_fp8", "e4m3", 2, 32, 8192, 128, True),
        # one 16k-token sequence of narrow heads
        _case("long_bf16_d64", "bf16", 1, 32, 16384, 64, False),
        # one 32k-token document, causal, sharper rows
        _case("document_bf16", "bf16", 1, 32, 32768, 128, True, mult=2.0),
    ]


def draw(rng):
    """A case of the same ranges: 128 to 32768 tokens, ragged counts
    among them, 1 to 32 sequences, the head widths above, every type, mask and layout."""
    dtype = rng.choice(("f16", "bf16", "bf16", "e4m3"))
    d = 128 if dtype == "e4m3" else rng.choice((64, 64, 128, 128, 128, 192))
    N = int(round(math.exp(rng.uniform(math.log(128), math.log(32768)))))
    if rng.random() < 0.3:
        N = max(128, N // 64 * 64)
    H = rng.choice((2, 8, 16, 32, 64))
    group = 1 if d == 192 else rng.choice((1, 1, 4, 8))
    Hkv = max(1, H // group)
    causal = rng.random() < 0.6
    layout = "bnhd" if d != 192 and rng.random() < 0.2 else "bhnd"
    mult = 2.0 if dtype != "e4m3" and rng.random() < 0.2 else 1.0
    # at most 16k tokens in all, and no more work than the largest listed case
    B = max(1, min(32, int(math.exp(rng.uniform(0.0, math.log(max(1.0, 16384 / N)))))))
    case = _case("", dtype, B, H, N, d, causal, Hkv=Hkv, dv=128 if d == 192 else d,
                 layout=layout, mult=mult)
    most = work(listed()[-1])["flops"]
    while work(case)["flops"] > most:
        case["N"] -= case["N"] // 8
    del case["name"]
    return case


def _shape(case, heads, width):
    if case["layout"] == "bnhd":
        return (case["B"], case["N"], heads, width)
    return (case["B"], heads, case["N"], width)


def _inputs(case, seed):
    """q, k, v and the FP8 scales (None for 16-bit types): normal draws, FP8 ones
    scaled per tensor so that the largest magnitude is 448."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    out, scales = [], []
    for i, (heads, width) in enumerate(((case["H"], case["d"]), (case["Hkv"], case["d"]),
                                        (case["Hkv"], case["dv"]))):
        x = torch.randn(_shape(case, heads, width), generator=gen, device="cuda")
        if i < 2 and case["mult"] != 1.0:
            x *= case["mult"]
        if case["dtype"] == "e4m3":
            s = float(x.abs().max()) / E4M3_MAX
            out.append((x / s).clamp_(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn))
            scales.append(s)
        else:
            out.append(x.to(torch.float16 if case["dtype"] == "f16" else torch.bfloat16))
    return out, (tuple(scales) or None)


def prepare(case, seed):
    (q, k, v), scales = _inputs(case, seed)
    return {"q": q, "k": k, "v": v, "scales": scales, "causal": case["causal"],
            "layout": case["layout"]}


def run(state):
    if state["scales"] is not None:
        return qa.fwd_fp8(state["q"], state["k"], state["v"], state["scales"],
                          causal=state["causal"], layout=state["layout"])
    return qa.fwd(state["q"], state["k"], state["v"], causal=state["causal"],
                  layout=state["layout"])


def work(case):
    B, H, N = case["B"], case["H"], case["N"]
    es = 1 if case["dtype"] == "e4m3" else 2
    pairs = N * (N + 1) // 2 if case["causal"] else N * N
    moved = B * N * (es * (H * case["d"] + case["Hkv"] * (case["d"] + case["dv"]))
                     + H * (2 * case["dv"] + 4))
    return {"bytes": moved, "flops": 2 * B * H * pairs * (case["d"] + case["dv"])}


def tolerance(case):
    """About four times the distance of the outputs from the 64-bit result: the
    storage type of the output and of the probabilities (FP8: 3 mantissa bits)."""
    return {"rel": {"f16": 1.2e-3, "bf16": 1e-2, "e4m3": 0.11}[case["dtype"]]}


def exact(case, seed):
    """(o, lse) in 64 bits: softmax(mask(scale q k^T)) v head by head, rows in blocks."""
    (q, k, v), scales = _inputs(case, seed)
    qs, ks, vs = scales or (1.0, 1.0, 1.0)
    B, H, N, dv = case["B"], case["H"], case["N"], case["dv"]
    scale = float(torch.tensor(1.0 / case["d"] ** 0.5, dtype=torch.float32)) * qs * ks
    o = torch.empty(_shape(case, H, dv), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, N), dtype=torch.float64, device="cuda")
    bnhd = case["layout"] == "bnhd"
    rows = max(1, min(N, (1 << 28) // N))
    keys = torch.arange(N, device="cuda")

    def head(t, b, h):
        x = t[b, :, h] if bnhd else t[b, h]
        return x.float().double().contiguous()

    for b in range(B):
        for h in range(H):
            g = h // (H // case["Hkv"])
            if h % (H // case["Hkv"]) == 0:
                kt, vh = head(k, b, g).t().contiguous(), head(v, b, g) * vs
            qh = head(q, b, h) * scale
            oh = o[b, :, h] if bnhd else o[b, h]
            for r in range(0, N, rows):
                e = min(N, r + rows)
                last = e if case["causal"] else N
                s = qh[r:e] @ kt[:, :last].contiguous()
                if case["causal"]:
                    s.masked_fill_(keys[None, :last] > keys[r:e, None], -math.inf)
                m = s.amax(dim=1, keepdim=True)
                s.sub_(m).exp_()
                total = s.sum(dim=1, keepdim=True)
                oh[r:e] = (s @ vh[:last]) / total
                lse[b, h, r:e] = (m + total.log())[:, 0]
    return o, lse
