"""The work this library is used for, as cases that can be timed and checked one by one.

A case is one of three kinds, all through the public binding:
  linear   one quantized linear layer y = x W^T, called eagerly with the plan and workspace that a program keeps
           per layer; batch 1..32 is decoding, larger batches are the tokens of a prompt (prefill);
  block    the linear layers of a decoder block as a serving loop issues them: q, k and v in one grouped call, o,
           gate and up in one grouped call, down; captured once in a HIP graph and replayed per token;
  grouped  layers that read the same activations in one eager grouped call.
Shapes and formats are those of the repository's workloads (synth/__init__.py) and ragged ones between them.
Formats are (v, m, g): vector length, codebooks, group size along K of the scales (-1: one scale per row).
"""
from __future__ import annotations

import math

import torch

import paper_2512_17970_amd as cg

# the (v, m, g) that the repository's workloads use
FORMATS = [(8, 2, -1), (8, 2, 128), (4, 1, -1), (4, 1, 128), (8, 1, -1), (8, 3, -1), (8, 2, 64), (8, 2, 32),
           (4, 1, 32), (8, 1, 128), (8, 1, 16), (16, 4, -1), (16, 3, 32), (8, 2, 16), (8, 2, 8), (4, 1, 4)]


def _linear(name, K, N, v, m, g, B, y_fp32=False):
    return {"name": name, "kind": "linear", "K": K, "N": N, "v": v, "m": m, "g": g, "B": B, "y_fp32": y_fp32}


def _block(name, hidden, kv, inter, v, m, g, B):
    return {"name": name, "kind": "block", "hidden": hidden, "kv": kv, "inter": inter, "v": v, "m": m, "g": g, "B": B}


def listed():
    return [
        # the smallest layer of the workloads, one eager call: launch latency
        _linear("tiny_512x512_v8m1_b1", 512, 512, 8, 1, -1, 1),
        # one token of a Llama-3-8B block in the format of the paper's latency table
        _block("block_8b_v4m1g128_b1", 4096, 1024, 14336, 4, 1, 128, 1),
        # one token of a Llama-3-70B block, 2 bits, one scale per row: the headline configuration
        _block("block_70b_v8m2_b1", 8192, 1024, 28672, 8, 2, -1, 1),
        # the largest single layer of the headline configuration, eagerly
        _linear("up_70b_v8m2_b1", 8192, 28672, 8, 2, -1, 1),
        # the same bits from four codebooks of long vectors (average-bits table), fp32 output
        _linear("up_70b_v16m4_b1_fp32", 8192, 28672, 16, 4, -1, 1, True),
        # a few sequences decoded together: 70B block with group scales, batch 4 of the appendix grid
        _block("block_70b_v8m2g128_b4", 8192, 1024, 28672, 8, 2, 128, 4),
        # batch 8 of the appendix grid on the 8B block
        _block("block_8b_v4m1g128_b8", 4096, 1024, 14336, 4, 1, 128, 8),
        # the batch sweep's middle on the 8B shapes, 2 bits
        _block("block_8b_v8m2_b16", 4096, 1024, 14336, 8, 2, -1, 16),
        # the batch sweep's end: 32 sequences through the down projection
        _linear("down_8b_v8m2_b32", 14336, 4096, 8, 2, -1, 32),
        # odd sizes: three codebooks, a height and a K that no tile divides, an odd batch, fp32 output
        _linear("ragged_v8m3_b5_fp32", 8 * 515, 11111, 8, 3, -1, 5, True),
        # a prompt of 500 tokens through the fused gate and up projections of the 8B block
        _linear("prefill_8b_v4m1g128_b500", 4096, 28672, 4, 1, 128, 500),
        # a long prompt through a square 70B projection
        _linear("prefill_70b_v8m2_b2048", 8192, 8192, 8, 2, -1, 2048),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    v, m, g = rng.choice(FORMATS)
    unit = max(v, g)
    kind = rng.choice(["linear", "linear", "linear", "block", "grouped"])
    if kind == "block":
        hidden = 128 * _log(rng, 8, 64)
        kv = hidden // rng.choice([1, 4, 8])
        inter = unit * max(1, int(hidden * rng.uniform(2.5, 4.0)) // unit)
        return {"kind": kind, "hidden": hidden, "kv": kv, "inter": inter, "v": v, "m": m, "g": g, "B": _log(rng, 1, 32)}
    K = unit * max(1, _log(rng, 512, 28672) // unit)
    N = _log(rng, 512, 28672)
    if kind == "grouped":
        N2 = max(64, N // rng.choice([1, 4, 8]))
        return {"kind": kind, "K": K, "N": N, "N2": N2, "v": v, "m": m, "g": g, "B": _log(rng, 1, 32)}
    B = rng.choice([1, _log(rng, 1, 32), _log(rng, 2, 2048)])
    B = max(1, min(B, 2048 * 8192 * 8192 // (4 * N * K)))          # within the cost of the largest listed case
    return {"kind": kind, "K": K, "N": N, "v": v, "m": m, "g": g, "B": B, "y_fp32": rng.random() < 0.25}


def _calls(case):
    """The calls of a pass: (K, heights of the layers that share one activation matrix)."""
    if case["kind"] == "block":
        h, kv, i = case["hidden"], case["kv"], case["inter"]
        return [(h, [h, kv, kv]), (h, [h]), (h, [i, i]), (i, [h])]
    if case["kind"] == "grouped":
        return [(case["K"], [case["N"], case["N2"], case["N2"]])]
    return [(case["K"], [case["N"]])]


def _tensors(case, seed):
    """Per call: the activations and, per layer, canonical codes, codebooks and scales; from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v, m, g, B = case["v"], case["m"], case["g"], case["B"]
    out = []
    for K, heights in _calls(case):
        x = torch.randn(B, K, generator=gen, device="cuda").half()
        layers = []
        for N in heights:
            codes = torch.randint(0, 256, (m, N, K // v), generator=gen, device="cuda", dtype=torch.uint8)
            books = (torch.randn(m, 256, v, generator=gen, device="cuda") * 0.02).half()
            shape = (N,) if g < 0 else (N, K // g)
            scales = (torch.rand(shape, generator=gen, device="cuda") + 0.5).half()
            layers.append((N, codes, books, scales))
        out.append((K, x, layers))
    return out


def prepare(case, seed):
    v, m, g, B = case["v"], case["m"], case["g"], case["B"]
    y_fp32 = case.get("y_fp32", False)
    stream = torch.cuda.current_stream().cuda_stream
    calls, ys, ws_bytes = [], [], 0
    for K, x, layers in _tensors(case, seed):
        members = []
        for N, codes, books, scales in layers:
            desc = cg.Desc.make(B, K, N, v, m, y_fp32=y_fp32, g=g)
            packed = torch.empty(cg.codegemm_packed_codes_bytes(desc), dtype=torch.uint8, device="cuda")
            cg.codegemm_pack_codes(desc, None, codes, packed, stream)
            if g > 0:
                ps = torch.empty(cg.codegemm_packed_scales_bytes(desc), dtype=torch.uint8, device="cuda")
                cg.codegemm_pack_scales(desc, scales, ps, stream)
                scales = ps
            y = torch.empty(B, N, dtype=torch.float32 if y_fp32 else torch.float16, device="cuda")
            members.append((N, packed, books, scales, y))
            ys.append(y)
        heights = [mb[0] for mb in members]
        desc = cg.Desc.make(B, K, sum(heights), v, m, y_fp32=y_fp32, g=g)
        plan = cg.codegemm_default_plan(desc)
        if len(members) > 1:
            ws_bytes = max(ws_bytes, cg.codegemm_grouped_workspace_bytes(desc, plan, heights))
        else:
            ws_bytes = max(ws_bytes, cg.codegemm_workspace_bytes(desc, plan))
        calls.append((desc, plan, x, members))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    cg.codegemm_workspace_init(ws, ws_bytes, stream)
    state = {"calls": calls, "ws": ws, "ws_bytes": ws_bytes, "ys": ys, "graph": None}
    if case["kind"] == "block":
        torch.cuda.synchronize()
        _issue(state)                                               # once eagerly, as a program warms up before it captures
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            _issue(state)
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = graph
    return state


def _issue(state):
    stream = torch.cuda.current_stream().cuda_stream
    ws, ws_bytes = state["ws"], state["ws_bytes"]
    for desc, plan, x, members in state["calls"]:
        if len(members) > 1:
            cg.codegemm_gemm_grouped(desc, plan, x, members, ws, ws_bytes, stream)
        else:
            _, packed, books, scales, y = members[0]
            cg.codegemm_gemm(desc, plan, x, packed, books, scales, y, ws, ws_bytes, stream)


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _issue(state)
    return state["ys"]


def work(case):
    v, m, g, B = case["v"], case["m"], case["g"], case["B"]
    nbytes = flops = 0
    for K, heights in _calls(case):
        nbytes += 2 * B * K
        for N in heights:
            nbytes += m * N * (K // v) + m * 256 * v * 2 + (2 * N if g < 0 else 2 * N * (K // g))
            nbytes += B * N * (4 if case.get("y_fp32", False) else 2)
            flops += 2 * B * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured against exact(): fp16 output 2.0e-4 to 2.2e-4 (the rounding of the result; one unit in the last place
    # of a value is 1e-3 of it), fp32 output 1.3e-7 to 1.4e-7 (fp32 sums of exact products over K).
    return {"rel": 1e-6, "max": 4e-5} if case.get("y_fp32", False) else {"rel": 9e-4, "max": 9e-3}


def exact(case, seed):
    """Dequantize and multiply in float64, some thousand rows of W at a time."""
    v, m, g = case["v"], case["m"], case["g"]
    out = []
    for K, x, layers in _tensors(case, seed):
        xd = x.double()
        for N, codes, books, scales in layers:
            parts = []
            for n0 in range(0, N, 4096):
                c = codes[:, n0:n0 + 4096].long()
                s = scales[n0:n0 + 4096].double()
                W = sum(books[i].double()[c[i]] for i in range(m)).reshape(c.shape[1], K)
                W *= s[:, None] if g < 0 else s.repeat_interleave(g, dim=1)
                parts.append(xd @ W.t())
            out.append(torch.cat(parts, dim=1))
    return out
