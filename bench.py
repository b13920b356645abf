#!/usr/bin/env python3
"""Benchmark of the CodeGEMM hot path on one MI355X.

A "step" is one call of codegemm_gemm for each of the four Llama-3-70B linear
layer shapes (8192->8192, 8192->1024, 8192->28672, 28672->8192) at batch 1,
2-bit (v=8, m=2), on synthetic seeded inputs already resident in HBM.  Every
step reads a different copy of the packed codes (the copies of one shape add up
to >= 1 GiB), so the weights come from HBM and not from the last-level cache.

Prints ONE JSON line: the metric is effective HBM bandwidth on compressed bytes
(codes + codebooks + scales + x + y per call, summed over the step, divided by
the step time), with a `roofline` object for the gather kernel and a
`cpu_baseline` object (the CPU oracle timed on this host).  Per-shape detail
(cold and cache-warm us/call, the dequantization comparator, the ratio) goes to
stderr and, with --detail-json FILE, to that file.
"""
from __future__ import annotations

import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0          # MI355X published HBM3E bandwidth
COLD_BYTES = 1 << 30            # rotating working set per shape


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--repeats", type=int, default=7,
                    help="the K timed steps are run this many times; ms_per_step is the median run, min and max go to config")
    ap.add_argument("--workload", default="c3", help="c1..c13 | a single case name from synth.workloads()")
    ap.add_argument("--launch", default="graph", choices=["graph", "direct"],
                    help="graph: the K timed steps are one captured HIP graph (no host launch cost); direct: plain launches")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-detail", action="store_true", help="skip the per-shape cold/warm/dequant table")
    ap.add_argument("--detail-json", default="", help="also write the per-shape detail to this file")
    ap.add_argument("--phases", action="store_true",
                    help="phase table of every shape of the workload from the diagnostic build (in-kernel clock stamps)")
    ap.add_argument("--sweep", action="store_true",
                    help="time every launch plan shape x K-split count for every shape of the workload (cold)")
    ap.add_argument("--psumbook", action="store_true",
                    help="instead of the GEMM: time the stand-alone Psumbook build (vector ALU and MFMA) at batch 1, 8, 32")
    ap.add_argument("--memcpy", action="store_true",
                    help="instead of the GEMM: time the runtime's device-to-device copy at the code sizes of the 70B shapes and at "
                         "1 GiB (reads and writes that many bytes each): what this machine's memory system gives a plain kernel")
    ap.add_argument("--ablate", type=int, default=0,
                    help="time an ablation build of the library instead (libcodegemm_ablate_<mask>.so; outputs are wrong on "
                         "purpose): 2 no gather, 4 no Psumbook build after the first, 8 no exchange between workgroups; "
                         "6, 8 and 14 are built by default")
    ap.add_argument("--plan", default="", help="override plan for every shape: waves,row_words,k_splits[,batch_group[,psum_dtype"
                    "[,build_waves[,centroid_rows,centroid_splits]]]] (psum_dtype 1 = fp16 Psumbook)")
    ap.add_argument("--psum-fp16", action="store_true",
                    help="every shape's default plan with the Psumbook stored as fp16 (batch 1; the group-scale shapes that "
                         "default to 16 wavefronts x 2 row words run with 1 row word)")
    return ap.parse_args()


class Layer:
    """One quantized layer on the GPU with R rotating copies of its packed codes."""

    def __init__(self, cg, torch, synth, case, plan_override, copies_bytes=COLD_BYTES, psum_fp16=False):
        self.cg, self.torch, self.case = cg, torch, case
        inp = synth.generate(case)
        self.inp = inp
        self.desc = cg.Desc.make(case.B, case.K, case.N, case.v, case.m, g=case.g)
        self.plan = plan_override if plan_override is not None else cg.codegemm_default_plan(self.desc)
        if psum_fp16 and plan_override is None:
            p = self.plan
            waves = 16 if p.waves == 14 else p.waves     # the fp16 Psumbook pairs up 8 or 16 wavefronts
            rw = 1 if (case.g > 0 and waves == 16) else min(p.row_words, 2)
            self.plan = cg.Plan.make(waves, rw, p.k_splits, 1, 1)
        dev = lambda a: torch.from_numpy(a).cuda()
        self.x, self.codes = dev(inp.x), dev(inp.codes)
        self.codebooks, self.scales = dev(inp.codebooks), dev(inp.scales)
        self.y = torch.empty((case.B, case.N), dtype=torch.float16, device="cuda")
        nbytes = cg.codegemm_packed_codes_bytes(self.desc, self.plan)
        self.R = max(2, -(-copies_bytes // nbytes))
        self.packed = torch.empty((self.R, nbytes), dtype=torch.uint8, device="cuda")
        s = torch.cuda.current_stream().cuda_stream
        cg.codegemm_pack_codes(self.desc, self.plan, self.codes, self.packed[0], s)
        for r in range(1, self.R):
            self.packed[r].copy_(self.packed[0])
        # group scales travel with the codes: one packed copy per copy of the codes
        self.gemm_scales = [self.scales] * self.R
        if case.g > 0:
            sbytes = cg.codegemm_packed_scales_bytes(self.desc)
            ps = torch.empty((self.R, sbytes), dtype=torch.uint8, device="cuda")
            cg.codegemm_pack_scales(self.desc, self.scales, ps[0], s)
            for r in range(1, self.R):
                ps[r].copy_(ps[0])
            self.gemm_scales = [ps[r] for r in range(self.R)]
        self.ws_bytes = cg.codegemm_workspace_bytes(self.desc, self.plan)
        self.ws = torch.empty(self.ws_bytes, dtype=torch.uint8, device="cuda")
        cg.codegemm_workspace_init(self.ws, self.ws_bytes, s)
        self.bytes = cg.compressed_bytes(case.B, case.K, case.N, case.v, case.m, case.g)
        self.i = 0

    def gemm(self, copy=None):
        r = self.i % self.R if copy is None else copy
        self.i += 1
        self.cg.codegemm_gemm(self.desc, self.plan, self.x, self.packed[r], self.codebooks, self.gemm_scales[r], self.y,
                              self.ws, self.ws_bytes, self.torch.cuda.current_stream().cuda_stream)

    def dequant(self):
        self.cg.codegemm_dequant_gemm(self.desc, self.x, self.codes, self.codebooks, self.scales, self.y,
                                      self.torch.cuda.current_stream().cuda_stream)


def time_region(torch, fn, reps):
    """Device time of `reps` back-to-back calls of fn() between two events on the launch stream (ms)."""
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(reps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1)


def graph_of(torch, fn, reps):
    """Captures `reps` calls of fn() (kernel launches only) into one HIP graph."""
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            for _ in range(reps):
                fn()
    torch.cuda.current_stream().wait_stream(side)
    return g


def per_shape_detail(torch, layers, launch):
    rows = []
    for L in layers:
        row = {"case": L.case.name, "plan": repr(L.plan), "compressed_bytes": L.bytes, "copies": L.R}
        for label, fn in (("cold", lambda: L.gemm()), ("warm", lambda: L.gemm(0))):
            n = 200
            for _ in range(20):
                fn()
            if launch == "graph":
                L.i = 0
                g = graph_of(torch, fn, n)
                ts = [time_region(torch, g.replay, 1) * 1e3 / n for _ in range(5)]
            else:
                ts = [time_region(torch, fn, n) * 1e3 / n for _ in range(5)]
            row[f"us_{label}_min"], row[f"us_{label}_median"] = min(ts), statistics.median(ts)
        dq_n = 20
        for _ in range(3):
            L.dequant()
        ts = [time_region(torch, L.dequant, dq_n) * 1e3 / dq_n for _ in range(3)]
        row["us_dequant_min"] = min(ts)
        row["GBps_cold"] = L.bytes / row["us_cold_min"] * 1e-3
        row["frac_of_peak_cold"] = row["GBps_cold"] / HBM_PEAK_GBPS
        row["GBps_warm"] = L.bytes / row["us_warm_min"] * 1e-3
        row["dequant_over_codegemm"] = row["us_dequant_min"] / row["us_cold_min"]
        rows.append(row)
        log(f"  {row['case']:28s} {row['plan']}: cold {row['us_cold_min']:.2f} us ({row['GBps_cold']:.0f} GB/s, "
            f"{100 * row['frac_of_peak_cold']:.1f}% of peak)  warm {row['us_warm_min']:.2f} us  "
            f"dequant {row['us_dequant_min']:.2f} us ({row['dequant_over_codegemm']:.1f}x)")
    return rows


def group_detail(torch, group, launch, n=100):
    """Cold time of one grouped launch (every call streams other copies of its members' codes)."""
    for _ in range(10):
        group.gemm()
    if launch == "graph":
        group.i = 0
        g = graph_of(torch, group.gemm, n)
        ts = [time_region(torch, g.replay, 1) * 1e3 / n for _ in range(5)]
    else:
        ts = [time_region(torch, group.gemm, n) * 1e3 / n for _ in range(5)]
    nbytes = sum(L.bytes for L, _ in group.members)
    row = {"members": [L.case.name for L, _ in group.members], "plan": repr(group.plan), "compressed_bytes": nbytes,
           "us_cold_min": min(ts), "GBps_cold": nbytes / min(ts) * 1e-3, "frac_of_peak_cold": nbytes / min(ts) * 1e-3 / HBM_PEAK_GBPS}
    log(f"  grouped {'+'.join(str(n_) for n_ in group.Ns)} rows {row['plan']}: cold {row['us_cold_min']:.2f} us "
        f"({row['GBps_cold']:.0f} GB/s, {100 * row['frac_of_peak_cold']:.1f}% of peak)")
    return row


def decoder_block_us(torch, layers, order, launch, blocks=30, runs=5):
    """All linear layers of one decoder block launched back to back on one stream, every launch
    on another copy of its weights: `blocks` blocks per timed run (one HIP graph), median of `runs`."""
    def block():
        for i in order:
            (layers[i] if isinstance(i, int) else i).gemm()

    for _ in range(3):
        block()
    if launch == "graph":
        for L in list(layers) + [i for i in order if not isinstance(i, int)]:
            L.i = 0
        g = graph_of(torch, lambda: [block() for _ in range(blocks)], 1)
        g.replay()
        ts = [time_region(torch, g.replay, 1) for _ in range(runs)]
    else:
        ts = [time_region(torch, block, blocks) for _ in range(runs)]
    return statistics.median(ts) * 1e3 / blocks


class Group:
    """Layers that read the same x (q/k/v, or gate/up) run as one grouped launch; members are
    (layer, copy offset) pairs, so that two members of one shape stream different copies."""

    def __init__(self, cg, torch, members):
        self.cg, self.torch, self.members = cg, torch, members
        first = members[0][0]
        c = first.case
        self.Ns = [L.case.N for L, _ in members]
        self.desc = cg.Desc.make(c.B, c.K, sum(self.Ns), c.v, c.m, g=c.g)
        self.plan = cg.codegemm_default_plan(self.desc)
        self.x = first.x
        self.ys = [torch.empty((c.B, n), dtype=torch.float16, device="cuda") for n in self.Ns]
        self.ws_bytes = cg.codegemm_grouped_workspace_bytes(self.desc, self.plan, self.Ns)
        if self.ws_bytes == 0:
            raise SystemExit(f"no grouped launch for {c.name} under {self.plan}")
        self.ws = torch.empty(self.ws_bytes, dtype=torch.uint8, device="cuda")
        cg.codegemm_workspace_init(self.ws, self.ws_bytes, torch.cuda.current_stream().cuda_stream)
        self.i = 0

    def gemm(self):
        mem = []
        for (L, off), n, y in zip(self.members, self.Ns, self.ys):
            r = (self.i * 2 + off) % L.R
            mem.append((n, L.packed[r], L.codebooks, L.gemm_scales[r], y))
        self.i += 1
        self.cg.codegemm_gemm_grouped(self.desc, self.plan, self.x, mem, self.ws, self.ws_bytes,
                                      self.torch.cuda.current_stream().cuda_stream)


def cpu_baseline(cases, synth, budget_s=12.0):
    """The CPU oracle, as it stands, on this host's cores, on a bounded sample."""
    import oracle
    inputs = [synth.generate(c) for c in cases]
    total_bytes = 0
    total_s = 0.0
    detail = []
    for c, inp in zip(cases, inputs):
        best = float("inf")
        t_start = time.perf_counter()
        reps = 0
        while reps < 3 or (time.perf_counter() - t_start < budget_s / len(cases) and reps < 20):
            t0 = time.perf_counter()
            oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
            best = min(best, time.perf_counter() - t0)
            reps += 1
        nbytes = c.m * c.N * c.J + c.m * 256 * c.v * 2 + 2 * c.N + 2 * c.B * c.K + 2 * c.B * c.N
        total_bytes += nbytes
        total_s += best
        detail.append({"case": c.name, "ms": best * 1e3, "reps": reps})
    cores = oracle.num_threads()
    one_s = 0.0
    oracle.set_num_threads(1)
    try:
        for inp in inputs:
            t0 = time.perf_counter()
            oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
            one_s += time.perf_counter() - t0
    finally:
        oracle.set_num_threads(cores)
    return {"value": total_bytes / total_s * 1e-9, "unit": "GB/s", "cores": cores, "kind": "oracle",
            "sample": "one oracle.gemm call per shape of the step (fp64 dequantize-then-multiply), best of >=3 each",
            "ms_per_step": total_s * 1e3, "detail": detail,
            "one_thread": {"value": total_bytes / one_s * 1e-9, "unit": "GB/s", "cores": 1, "ms_per_step": one_s * 1e3,
                           "sample": "the same calls once each on one thread"}}


def psumbook_bench(torch, cg, synth):
    """Stand-alone Eq. 2 build for the batch-sweep shapes: us per call, vector ALU vs matrix cores."""
    for K in (4096, 14336):
        for B in (1, 8, 32):
            case = synth.custom_case(K, 256, 8, 2, B, seed=3)
            inp = synth.generate(case)
            desc = cg.Desc.make(B, K, 256, 8, 2)
            x = torch.from_numpy(inp.x).cuda()
            cb = torch.from_numpy(inp.codebooks).cuda()
            P = torch.empty((B, 2, K // 8, 256), dtype=torch.float32, device="cuda")
            for use_mfma in (False, True):
                fn = lambda: cg.codegemm_psumbook_build(desc, x, cb, P, use_mfma, torch.cuda.current_stream().cuda_stream)
                for _ in range(5):
                    fn()
                us = min(time_region(torch, fn, 50) * 1e3 / 50 for _ in range(3))
                macs = 2 * 256 * K * B
                log(f"  psumbook_build K={K} B={B} {'mfma' if use_mfma else 'valu'}: {us:.2f} us, "
                    f"{P.numel() * 4 / us * 1e-3:.0f} GB/s written, {2 * macs / us * 1e-6:.2f} TFLOP/s")


def memcpy_report(torch):
    """Device-to-device copies through the runtime's own copy kernel, back to back in one HIP graph, rotating over a
    2 GiB pool so that nothing is served from the caches: us per copy and GB/s counting bytes read + bytes written."""
    pool = torch.empty(2 << 30, dtype=torch.uint8, device="cuda").fill_(1)
    rows = []
    for nbytes in (16777216, 58720256, 1 << 30):
        half = pool.numel() // 2
        slots = max(1, half // nbytes)
        n = 100 if nbytes < (1 << 28) else 4
        state = {"i": 0}

        def copy():
            k = state["i"] % slots
            state["i"] += 1
            pool[half + k * nbytes: half + (k + 1) * nbytes].copy_(pool[k * nbytes:(k + 1) * nbytes])

        for _ in range(3):
            copy()
        g = graph_of(torch, copy, n)
        g.replay()
        us = statistics.median(time_region(torch, g.replay, 1) for _ in range(5)) * 1e3 / n
        row = {"bytes": nbytes, "us_per_copy": us, "GBps_read_plus_write": 2 * nbytes / us * 1e-3}
        log(f"  copy of {nbytes} bytes: {us:.2f} us, {2 * nbytes / us * 1e-3:.0f} GB/s (read + write)")
        # read-only reference: torch's reduction kernel over the same bytes (reads nbytes, writes a scalar)
        words = pool.view(torch.int64)
        out = torch.zeros((), dtype=torch.int64, device="cuda")
        state["i"] = 0

        def reduce():
            k = state["i"] % (2 * slots)
            state["i"] += 1
            torch.sum(words[k * nbytes // 8:(k + 1) * nbytes // 8], dim=0, out=out)

        for _ in range(3):
            reduce()
        us_r = statistics.median(time_region(torch, reduce, n) for _ in range(5)) * 1e3 / n
        row.update({"us_per_read_only_reduction": us_r, "GBps_read_only": nbytes / us_r * 1e-3})
        log(f"  read-only reduction (torch.sum) of {nbytes} bytes: {us_r:.2f} us, {nbytes / us_r * 1e-3:.0f} GB/s")
        rows.append(row)
    # the floor of a launch: the library's fill kernel on 4 bytes, 200 launches per HIP graph
    import paper_2512_17970_amd as cg
    tiny = torch.zeros(64, dtype=torch.uint8, device="cuda")
    launch = lambda: cg.codegemm_workspace_init(tiny, 4, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        launch()
    g = graph_of(torch, launch, 200)
    g.replay()
    us0 = statistics.median(time_region(torch, g.replay, 1) for _ in range(5)) * 1e3 / 200
    log(f"  a 4-byte fill kernel, back to back in a HIP graph: {us0:.2f} us per launch")
    print(json.dumps({"memcpy": rows, "empty_launch_us": us0}))


def phases_report(torch, cg, layers):
    """Where the time of one call goes, per shape: clock stamps of the workgroups (diagnostic build)."""
    from paper_2512_17970_amd import phases
    out = {}
    flush = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")     # 4x the memory-side cache
    for L in layers:
        rows = phases.phase_table(torch, L.desc, L.plan, L.x, L.packed[0], L.codebooks, L.gemm_scales[0], L.y,
                                  L.ws, L.ws_bytes, flush=flush)
        out[L.case.name] = {"plan": repr(L.plan), "phases": rows}
        log(f"{L.case.name}  {L.plan}  ({phases.workgroups(L.desc, L.plan)} workgroups per batch group; cold, one call)")
        log(f"  {'phase':28s} {'workgroups':>10s} {'mean us':>9s} {'min us':>9s} {'max us':>9s}")
        for r in rows:
            log(f"  {r['phase']:28s} {r['workgroups']:10d} {r['mean_us']:9.2f} {r['min_us']:9.2f} {r['max_us']:9.2f}")
    print(json.dumps({"phases": out}))


def sweep_report(torch, cg, synth, cases, launch):
    """Cold time of every offered plan shape of both kinds of kernels and a range of K-split counts, per shape."""
    out = {}
    for case in cases:
        d = cg.Desc.make(case.B, case.K, case.N, case.v, case.m, g=case.g)
        default = cg.codegemm_default_plan(d)
        bg = default.batch_group
        ngr, nkt = -(-case.N // 128), -(-case.J // 32)
        groups = -(-case.B // bg) if bg == 4 else 1
        res = []
        for waves, rw, bw in [(8, 1, 0), (16, 1, 0), (8, 2, 0), (16, 2, 0), (14, 2, 0), (16, 2, 2), (16, 4, 0), (8, 4, 0)]:
            rows = rw * (waves - bw) * (32 if bg == 4 else 16)            # rows of one workgroup
            nblk = -(-ngr * 128 // rows) * groups
            cands = set()
            for target in (128, 192, 224, 256, 384, 512):
                ks = max(1, min(nkt, target // nblk))
                cands.add(-(-nkt // -(-nkt // ks)))
            for ks in sorted(cands):
              for psum in ((0, 1) if bg == 1 else (0,)):                # Psumbook stored as fp32 / fp16
                plan = cg.Plan.make(waves, rw, ks, bg, psum, bw)
                if cg.codegemm_workspace_bytes(d, plan) == 0:
                    continue                                            # plan not offered for this format
                L = Layer(cg, torch, synth, case, plan, copies_bytes=COLD_BYTES // 2)
                call = graph_of(torch, L.gemm, 50).replay if launch == "graph" else (lambda L=L: [L.gemm() for _ in range(50)])
                call(); call()
                us = min(time_region(torch, call, 1) for _ in range(4)) * 1e3 / 50
                res.append({"waves": waves, "row_words": rw, "k_splits": ks, "batch_group": bg, "psum_dtype": "fp16" if psum else "fp32", "build_waves": bw,
                            "workgroups": nblk * ks, "us_cold": us})
                log(f"  {case.name} waves={waves}{'(14+2)' if bw else ''} row_words={rw} k_splits={ks} psum={'fp16' if psum else 'fp32'} workgroups={nblk * ks}: {us:.2f} us")
                del L
                torch.cuda.empty_cache()
        # the centroid kernel: block heights and K ranges (a height is raised where the problem needs a higher one)
        takes = not (case.v == 4 and case.m > 2) and (case.g < 0 or case.g >= (8 if case.v == 4 else 4) * case.v)
        for rows in (32, 64, 128) if takes else ():
            for ks in (1, 2, 3, 4, 6, 8, 16, 32):
                if ks > nkt or -(-case.N // rows) * ks > 1024:
                    continue
                plan = cg.Plan.from_buffer_copy(default)
                plan.centroid_rows, plan.centroid_splits, plan.k_splits = rows, ks, max(ks, default.k_splits)
                L = Layer(cg, torch, synth, case, plan, copies_bytes=COLD_BYTES // 2)
                call = graph_of(torch, L.gemm, 50).replay if launch == "graph" else (lambda L=L: [L.gemm() for _ in range(50)])
                call(); call()
                us = min(time_region(torch, call, 1) for _ in range(4)) * 1e3 / 50
                res.append({"centroid_rows": rows, "centroid_splits": ks, "workgroups": -(-case.N // rows) * ks, "us_cold": us})
                log(f"  {case.name} centroid_rows={rows} centroid_splits={ks} workgroups={-(-case.N // rows) * ks}: {us:.2f} us")
                del L
                torch.cuda.empty_cache()
        res.sort(key=lambda r: r["us_cold"])
        out[case.name] = {"default": repr(default), "plans": res}
        name = lambda r: (f"centroid {r['centroid_rows']},{r['centroid_splits']}" if "centroid_rows" in r else
                          f"{r['waves']},{r['row_words']},{r['k_splits']},{r['psum_dtype']}")
        log(f"BEST {case.name}: " + ", ".join(f"({name(r)}) {r['us_cold']:.2f}" for r in res[:3]) + f"   default {default}")
    print(json.dumps({"sweep": out}))


def kernel_of(plan, batch):
    """Name of the kernel that a layer runs under its plan."""
    if plan.centroid_rows and plan.psum_dtype == 0:
        # staged operands: some formats, from 5 rows on at any block height, 128-row blocks from a K on that depends on format and batch; large batches of many workgroups are prompts
        staged = batch > 4 or (plan.centroid_rows == 128 and batch > 1)
        return "cg::gemm_centroid_kernel" + (" or cg::gemm_staged_kernel" if staged else "") + (" or cg::gemm_prompt_kernel" if batch > 32 else "")
    return "cg::gemm_batch_kernel" if plan.batch_group == 4 else "cg::gemm_kernel"


def read_traffic(key):
    """HBM bytes per launch of this workload (mean over its gemm_kernel launches) from the
    committed rocprofv3 --pmc summary, if it covers the workload."""
    path = os.path.join(ROOT, "profiles", "gemm_kernel_hbm_traffic_pmc.txt")
    try:
        for line in open(path):
            if line.startswith(f"traffic_bytes_per_launch_{key}="):
                return float(line.split("=", 1)[1])
    except OSError:
        pass
    return None


def main():
    args = parse()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU only; --gpus N with N > 1 is not supported "
              "(the path would shard by output rows without any exchange)", file=sys.stderr)
        sys.exit(2)
    import torch
    import synth
    import paper_2512_17970_amd as cg
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the hot path has no CPU fallback", file=sys.stderr)
        sys.exit(3)
    if args.ablate:
        from paper_2512_17970_amd import build as cg_build
        cg.binding.use_library(cg_build.ablate_lib(args.ablate))
        args.no_cpu_baseline = True
    cg.load()
    if args.psumbook:
        psumbook_bench(torch, cg, synth)
        return
    if args.memcpy:
        cg.load()
        memcpy_report(torch)
        return
    wl = synth.workloads()
    key = args.workload.lower()
    if key[:1] == "c" and key[1:].isdigit() and int(key[1:]) in wl:
        cases = wl[int(key[1:])]
    else:
        cases = [synth.find_case(args.workload)]
    plan_override = None
    if args.plan:
        plan_override = cg.Plan.make(*[int(t) for t in args.plan.split(",")])
    log(f"device: {torch.cuda.get_device_name(0)}; workload {key}: {[c.name for c in cases]}")
    if args.sweep:
        sweep_report(torch, cg, synth, cases, args.launch)
        return
    layers = [Layer(cg, torch, synth, c, plan_override, psum_fp16=args.psum_fp16) for c in cases]
    torch.cuda.synchronize()
    if args.ablate:                                     # the ablation builds leave parts of the Psumbook kernel out
        for L in layers:
            L.plan.centroid_rows = L.plan.centroid_splits = 0
    if args.phases:
        phases_report(torch, cg, layers)
        return

    def step():
        for L in layers:
            L.gemm()

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    if args.launch == "graph":
        g = graph_of(torch, step, args.steps)
        g.replay()                      # untimed: first replay uploads the graph
        runs = [time_region(torch, g.replay, 1) for _ in range(max(1, args.repeats))]
    else:
        runs = [time_region(torch, step, args.steps) for _ in range(max(1, args.repeats))]
    ms = statistics.median(runs)        # each run times exactly args.steps steps
    ms_per_step = ms / args.steps
    step_bytes = sum(L.bytes for L in layers)
    launches = len(layers) * args.steps
    value = step_bytes / (ms_per_step * 1e-3) * 1e-9
    us_per_launch = ms * 1e3 / launches
    def operands_of(kernels, layers):
        kinds = ["centroids times x on the matrix cores"] if any("centroid" in k for k in kernels) else []
        if any("centroid" not in k for k in kernels):
            kinds.append("f16 Psumbook" if any(L.plan.psum_dtype for L in layers) else "f32 Psumbook")
        return " or ".join(kinds)

    kernels = sorted({kernel_of(L.plan, L.case.B) for L in layers})
    recorded = kernels == ["cg::gemm_kernel"]              # what the recorded traffic is of
    roofline = {"bound": "hbm", "achieved": value, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                "frac": value / HBM_PEAK_GBPS, "traffic": read_traffic(key) if recorded else None,
                "traffic_source": "profiles/gemm_kernel_hbm_traffic_pmc.txt: separate rocprofv3 --pmc runs of this "
                                  "command (FETCH_SIZE, WRITE_SIZE), not measured in this run" if recorded else
                                  "not recorded for these kernels",
                "kernel": ", ".join(kernels), "avg_launch_us": us_per_launch,
                "algorithmic_bytes_per_launch": step_bytes / len(layers)}
    out = {
        "metric": "effective HBM GB/s on compressed bytes, Llama-3-70B layer shapes, bs=1, 2-bit (us/call in config)",
        "value": value, "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"{key}: " + ", ".join(c.name for c in cases),
                   "calls_per_step": len(layers), "operands": f"f16 x, codebooks, scales; u8 codes; {operands_of(kernels, layers)}, f32 accumulation; f16 y", "us_per_step": ms_per_step * 1e3,
                   "timed_runs": len(runs), "us_per_step_min": min(runs) / args.steps * 1e3,
                   "us_per_step_max": max(runs) / args.steps * 1e3, "launch": args.launch,
                   "cold_copies_bytes_per_shape": COLD_BYTES},
        "roofline": roofline,
    }
    if args.ablate:
        out["ablation"] = {"mask": args.ablate, "note": "diagnostic build with parts of the kernel compiled out; "
                           "outputs are wrong on purpose, the number is a ceiling study, not a result"}
    detail = None
    if not args.no_detail:
        log("per-shape (min of 5 x 200 calls):")
        detail = per_shape_detail(torch, layers, args.launch)
        out["config"]["us_per_call_cold"] = {r["case"]: round(r["us_cold_min"], 3) for r in detail}
        t = [r["us_cold_min"] for r in detail]
        # The shapes that dominate the step's time (here the two 58.7 MB ones, one kernel instantiation): their own
        # roofline, from the cold per-call times just measured (HIP events over graph replays on the launch stream).
        top = max(r["compressed_bytes"] for r in detail)
        dom = [r for r in detail if r["compressed_bytes"] >= 0.9 * top]
        dom_us = sum(r["us_cold_median"] for r in dom) / len(dom)
        dom_bytes = sum(r["compressed_bytes"] for r in dom) / len(dom)
        out["roofline"]["dominant_shapes"] = {
            "cases": [r["case"] for r in dom], "plans": [r["plan"] for r in dom],
            "avg_launch_us": round(dom_us, 3), "algorithmic_bytes_per_launch": dom_bytes,
            "achieved": dom_bytes / dom_us * 1e-3, "frac": dom_bytes / dom_us * 1e-3 / HBM_PEAK_GBPS,
            "note": "median of 5 graph replays of 200 cold calls per shape, HIP events: the time per call includes the "
                    "dispatch gap between consecutive kernels (a few tenths of a microsecond), which the kernel-trace "
                    "durations under profiles/ do not; roofline.frac above is the whole step"}
        if key in ("c2", "c3", "c7", "c8"):
            # the paper's Table 2 quantity: the 7 linears of a decoder block = 2 q/o + 2 k/v + gate + up + down
            out["config"]["decoder_block_sum_us"] = round(2 * t[0] + 2 * t[1] + 2 * t[2] + t[3], 3)
            order = [0, 1, 1, 0, 2, 2, 3]                               # q, k, v, o, gate, up, down
        elif key in ("c9", "c10"):
            out["config"]["decoder_block_sum_us"] = round(sum(t), 3)    # fused QKV + o + fused gate-up + down
            order = [0, 1, 2, 3]
        else:
            order = None
        if order is not None:
            out["config"]["decoder_block_us"] = round(decoder_block_us(torch, layers, order, args.launch), 3)
            log(f"decoder block, {len(order)} linears launched back to back (timed): {out['config']['decoder_block_us']:.2f} us; "
                f"sum of the per-shape times: {out['config']['decoder_block_sum_us']:.2f} us")
            if key in ("c2", "c3", "c7", "c8"):
                # the same seven layers as four launches: q, k and v grouped, o, gate and up grouped, down
                gorder = [Group(cg, torch, [(layers[0], 0), (layers[1], 0), (layers[1], 1)]), 0,
                          Group(cg, torch, [(layers[2], 0), (layers[2], 1)]), 3]
                out["config"]["grouped_launches"] = [group_detail(torch, gr, args.launch) for gr in gorder if not isinstance(gr, int)]
                out["config"]["decoder_block_grouped_us"] = round(decoder_block_us(torch, layers, gorder, args.launch), 3)
                log(f"decoder block with grouped launches (q,k,v | o | gate,up | down): "
                    f"{out['config']['decoder_block_grouped_us']:.2f} us")
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cases, synth)
        log(f"cpu oracle: {out['cpu_baseline']['ms_per_step']:.1f} ms per step on {out['cpu_baseline']['cores']} threads")
    else:
        out["cpu_baseline"] = None
    if detail is not None and args.detail_json:
        with open(args.detail_json, "w") as f:
            json.dump({"summary": out, "per_shape": detail}, f, indent=1)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
