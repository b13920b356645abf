"""GPU parity of the centroid kernel (plans with centroid_rows != 0): every block height, batch tile, format and
K split against the CPU oracle at the acceptance bar, bit for bit on integer cases, and as a member of a group."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

cg = pytest.importorskip("paper_2512_17970_amd")
from gpu_util import DeviceLayer, Guarded, check_against_oracle, dev, exact_on_gpu, stream  # noqa: E402


def least_rows(B, v=8, m=2, g=-1, fp32=False):
    if v == 16:
        return 32 if B <= 4 else 64 if B <= 8 else 128
    if not fp32 and (v, m) in ((8, 1), (8, 2), (4, 1)):                 # the staged kernel's
        return 32
    return 32 if B <= 8 or m == 1 or (g < 0 and not fp32) else 64 if g < 0 or (g >= 128 and not fp32) else 128


def plan_of(case, rows, splits):
    p = cg.codegemm_default_plan(cg.Desc.make(case.B, case.K, case.N, case.v, case.m, g=case.g))
    p.centroid_rows, p.centroid_splits = rows, splits
    p.k_splits = max(p.k_splits, splits)                                # which bounds them
    return p


def run(case, rows, splits, y_fp32=False):
    print(f"[centroid] {case.name} rows={rows} splits={splits}", flush=True)
    inp = synth.generate(case)
    y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
    layer = DeviceLayer(inp, plan=plan_of(case, rows, splits), y_fp32=y_fp32)
    first = layer.gemm().clone()
    again = layer.gemm()                                                # on the workspace the first call left
    torch.cuda.synchronize()
    assert torch.equal(first, again)
    rel = check_against_oracle(first.cpu().numpy(), y_ref, T, f"{case.name} rows={rows} splits={splits}")
    # fp32 output: fp32 sums of K m / v exact products, in order 1e-7 apart; fp16 output: its rounding, 2.8e-4
    assert rel < (5e-6 if y_fp32 else 6e-4), rel
    # counters and pair words are all zero again
    assert not bool(layer.ws[:65536 + (2 << 20)].any().item())


FORMATS = [(8, 2, -1), (8, 1, -1), (4, 1, -1), (8, 3, -1), (8, 4, -1), (4, 2, -1), (16, 1, -1), (16, 2, -1), (16, 3, -1), (16, 4, -1),
           (8, 2, 128), (8, 1, 256), (4, 1, 128), (8, 3, 1024), (4, 2, 512), (8, 4, 128), (16, 2, 256), (16, 3, 512), (16, 4, 1024),
           (8, 2, 64), (8, 2, 32), (8, 1, 32), (8, 3, 64), (8, 4, 32), (4, 1, 64), (4, 1, 32), (4, 2, 32), (16, 1, 128), (16, 2, 64), (16, 4, 64)]


@pytest.mark.parametrize("B", [1, 2, 4, 5, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("v,m,g", FORMATS)
def test_formats_and_batches(v, m, g, B):
    """Every batch tile at its edges; ragged N (not a multiple of 8, 32 or 128), K with a ragged last unit where the
    scales allow one (an odd number of sub-vectors for v = 4), more K ranges than a wavefront's share of steps."""
    unit = max(g, 32 * v)
    K = unit * 5 + (g if g > 0 else 7 * v)
    for N, splits, fp32 in ((301, 1, True), (130, 3, False), (33, 1000, True)):
        run(synth.custom_case(K, N, v, m, B, seed=3000 + N + B, g=g), 128, splits, fp32)


@pytest.mark.parametrize("rows", [32, 64, 128])
@pytest.mark.parametrize("splits", [1, 2, 4, 5])
@pytest.mark.parametrize("B", [1, 3, 7, 13, 21, 40])
@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (8, 1, -1), (4, 1, 128), (4, 2, -1), (16, 4, -1), (8, 3, 128), (8, 4, -1), (8, 2, 32), (8, 1, 64), (4, 1, 32)])
def test_block_heights(v, m, g, B, splits, rows):
    """Blocks of 32 and 64 rows (the batches that have them), ragged at either end of a granule; pairwise words and
    tickets between the K ranges; both output types (fp32 output has kernels of its own)."""
    if rows < least_rows(B, v, m, g):
        pytest.skip("block height not offered for this batch")
    for fp32 in (False, True):
        if rows < least_rows(B, v, m, g, fp32):
            continue
        for N in (rows, rows + 1, 1000):
            run(synth.custom_case(max(g, 32 * v) * 6, N, v, m, B, seed=3100 + N, g=g), rows, splits, fp32)


@pytest.mark.parametrize("B,rows", [(1, 32), (1, 128), (2, 32), (2, 64), (3, 128), (6, 32), (6, 64), (8, 128), (12, 32), (12, 64), (16, 128), (40, 128)])
@pytest.mark.parametrize("v,m,g", [(4, 1, -1), (8, 1, -1), (16, 1, -1), (8, 2, -1), (8, 3, -1), (4, 2, 64), (8, 1, 64), (8, 2, 128), (8, 3, 32), (16, 2, 64)])
def test_fp32_sums_at_every_length_of_a_slice(v, m, g, B, rows):
    """fp32 output: chains, sums and totals with slices of K that end at every place of the load ring and of the moves
    from sums to totals: 0, 1, 2 .. 10 steps per wavefront, 40 and more, an odd number of sub-vectors.  A sum of n
    additions rounded to 2^-24 has an error of about 0.25e-7 sqrt(n / 2), two levels of at most 12 and 10 of them after
    0.6e-7 for a chain 0.9e-7, the tree over slices, lanes and ranges below 1e-7 more: 2e-7, and half as much again
    for a row of few outputs."""
    if rows < least_rows(B, v, m, g, True):
        pytest.skip("block height not offered for this batch")
    step = 16 * v if v > 4 else 128                                     # elements of K
    unit = max(g, v)
    for steps in (1, 7, 8, 12, 17, 25, 32, 42, 50, 58, 66, 83, 333):
        K = -(-steps * step // unit) * unit - (unit if g > 0 or steps > 1 else 0) * (steps % 2)
        case = synth.custom_case(max(K, unit), 70, v, m, B, seed=3150 + steps, g=g)
        print(f"[slices] {case.name} rows={rows}", flush=True)
        inp = synth.generate(case)
        y_ref, _ = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        y = DeviceLayer(inp, plan=plan_of(case, rows, 1), y_fp32=True).gemm()
        torch.cuda.synchronize()
        err = np.linalg.norm(y.cpu().numpy() - y_ref) / np.linalg.norm(y_ref)
        assert err < 3e-7, (case.name, err)


@pytest.mark.parametrize("K,N", [(8, 1), (256, 31), (8 * 33, 128)])
@pytest.mark.parametrize("B", [1, 4, 6, 12, 20])
def test_fewer_steps_than_wavefronts(K, N, B):
    run(synth.custom_case(K, N, 8, 2, B, seed=3200), 128, 1, True)


@pytest.mark.parametrize("B,rows", [(5, 32), (8, 64), (9, 32), (16, 64), (16, 32), (17, 64), (32, 32), (37, 64)])
@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (8, 1, -1), (4, 1, -1), (8, 2, 128), (8, 1, 256), (4, 1, 128), (8, 2, 32), (8, 2, 64), (8, 1, 32), (8, 1, 64), (4, 1, 32), (4, 1, 64)])
def test_low_staged_blocks_at_every_length_of_a_slice(v, m, g, B, rows):
    """fp16 output, blocks of 32 and 64 rows from 5 batch rows on: slices of no stage, one, two, three and many, stages that reach past
    the end of K, heights that end in the first and the last octet of a block and of a granule.  The error is the rounding of the output (run)."""
    unit = max(g, v)
    for elements in (unit, 64, 8 * 128, 8 * 128 + 64, 9 * 128, 17 * 128 + 32, 24 * 128, 41 * 128 + 96, 8192):
        K = max(unit, elements // unit * unit)
        for N in (rows - 7, 128 + rows + 1):
            run(synth.custom_case(K, N, v, m, B, seed=3220 + N, g=g), rows, 1 + (K > 4000))


@pytest.mark.parametrize("B", [1, 4, 8, 16, 32])
def test_integer_cases_are_exact(B):
    """+-1 and 0/2 codebooks with small integer activations: every sum is an integer that fp32 holds, in any order."""
    v, K, N = 8, 4096, 700
    rng = np.random.default_rng(31)
    i = np.arange(256)[:, None]
    inp = synth.generate(synth.custom_case(K, N, v, 2, B, seed=3))
    bits = (i >> np.arange(v)[None, :]) & 1
    inp.codebooks = np.stack([np.where(bits, 1.0, -1.0), np.where(bits, 2.0, 0.0)]).astype(np.float16)
    inp.x = rng.integers(-8, 9, (B, K)).astype(np.float16)
    inp.scales = np.ones(N, np.float16)
    y_ref, _ = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
    for rows, splits in ((128, 1), (128, 3), (least_rows(B, fp32=True), 2)):
        y = DeviceLayer(inp, plan=plan_of(inp.case, rows, splits), y_fp32=True).gemm()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref), (rows, splits)


@pytest.mark.parametrize("v,m,g,B,rows", [(8, 2, -1, 3, 128), (8, 2, -1, 7, 64), (8, 3, -1, 40, 128), (4, 1, -1, 64, 128), (16, 2, -1, 12, 128), (8, 2, 512, 20, 128)])
def test_fp32_output_keeps_chains_of_sums_short(v, m, g, B, rows):
    """A chain of n roundings to 2^-24 ends with a relative error of 2^-24 sqrt(n / 6) (uniform, partial sums growing as
    sqrt): 2e-7 for n = 64.  With all of a wavefront's MFMAs on one accumulator (K m / 256, here 224 to 336 over 32
    products each, which round more than once) 40 rows of this K show 3.8e-7 to 4.7e-7.  With group scales the chains have
    a sum per round (K / 256: 56), so half of the K."""
    case = synth.custom_case(28672 if g < 0 else 14336, 256, v, m, B, seed=3250, g=g)
    inp = synth.generate(case)
    y_ref, _ = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
    y = DeviceLayer(inp, plan=plan_of(case, rows, 1), y_fp32=True).gemm()
    torch.cuda.synchronize()
    err = np.linalg.norm(y.cpu().numpy() - y_ref) / np.linalg.norm(y_ref)
    assert err < 2e-7, err


@pytest.mark.parametrize("B,row", [(3, 1), (6, 4), (13, 0), (20, 19), (70, 33)])
def test_non_finite_activations_stay_in_their_row(B, row):
    """The batch rows share instructions (and, up to 8 rows, result tiles whose other elements are discarded): an
    infinity or NaN in one row of x reaches that row of y alone.  At every block height: 64 and 32 rows are staged from 5 batch rows on, with a row
    of zeros beside up to 8."""
    for rows, g in ((128, -1), (64, -1), (32, -1), (64, 32), (32, 128)):
        case = synth.custom_case(8 * 32 * 4, 300, 8, 2, B, seed=3300, g=g)
        inp = synth.generate(case)
        clean = DeviceLayer(inp, plan=plan_of(case, rows, 1)).gemm().clone()
        inp.x = inp.x.copy()
        inp.x[row, ::97] = np.inf
        inp.x[row, 5] = np.nan
        y = DeviceLayer(inp, plan=plan_of(case, rows, 1)).gemm()
        torch.cuda.synchronize()
        others = [b for b in range(B) if b != row]
        assert torch.equal(y[others], clean[others]), (rows, g)
        assert not bool(torch.isfinite(y[row]).any().item()), (rows, g)


@pytest.mark.parametrize("B,rows,splits,g", [(1, 32, 1, -1), (1, 64, 2, 128), (4, 32, 3, -1), (8, 64, 4, -1), (6, 32, 1, 128),
                                             (16, 128, 2, 128), (16, 32, 2, -1), (3, 32, 1, 32), (11, 128, 2, 64), (13, 64, 1, 128), (32, 128, 5, -1), (32, 64, 2, -1),
                                             (9, 32, 2, 32), (16, 64, 4, 64), (32, 32, 3, 32), (20, 64, 2, 32), (7, 32, 4, 64)])
def test_grouped_members_equal_their_single_calls(B, rows, splits, g):
    K, Ns = 2048, [300, 130, 65]
    desc = cg.Desc.make(B, K, sum(Ns), 8, 2, g=g)
    plan = cg.codegemm_default_plan(desc)
    plan.centroid_rows, plan.centroid_splits = rows, splits
    plan.k_splits = max(plan.k_splits, splits)
    inps = [synth.generate(synth.custom_case(K, n, 8, 2, B, seed=3400 + k, g=g)) for k, n in enumerate(Ns)]
    layers = []
    for inp in inps:
        inp.x = inps[0].x
        layers.append(DeviceLayer(inp, plan=plan))
    ws_bytes = cg.codegemm_grouped_workspace_bytes(desc, plan, Ns)
    ws = Guarded(ws_bytes)
    cg.codegemm_workspace_init(ws.t, ws_bytes, stream())
    ys = [layer.new_y() for layer in layers]
    members = [(n, l.packed, l.codebooks, l.gemm_scales, y) for n, l, y in zip(Ns, layers, ys)]
    for _ in range(2):
        cg.codegemm_gemm_grouped(desc, plan, layers[0].x, members, ws.t, ws_bytes, stream())
        torch.cuda.synchronize()
        assert ws.intact()
        for layer, y, inp in zip(layers, ys, inps):
            layer.check_guards("grouped launch")
            y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
            check_against_oracle(y.cpu().numpy(), y_ref, T, "grouped member")
            alone = layer.gemm()
            torch.cuda.synchronize()
            assert torch.equal(alone, y)


@pytest.mark.parametrize("B0", [1, 3, 12, 200])
@pytest.mark.parametrize("v,m,g0", [(8, 2, 128), (8, 2, -1), (8, 1, 32), (4, 1, 128), (8, 3, -1), (16, 2, -1), (4, 2, -1)])
def test_default_plans_at_other_batches(v, m, g0, B0):
    """The default plan of one batch, kept for other batches, output types and groups of the same layer: blocks that are
    raised from 32 rows to what those need, formats that fall back to the Psumbook fields, batches above one launch."""
    K, N = 32 * v * 5, 4100 if B0 == 1 else 700
    plan = cg.codegemm_default_plan(cg.Desc.make(B0, K, N, v, m, g=g0))
    if not plan.centroid_rows:
        pytest.skip("the Psumbook kernels' plan")
    for B, g, fp32 in ((1, -1, True), (4, g0, True), (9, g0, False), (16, 4 * v, False), (20, -1, True), (33, 8 * v, True), (70, 2 * v, False), (5, v, True), (150, g0, False)):
        case = synth.custom_case(K, N, v, m, B, seed=3450 + B, g=g)
        print(f"[kept plan] {case.name} fp32={fp32} {plan}", flush=True)
        inp = synth.generate(case)
        y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        y = DeviceLayer(inp, plan=plan, y_fp32=fp32).gemm()
        torch.cuda.synchronize()
        rel = check_against_oracle(y.cpu().numpy(), y_ref, T, case.name)
        assert rel < (5e-6 if fp32 else 6e-4), rel


def test_fp16_psumbook_of_a_default_plan():
    """psum_dtype = 1 on a default plan that has centroid_rows: the fp16 Psumbook, bit for bit that of the same plan
    without them, and not the centroid kernel's result."""
    case = synth.custom_case(1024, 4100, 8, 2, 1, seed=3470)
    inp = synth.generate(case)
    plans = [cg.codegemm_default_plan(cg.Desc.make(1, case.K, case.N, 8, 2)) for _ in range(3)]
    assert plans[0].centroid_rows and plans[0].batch_group == 1
    plans[0].psum_dtype = plans[1].psum_dtype = cg.binding.PSUM_FP16
    plans[1].centroid_rows = plans[1].centroid_splits = 0
    ys = []
    for plan in plans:
        ys.append(DeviceLayer(inp, plan=plan, y_fp32=True).gemm())
        torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1]) and not torch.equal(ys[0], ys[2])


def test_replays_from_a_hip_graph():
    """Captured calls give the eager bits on every replay, with eager calls on the same workspace in between."""
    layers = [DeviceLayer(synth.generate(synth.custom_case(K, N, 8, 2, B, seed=3500 + B)), plan=None)
              for K, N, B in ((4096, 1000, 4), (2048, 700, 16), (1024, 4200, 1))]
    for rows, splits, B, g in ((32, 2, 6, -1), (64, 4, 16, 32), (32, 3, 24, 64), (64, 1, 12, 128)):                   # low staged blocks
        case = synth.custom_case(4096, 300, 8, 2, B, seed=3510 + B, g=g)
        layers.append(DeviceLayer(synth.generate(case), plan=plan_of(case, rows, splits)))
    eager = [l.gemm().clone() for l in layers]
    outs = [torch.empty_like(e) for e in eager]
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        for l, y in zip(layers, outs):
            l.gemm(y, check=False)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for y in outs:
            y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for l, y, e in zip(layers, outs, eager):
            assert torch.equal(y, e)
            assert torch.equal(l.gemm(), e)


@pytest.mark.parametrize("v,m,g,B,K,N", [
    (8, 2, -1, 2, 1024, 8192), (8, 4, -1, 2, 1024, 8192), (8, 3, 64, 3, 1024, 8192), (8, 2, 32, 2, 512, 8192), (8, 1, -1, 1, 5120, 16000),
    (8, 1, 128, 2, 28672, 5000), (8, 2, -1, 16, 768, 4096), (4, 2, -1, 12, 512, 4096), (8, 4, -1, 64, 27648, 811), (16, 1, -1, 64, 1024, 1000),
    (16, 2, -1, 200, 26624, 1190), (8, 2, 64, 100, 1024, 1500), (8, 3, 64, 200, 2048, 700), (4, 1, 32, 500, 28672, 700),
    (8, 1, 128, 512, 8192, 8192), (8, 2, 32, 512, 4096, 8192), (4, 1, 128, 1024, 4096, 4096), (8, 1, -1, 600, 14336, 8192), (4, 2, -1, 512, 1536, 8192)])
def test_fp32_output_is_no_further_from_64_bits_than_the_psumbook_kernels(v, m, g, B, K, N):
    """The default plan against the same plan without centroid_rows.  Each error is a root mean square over B N >= 16384
    outputs, so known to 1 / sqrt(2 B N) < 0.6 %: 3 % above is more than three standard deviations of their ratio."""
    case = synth.custom_case(K, N, v, m, B, seed=3260 + B, g=g)
    inp = synth.generate(case)
    layer = DeviceLayer(inp, y_fp32=True)
    ref = exact_on_gpu(layer, inp)
    err = lambda y: ((y.double() - ref).norm() / ref.norm()).item()
    now = err(layer.gemm())
    print(f"[fp32 error] {case.name} {layer.plan} {now:.3e}", flush=True)
    layer.plan.centroid_rows = layer.plan.centroid_splits = 0
    then = err(layer.gemm())
    assert now <= 1.03 * then, (now, then)


@pytest.mark.parametrize("v,m,g,B", [(8, 2, -1, 5), (8, 2, -1, 16), (8, 2, -1, 17), (8, 2, -1, 33), (4, 1, -1, 7), (4, 1, -1, 32), (8, 1, -1, 16), (8, 2, 128, 2), (8, 2, 256, 4),
                                     (8, 2, 128, 9), (8, 1, 128, 3), (8, 1, 256, 8), (4, 1, 128, 4), (4, 1, 128, 16), (4, 1, 256, 20),
                                     (8, 2, 32, 9), (8, 2, 32, 20), (8, 2, 64, 6), (4, 1, 32, 7), (4, 1, 32, 16), (4, 1, 64, 20)])
def test_staged_operands(v, m, g, B):
    """128-row blocks, fp16 output: codes and x pass through a ring of stages (8 or 16 chunks of 16 bytes of x) in LDS.  Slices of 0, 1,
    2 .. stages per wavefront, a last stage that the rows of x end inside of (at every number of chunks, half a chunk for v = 4)
    or that lies wholly behind them, K ranges, ragged N.  (Short ones of 2 to 8 rows are the centroid kernel's: up to 8192 elements.)"""
    unit = max(g, v)
    Ks = [v, 32 * v, 3072, 3072 + 64 * v, 8192] + [2048 + c * v for c in (1, 2, 7, 9, 15, 17, 31, 33)]
    for K in sorted({max(unit, K // unit * unit) for K in Ks}):
        case = synth.custom_case(K, 200, v, m, B, seed=3400 + K, g=g)
        for splits in (1, 2, 5):
            run(case, 128, splits)


def test_staged_operands_leave_the_neighbours_of_x_alone():
    """The last row of x is followed by other memory, here NaN: what a stage reads past the end of a row counts for nothing."""
    for v, m, K, B, g in ((8, 2, 1032, 6, -1), (8, 1, 1096, 13, -1), (8, 1, 2120, 13, -1), (8, 1, 8200, 7, -1), (4, 1, 1028, 16, -1), (4, 1, 2052, 5, -1), (8, 2, 2056, 31, -1),
                          (8, 2, 1056, 11, 32), (8, 2, 2112, 8, 64), (4, 1, 1184, 6, 32), (4, 1, 1312, 32, 32), (8, 1, 1120, 8, 32)):
        inp = synth.generate(synth.custom_case(K, 130, v, m, B, seed=3500 + K, g=g))
        y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        for rows in (128, 64, 32):
            layer = DeviceLayer(inp, plan=plan_of(inp.case, rows, 1))
            wide = torch.full((B * K + 4096,), float("nan"), dtype=torch.float16, device="cuda")
            wide[:B * K] = torch.from_numpy(inp.x.reshape(-1)).cuda()
            layer.x = wide[:B * K].view(B, K)
            y = layer.gemm()
            torch.cuda.synchronize()
            check_against_oracle(y.cpu().numpy(), y_ref, T, f"{inp.case.name} rows={rows}")


@pytest.mark.parametrize("v,m,g,B", [(8, 1, -1, 5), (8, 1, -1, 8), (8, 2, -1, 6), (4, 1, -1, 7), (4, 1, 128, 5), (4, 1, 256, 8), (8, 1, -1, 9), (8, 1, -1, 16)])
def test_blocks_of_128_rows_on_either_side_of_the_staged_kernel(v, m, g, B):
    """5 to 16 rows: with a short K operands go through registers, from a K of 1024 to 8192 on through LDS."""
    unit = max(g, v)
    for K in sorted({max(unit, K // unit * unit) for K in (v, 33 * v, 1000, 1030, 2000, 2500, 8000, 8700)}):
        for splits in (1, 3):
            run(synth.custom_case(K, 200, v, m, B, seed=3550 + K, g=g), 128, splits)


@pytest.mark.parametrize("v,m,g,B,least", [(8, 2, 128, 2, 4096), (8, 2, 256, 4, 4096), (8, 1, 128, 3, 3072), (8, 1, 256, 4, 3072), (4, 1, 128, 4, 7168), (4, 1, 256, 2, 7168), (8, 1, -1, 6, 8192)])
def test_staged_operands_of_few_rows(v, m, g, B, least):
    """From the K on that these formats are staged at: odd numbers of steps, slices of unequal length, a last unit that K ends inside of, K ranges."""
    step = max(g, 8 * v)
    for K in (least, least + step, least + 3 * step, least + 13 * step):
        run(synth.custom_case(K, 200, v, m, B, seed=3580 + K, g=g), 128, 1)
    for splits in (2, 3):
        run(synth.custom_case(splits * least + 5 * step, 200, v, m, B, seed=3590 + splits, g=g), 128, splits)
