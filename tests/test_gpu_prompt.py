"""GPU parity of calls with many batch rows under default plans: the prompt kernel (fp16 output, enough workgroups) and the
centroid kernel's tiles (fp32 output, or fewer): formats, ragged N, K and batch against the CPU oracle, exact on integer
cases, non-finite rows kept apart."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

cg = pytest.importorskip("paper_2512_17970_amd")
from gpu_util import DeviceLayer, check_against_oracle, exact_on_gpu  # noqa: E402


def batch_for(v, m, g, N, extra):
    """A batch whose tiles of 64 (or 32) rows give at least 128 workgroups of 1024 rows, the last tile ragged."""
    tile = 32 if g > 0 or m >= 3 or (v == 4 and m == 2) else 64
    return tile * -(-128 // -(-N // 1024)) - tile + extra


@pytest.mark.parametrize("N,extra", [(1031, 1), (2048, 33), (3000, 32)])
@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (8, 1, -1), (4, 1, -1), (8, 3, -1), (8, 4, -1), (4, 2, -1), (8, 2, 128), (8, 1, 512), (4, 1, 128), (4, 2, 256), (8, 2, 32), (8, 1, 64), (4, 1, 32), (8, 3, 64), (4, 2, 64)])
def test_formats(v, m, g, N, extra):
    """K of one to three units with an odd number of steps or a ragged last one; N that 8, 128 or 1024 does not divide
    (scalar and vector stores of y); fp16 output through the prompt kernel, fp32 output through tiles."""
    for units, fp32 in ((1, True), (1, False), (3, False)):
        K = max(g, 32 * v) * units + (g if g > 0 else 5 * v)
        case = synth.custom_case(K, N, v, m, batch_for(v, m, g, N, extra), seed=3600 + N + units, g=g)
        print(f"[prompt] {case.name}", flush=True)
        inp = synth.generate(case)
        y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        layer = DeviceLayer(inp, y_fp32=fp32)
        assert layer.plan.centroid_rows
        y = layer.gemm()
        torch.cuda.synchronize()
        rel = check_against_oracle(y.cpu().numpy(), y_ref, T, case.name)
        assert rel < (5e-6 if fp32 else 6e-4), rel


def test_integer_case_is_exact_and_rows_are_independent():
    v, K, N, B, row = 8, 1024, 1100, 64 * 63 + 7, 77
    rng = np.random.default_rng(37)
    i = np.arange(256)[:, None]
    inp = synth.generate(synth.custom_case(K, N, v, 2, B, seed=4))
    bits = (i >> np.arange(v)[None, :]) & 1
    inp.codebooks = np.stack([np.where(bits, 1.0, -1.0), np.where(bits, 2.0, 0.0)]).astype(np.float16)
    inp.x = rng.integers(-8, 9, (B, K)).astype(np.float16)
    inp.scales = np.ones(N, np.float16)
    y_ref, _ = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
    y = {}
    for fp32 in (True, False):
        y[fp32] = DeviceLayer(inp, y_fp32=fp32).gemm()
        torch.cuda.synchronize()
        assert np.array_equal(y[fp32].cpu().numpy(), y_ref.astype(np.float32 if fp32 else np.float16))
    inp.x = inp.x.copy()
    inp.x[row, 3] = np.nan
    inp.x[row, 200] = np.inf
    for fp32 in (True, False):
        z = DeviceLayer(inp, y_fp32=fp32).gemm()
        torch.cuda.synchronize()
        others = torch.arange(B, device=z.device) != row
        assert torch.equal(z[others], y[fp32][others])
        assert not bool(torch.isfinite(z[row]).any().item())


@pytest.mark.parametrize("steps", [20, 21, 64, 65])
@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (4, 1, -1), (4, 2, -1), (8, 3, -1), (8, 2, 32), (8, 1, 128), (4, 1, 128)])
def test_long_k(v, m, g, steps):
    """Many turns of the double-buffered loop, odd and even, against float64: fp16 output (its rounding: 2.1e-4) and fp32
    output through tiles (two levels of short sums: below 1.3e-7 in these formats, 2e-7 the bound of its other tests)."""
    K, N = 128 * steps, 1500
    case = synth.custom_case(K, N, v, m, batch_for(v, m, g, N, 5), seed=3650 + steps, g=g)
    print(f"[prompt] {case.name}", flush=True)
    inp = synth.generate(case)
    for fp32, bound in ((False, 3e-4), (True, 2e-7)):
        layer = DeviceLayer(inp, y_fp32=fp32)
        ref = exact_on_gpu(layer, inp)
        err = ((layer.gemm().double() - ref).norm() / ref.norm()).item()
        assert err < bound, (fp32, err)


@pytest.mark.parametrize("B", [33, 64, 96, 200])
def test_batches_between_a_launch_and_a_prompt(B):
    """More than 32 rows but too few workgroups for the prompt kernel: tiles of the centroid kernel along the grid."""
    for v, m, g in ((8, 2, -1), (4, 1, 128)):
        inp = synth.generate(synth.custom_case(2048, 515, v, m, B, seed=3700, g=g))
        y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        y = DeviceLayer(inp).gemm()
        torch.cuda.synchronize()
        check_against_oracle(y.cpu().numpy(), y_ref, T, inp.case.name)


def test_fp16_output_rounds_the_fp32_product():
    """y is the fp32 product of sum and scale, rounded to fp16, as every other kernel stores it: rounding the exact
    product at once differs where fp32 rounding makes a tie, about once in 2^13 outputs."""
    K, N, B = 64, 1100, 64 * 64
    inp = synth.generate(synth.custom_case(K, N, 8, 1, B, seed=5))
    inp.x = inp.x.copy()
    inp.x[:, 1:] = 0                                    # a sum is one product of two fp16 values, exact in fp32
    y = DeviceLayer(inp).gemm()
    torch.cuda.synchronize()
    acc = inp.x[:, :1].astype(np.float32) * inp.codebooks[0, inp.codes[0, :, 0], 0].astype(np.float32)
    want = (acc * inp.scales.astype(np.float32)).astype(np.float16)
    assert np.array_equal(y.cpu().numpy(), want)


@pytest.mark.parametrize("g", [32, 64, 128, 512])
@pytest.mark.parametrize("N,extra", [(1024, 0), (1025, 1), (1028, 17), (1156, 31), (1502, 16), (4093, 2)])
def test_half_octets(N, extra, g):
    """v = 4, one codebook, group scales: two wavefronts share a granule, each with 4 rows of every octet and 64 batch rows.  Heights that end
    in either half, at 4 and at 8 rows, within a workgroup's first granule or its last; odd numbers of steps and sub-vectors."""
    for K in (max(g, 128), max(g, 128) * 3, 1024 + g):
        case = synth.custom_case(K, N, 4, 1, batch_for(4, 1, g, N, extra), seed=3700 + N + K, g=g)
        print(f"[prompt] {case.name}", flush=True)
        inp = synth.generate(case)
        y_ref, T = oracle.gemm(inp.x, inp.codes, inp.codebooks, inp.scales)
        y = DeviceLayer(inp).gemm()
        torch.cuda.synchronize()
        assert check_against_oracle(y.cpu().numpy(), y_ref, T, case.name) < 6e-4


@pytest.mark.parametrize("g", [32, 64, 128, 512])
@pytest.mark.parametrize("N,B", [(28672, 257), (27001, 288), (3004, 2713)])
def test_whole_octets(N, B, g):
    """The same format where half octets would take one more round of workgroups: 1024 rows and 32 batch rows each.  Odd numbers of steps and
    sub-vectors, ragged last workgroups of rows and of batch rows."""
    K = max(g, 128) + g
    case = synth.custom_case(K, N, 4, 1, B, seed=3800 + K, g=g)
    print(f"[prompt] {case.name}", flush=True)
    inp = synth.generate(case)
    layer = DeviceLayer(inp)
    ref = exact_on_gpu(layer, inp)
    y = layer.gemm().double()
    torch.cuda.synchronize()
    assert ((y - ref).norm() / ref.norm()).item() < 3e-4               # the rounding of the output: 2.1e-4
    assert ((y - ref).abs().max() / ref.square().mean().sqrt()).item() < 5e-3    # half a unit in the last place at 8 times the root mean square: 3.9e-3
