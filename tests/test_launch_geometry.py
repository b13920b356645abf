"""The launch geometry behind a plan, as the library derives it (host code of the built library, no kernel is launched):
members of a group and the same layers alone, and what default plans of few rows run."""
import os
import random
import shutil
import subprocess

import pytest

import paper_2512_17970_amd as cg
from paper_2512_17970_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))

pytestmark = pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no hipcc")


@pytest.fixture(scope="module")
def geometry(tmp_path_factory):
    """A function: problem lines -> per problem (status, members, alone), the latter two lists of dicts."""
    cg.load()                                                      # built if it is not there
    exe = str(tmp_path_factory.mktemp("geometry") / "geometry_lines")
    subprocess.run([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-Wno-unused-result", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(HERE, "host", "geometry_lines.cpp"), "-o", exe, "-L", build.PKG, "-l:" + os.path.basename(build.LIB), "-Wl,-rpath," + build.PKG], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True).stdout.splitlines()
        res = []
        for line in out:
            word, rest = line.split(" ", 1)
            if word == "group":
                res.append((int(rest), [], []))
            else:
                res[-1][1 if word == "member" else 2].append({k: int(v) for k, v in (f.split("=") for f in rest.split())})
        assert len(res) == len(lines)
        return res
    return run


def line(B, K, Ns, v, m, g, fp32=0, plan_batch=None, plan=None):
    tail = [plan_batch or B] if plan is None else [0, *plan]
    return " ".join(str(t) for t in (B, K, v, m, g, fp32, len(Ns), *Ns, *tail))


def same(member, alone):
    """What decides the bits: the kernel, its tiles and how K is cut.  (Two or four ranges meet in the same order by either protocol.)"""
    skip = {"pairs"}
    return {k: x for k, x in member.items() if k not in skip} == {k: x for k, x in alone.items() if k not in skip}


def test_group_members_and_single_calls_run_alike(geometry):
    rng = random.Random(5)
    problems = []
    for B, K, Ns, v, m, g in ((4, 28672, (4096, 4096), 8, 2, 128), (4, 12288, (12288, 1536, 1536), 8, 1, 128), (3, 16384, (8192, 1024, 1024), 8, 2, 128), (4, 4096, (20000, 20000), 8, 1, 128)):
        problems.append((B, K, Ns, v, m, g, 0, None, None))
    for _ in range(4000):
        v, m = rng.choice([(8, 1), (8, 2), (8, 2), (8, 3), (4, 1), (4, 2), (16, 2), (16, 4)])
        g = rng.choice([-1, 4 * v, 16 * v, 128, 256])
        if g > 0 and g < v:
            g = v
        unit = max(v, g)
        K = unit * max(1, int(2 ** rng.uniform(9, 15)) // unit)
        n0 = int(2 ** rng.uniform(7, 15))
        Ns = [n0] + [max(1, n0 // rng.choice([1, 2, 4, 8])) for _ in range(rng.randrange(4))]
        B = rng.choice([1, 2, 3, 4, 4, 5, 8, 12, 16, 24, 32])
        plan = None
        if rng.random() < 0.3:
            k = rng.choice([1, 2, 3, 4, 8])
            plan = (8, 1, k, 4, 0, 0, rng.choice([32, 64, 128]), rng.randint(1, 8))
        problems.append((B, K, Ns, v, m, g, rng.randrange(2), rng.choice([None, None, 1, 4, 32]), plan))
    raised = 0
    for p, (st, members, alone) in zip(problems, geometry([line(*p) for p in problems])):
        assert st == 0, p
        for a, b in zip(members, alone):
            assert same(a, b), (p, a, b)
            raised += a["staged"] and a["bg"] == 4 and a["rows"] == 128
    assert raised > 30                                              # the long K that 128-row blocks at 2 to 4 rows take


def test_explicit_block_heights_of_few_rows_are_kept(geometry):
    """8192 rows and K = 28672 at 4 rows, where the default plan takes 128-row blocks in four ranges: lower ones when asked for."""
    for rows in (32, 64, 128):
        for splits in (1, 2, 3, 4):
            [(st, members, _)] = geometry([line(4, 28672, [8192], 8, 2, 128, plan=(16, 1, 6, 4, 0, 0, rows, splits))])
            assert st == 0 and (members[0]["rows"], members[0]["nks"]) == (rows, splits)


def test_two_and_four_ranges_of_the_centroid_kernels_meet_pairwise(geometry):
    """At every batch; the batched Psumbook kernel, which takes 4 rows per pass too, combines four ranges through the ticket."""
    for B in (1, 2, 4, 5, 8, 16, 32):
        for splits, words in ((1, 0), (2, 1), (3, 0), (4, 3), (8, 0)):
            [(st, members, alone)] = geometry([line(B, 8192, [1000], 8, 2, 128, plan=(8, 1, 8, 4, 0, 0, 128, splits))])
            assert st == 0 and alone[0]["nks"] == splits and alone[0]["pairs"] == members[0]["pairs"] == B * words * 1024, (B, splits)
    for splits, words in ((2, 1), (4, 0)):
        [(st, _, alone)] = geometry([line(8, 8192, [1000], 8, 2, 128, plan=(8, 1, splits, 4, 0, 0, 0, 0))])
        assert st == 0 and alone[0]["pairs"] == 8 * words * 1024


def test_half_octets_take_no_extra_round(geometry):
    """Prompts of v4 m1 with group scales: tiles of 512 rows x 64 batch rows, but of 1024 x 32 where those take fewer rounds of 256
    workgroups (by more than the 8 % that the former are faster)."""
    rounds = lambda N, B, granules, rows: -(-(-(--(-N // 128) // granules) * -(-B // rows)) // 256)
    rng = random.Random(6)
    cases = [(28672, B) for B in (224, 256, 257, 270, 288, 289, 500)] + [(int(2 ** rng.uniform(10, 15)), int(2 ** rng.uniform(5.1, 12))) for _ in range(2000)]
    half = {}
    for (N, B), (_, _, [alone]) in zip(cases, geometry([line(B, 4096, [N], 4, 1, 128) for N, B in cases])):
        if alone["prompt"]:
            half[N, B] = alone["half"]
            assert alone["half"] == (12 * rounds(N, B, 4, 64) <= 13 * rounds(N, B, 8, 32)), (N, B)
        else:
            assert not alone["half"]
    assert [half[28672, B] for B in (224, 256, 257, 270, 288, 289, 500)] == [1, 1, 0, 0, 0, 1, 1]
    assert len(half) > 500 and all(rounds(N, B, 4, 64) <= 1.09 * rounds(N, B, 8, 32) for (N, B), h in half.items() if h)
    for [alone] in (a for _, _, a in geometry([line(270, 4096, [28672], v, m, g) for v, m, g in ((4, 1, -1), (8, 2, 128), (4, 2, 128))])):
        assert alone["prompt"] and not alone["half"]


@pytest.mark.parametrize("v,m,g,B,least", [
    (8, 2, 128, 4, 4096), (8, 1, 128, 2, 3072), (4, 1, 128, 3, 7168), (8, 2, -1, 4, None), (8, 1, -1, 2, None), (8, 2, 64, 4, None),
    (8, 2, -1, 5, 1024), (8, 1, -1, 8, 8192), (4, 1, -1, 6, 2048), (4, 1, 128, 7, 2048), (8, 2, 128, 8, 0), (8, 1, 128, 5, 0),
    (8, 2, -1, 9, 0), (8, 1, -1, 16, 2048), (8, 1, 128, 12, None), (4, 1, -1, 16, 0), (4, 1, 128, 9, 0),
    (8, 2, -1, 17, 0), (8, 1, -1, 32, None), (4, 1, 128, 24, 0), (8, 2, 128, 1, None), (8, 3, -1, 16, None)])
def test_staged_kernel_from_a_k_on(geometry, v, m, g, B, least):
    """128-row blocks: the K of a workgroup, whole units of 32 sub-vectors, from which on it stages its operands.  None: never."""
    Ks = sorted({k for K in (1024, 2048, 3072, 4096, 7168, 8192, 28672) for k in (K, K - 32 * v)})
    cases = [(k, splits, fp32) for k in Ks for splits in (1, 2) for fp32 in (0, 1)]
    lines = [line(B, k * splits, [3000], v, m, g, fp32=fp32, plan=(8, 1, 2, 4, 0, 0, 128, splits)) for k, splits, fp32 in cases]
    for (k, splits, fp32), (st, [member], [alone]) in zip(cases, geometry(lines)):
        assert st == 0 and member["kpw"] * 32 * v == k and same(member, alone)
        assert member["staged"] == (not fp32 and least is not None and k >= least), (k, splits, fp32)
