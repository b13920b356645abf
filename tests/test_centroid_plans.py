"""Host logic of plans with centroid_rows != 0: what is offered, sized and refused, and that the default plan asks for
no more workspace than the Psumbook kernels' fields of the same plan do.  No kernel is launched."""
import pytest

import paper_2512_17970_amd as cg


def ws(d, rows, splits, base=(8, 1, 4, 4)):
    return cg.codegemm_workspace_bytes(d, cg.Plan.make(*base, 0, 0, rows, splits))


def test_offered_and_refused():
    d = cg.Desc.make(4, 4096, 1000, 8, 2)
    assert ws(d, 32, 1) > 0 and ws(d, 64, 2) > 0 and ws(d, 128, 1000) > 0
    for rows, splits in ((16, 1), (96, 1), (256, 1), (128, 0), (128, -1), (0, 1), (-128, 1)):
        assert ws(d, rows, splits) == 0
    # more blocks than a grid has: the Psumbook fields hold, whose K ranges need more counters than there are here
    assert ws(cg.Desc.make(2, 512, 65536 * 128, 8, 1), 128, 1) == 0
    assert ws(cg.Desc.make(2, 512, 65536 * 128, 8, 1), 128, 1, (8, 1, 1, 4)) > 0


@pytest.mark.parametrize("g", [-1, 128, 8])
def test_a_group_refuses_the_plans_that_a_layer_refuses(g):
    """The plan as given is what counts: raising blocks, cutting ranges or falling back to the Psumbook fields must not make a valid one of it."""
    for B, K, heights in ((4, 4096, [700, 300]), (4, 28672, [4096, 4096])):
        d = cg.Desc.make(B, K, sum(heights), 8, 2, g=g)
        for rows, splits in ((32, 0), (64, -1), (128, 0), (16, 1), (31, 1), (96, 1), (-128, 1), (1, 1), (0, 1)):
            assert ws(d, rows, splits) == 0
            assert cg.codegemm_grouped_workspace_bytes(d, cg.Plan.make(8, 1, 4, 4, 0, 0, rows, splits), heights) == 0, (g, rows, splits)
        assert cg.codegemm_grouped_workspace_bytes(d, cg.Plan.make(8, 1, 4, 4, 0, 0, 32, 1), heights) > 0


BATCHES = (1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 64, 500)


@pytest.mark.parametrize("v,m", [(8, 2), (8, 1), (8, 3), (8, 4), (4, 1), (4, 2), (4, 3), (16, 1), (16, 2), (16, 4)])
def test_a_plan_serves_every_batch_output_type_and_group_size(v, m):
    """A plan chosen for one batch of a layer was always accepted for the others (the Psumbook fields are): blocks grow
    where 32 rows do not fit, formats without the centroid kernel fall back to the Psumbook fields.  The workspace is that
    of the Psumbook fields throughout, so it grows with the batch alone and one of the largest batch serves them all."""
    groups = (-1, 32 * v, 16 * v, 8 * v, 4 * v, 2 * v, v)
    for K, N in ((32 * v * 20, 1000), (32 * v * 8, 4096), (32 * v * 80, 300)):
        for g0 in groups[:5]:
            for B0 in BATCHES:
                for fp32 in (False, True):
                    p = cg.codegemm_default_plan(cg.Desc.make(B0, K, N, v, m, y_fp32=fp32, g=g0))
                    if not p.centroid_rows:
                        continue
                    q = cg.Plan.from_buffer_copy(p)
                    q.centroid_rows = q.centroid_splits = 0
                    for g in groups:
                        last = 0
                        for B in BATCHES:
                            d = cg.Desc.make(B, K, N, v, m, y_fp32=not fp32, g=g)
                            need = cg.codegemm_workspace_bytes(d, q)
                            assert cg.codegemm_workspace_bytes(d, p) == need >= last, (B0, g0, B, g, p)
                            if need and B <= 32:
                                assert cg.codegemm_grouped_workspace_bytes(d, p, [N - 100, 70, 30]) == cg.codegemm_grouped_workspace_bytes(d, q, [N - 100, 70, 30]) > 0
                            last = need


def test_k_splits_bounds_the_workspace_of_an_edited_default_plan():
    d = cg.Desc.make(2, 16384, 512, 8, 2)
    p = cg.codegemm_default_plan(d)
    assert p.centroid_rows and p.centroid_splits > 2
    for k in (1, 2):
        p.k_splits = k
        assert cg.codegemm_workspace_bytes(d, p) == 65536 + (2 << 20) + 2 * k * 512 * 4


def test_plans_of_small_layers_fit_large_ones():
    """Blocks of 32 rows would be more than a grid has, or than there are ticket counters for several K ranges."""
    p = cg.codegemm_default_plan(cg.Desc.make(2, 8192, 512, 8, 2))
    assert p.centroid_rows == 32 and p.centroid_splits > 1
    p.k_splits = 1
    for N in (1 << 19, (1 << 19) + 1, 1 << 20, 1 << 22, 1 << 24):
        d = cg.Desc.make(2, 8192, N, 8, 2)
        assert cg.codegemm_workspace_bytes(d, p) > 0
        if N < 1 << 24:                                                # the Psumbook kernels' row blocks of a group end at 65535
            assert cg.codegemm_grouped_workspace_bytes(d, p, [N - 1000, 900, 99, 1]) > 0


@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (4, 1, 128), (8, 1, -1), (8, 3, -1), (16, 4, -1), (8, 2, 128), (8, 2, 32), (4, 4, -1)])
def test_default_plan_asks_for_no_more_workspace(v, m, g):
    for B in (1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 64, 70, 500, 5000, 65535):
        for K, N in ((512, 512), (2048, 2048), (8192, 1024), (4096, 4096), (14336, 4096), (8192, 28672), (28672, 8192), (1024, 1)):
            d = cg.Desc.make(B, K, N, v, m, g=g)
            p = cg.codegemm_default_plan(d)
            q = cg.Plan.from_buffer_copy(p)
            q.centroid_rows = q.centroid_splits = 0
            assert cg.codegemm_workspace_bytes(d, p) == cg.codegemm_workspace_bytes(d) <= cg.codegemm_workspace_bytes(d, q), (B, K, N)


@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (4, 1, 128), (4, 1, 32), (8, 1, -1), (8, 1, 128), (8, 3, -1), (16, 4, -1), (8, 2, 128), (8, 2, 32)])
def test_default_blocks_and_ranges_of_few_rows(v, m, g):
    """Up to 4 batch rows: one round of 256 workgroups wherever a block height allows it, K ranges that are powers of two and
    all of one length but the last (two and four meet pairwise, three, five or seven would take the slower ticket).  Blocks are
    as low as that allows, but for 2 to 4 rows with v = 8, at most two codebooks, fp16 output and groups of at least 16 chunks, where
    128-row blocks in two or four ranges that come to 160 to 256 workgroups with a K of 6144 (two codebooks: 7168) or more each take over."""
    seen = set()
    for B in (1, 2, 3, 4):
        for N in (512, 700, 1300, 1500, 2000, 2900, 4096, 8192, 8193, 10000, 14336, 16384, 17000, 20000, 28672):
            for K in (512, 1024, 2560, 4096, 5120, 7168, 9216, 12288, 18944, 28672):
                for fp32 in (False, True):
                    p = cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, y_fp32=fp32, g=g))
                    if not p.centroid_rows:
                        continue
                    blocks, s, nkt = -(-N // p.centroid_rows), p.centroid_splits, -(-(K // v) // 32)
                    assert blocks <= 256 or p.centroid_rows == 128, (B, K, N, p)
                    tall = -(-N // 128)
                    ranges = 4 if 4 * tall <= 256 else 2
                    if (2 <= B <= 4 and v == 8 and m <= 2 and g >= 128 and not fp32 and 160 <= ranges * tall <= 256
                            and -(-nkt // ranges) * 32 * v >= (6144 if m == 1 else 7168)):
                        assert (p.centroid_rows, s) == (128, ranges), (B, K, N, p)
                    else:
                        assert p.centroid_rows == 32 or -(-N // (p.centroid_rows // 2)) > 256, (B, K, N, p)
                    assert s & (s - 1) == 0 and -(-nkt // -(-nkt // s)) == s and (s == 1 or s * blocks <= 256), (B, K, N, p)
                    seen.add((p.centroid_rows, s))
    assert {r for r, _ in seen} == {32, 64, 128} and {1, 2, 4, 8} <= {s for _, s in seen}


@pytest.mark.parametrize("m,K,N,want", [
    (2, 28672, 8192, (128, 4)), (2, 28672, 8193, (64, 1)),             # 4 x 64 workgroups, one block more
    (2, 28672, 5120, (128, 4)), (2, 28672, 4992, (32, 1)),             # 160 workgroups, 156
    (2, 28672, 10240, (128, 2)), (2, 28672, 10112, (64, 1)),           # two ranges: 160 workgroups, 158
    (2, 28672, 16384, (128, 2)), (2, 28672, 16385, (0, 0)),            # two ranges: 256 workgroups; 129 blocks are the Psumbook kernels'
    (2, 14336, 16384, (128, 2)), (2, 13824, 16384, (64, 1)),           # K of a workgroup: 7168, 6912
    (1, 12288, 16384, (128, 2)), (1, 11776, 16384, (64, 1)),           # .. 6144, 5888
])
def test_tall_blocks_of_few_rows(m, K, N, want):
    for B in (2, 3, 4):
        p = cg.codegemm_default_plan(cg.Desc.make(B, K, N, 8, m, g=128))
        assert (p.centroid_rows, p.centroid_splits) == want and p.k_splits >= want[1]
    for kept in (cg.Desc.make(4, K, N, 8, m), cg.Desc.make(4, K, N, 8, m, g=64), cg.Desc.make(4, K, N, 8, m, g=128, y_fp32=True), cg.Desc.make(4, K, N, 8, 3, g=128)):
        p = cg.codegemm_default_plan(kept)
        if N <= 16384:
            assert p.centroid_rows in (32, 64), (kept, p)


def test_default_plan_keeps_the_other_kernels_where_they_win():
    plan = lambda B, K, N, v, m, g=-1: cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, g=g))
    assert plan(1, 8192, 28672, 8, 2).centroid_rows == 0 and plan(1, 2048, 2048, 8, 2).centroid_rows == 0
    assert plan(1, 8192, 8192, 16, 4).centroid_rows == 0
    assert (plan(1, 4096, 4096, 8, 2).centroid_rows, plan(1, 4096, 4096, 8, 2).centroid_splits) == (32, 1)
    fp32 = lambda B, K, N, v, m: cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, y_fp32=True))
    assert fp32(1, 4096, 4096, 8, 2).centroid_rows == 0 and fp32(1, 4096, 4096, 8, 1).centroid_rows == 32
    assert fp32(4, 8192, 8192, 16, 4).centroid_rows == 0 and fp32(16, 8192, 8192, 16, 2).centroid_rows == 0 and fp32(4, 8192, 8192, 16, 2).centroid_rows == 32
    assert plan(4, 8192, 8192, 8, 2, 16).centroid_rows == 0             # groups smaller than an MFMA's contraction
    assert plan(16, 2048, 2048, 8, 3, 32).centroid_rows == 0 and plan(16, 2048, 2048, 8, 1, 32).centroid_rows != 0
    assert plan(2, 8192, 8192, 16, 4, 64).centroid_rows == 0 and plan(4, 8192, 8192, 16, 4, 64).centroid_rows != 0
    for B in (2, 8, 32, 500):
        assert plan(B, 8192, 28672, 8, 2).centroid_rows != 0
    assert plan(2, 512, (1 << 24), 8, 1).centroid_rows == 0             # more blocks than a grid has


@pytest.mark.parametrize("g", [32, 64])
def test_small_matrices_with_short_groups(g):
    """v8 m2, fp16 output: low staged blocks at every size (2048^2 g32, 16 rows: Psumbook kernels 7.8 us, staged 4.7; 5376->768 9.7, 6.0; 512->627 g64,
    24 rows 6.7, 4.2).  fp32 output has no such blocks."""
    for B in (8, 9, 16, 17, 32, 33):
        for K, N in ((512, 627), (1024, 1024), (2048, 2048), (4096, 1024), (5376, 768), (16384, 128)):
            assert cg.codegemm_default_plan(cg.Desc.make(B, K, N, 8, 2, g=g)).centroid_rows == 32, (B, K, N)
            if 9 <= B <= 32:
                assert cg.codegemm_default_plan(cg.Desc.make(B, K, N, 8, 2, g=g, y_fp32=True)).centroid_rows == 0, (B, K, N)


def test_two_rounds_of_tall_blocks():
    """5 to 8 rows, v8 m2, more than 256 blocks of 128 rows: no three rounds of lower ones, at any K (these tie, and cost up to 4 % more: K = 27216,
    37725 rows of W, 6 batch rows, 64 / 128 rows 93.1 / 89.6 us in one run, 88.9 / 89.7 in another; K = 8224, 33591 rows 32.8 / 32.6)."""
    for B, K, N in ((6, 3864, 33410), (8, 5216, 42881), (8, 6240, 40871), (6, 8160, 33591), (6, 8224, 33591), (5, 16384, 49152), (6, 27216, 37725)):
        p = cg.codegemm_default_plan(cg.Desc.make(B, K, N, 8, 2))
        assert (p.centroid_rows, p.centroid_splits) == (128, 1), (B, K, N, p)


@pytest.mark.parametrize("m,v,K,least", [(1, 8, 4096, 3072), (2, 8, 8192, 4096), (1, 4, 8192, 7168)])
def test_two_rounds_of_staged_blocks_or_more_of_lower_ones(m, v, K, least):
    """2 to 4 rows with group scales, more than 256 blocks of 128 rows: 64-row blocks while there are at most 768 of them, from the K on
    that tall blocks are staged at.  A group of that height follows the same plan."""
    rows = lambda B, K, N, g=128: cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, g=g)).centroid_rows
    for B in (2, 3, 4):
        assert [rows(B, K, N) for N in (32768, 32769, 40000, 49152, 49153, 57344, 65536)] == [128, 64, 64, 64, 128, 128, 128]
        assert rows(B, least, 40000) == 64 and rows(B, least - 32 * v, 40000) == 128
        assert rows(B, K, 40000, -1) == 128
