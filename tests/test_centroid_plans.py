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
    for B in (5, 8, 9, 16, 17, 32, 33):                                 # v = 16 and wide group scales: registers
        for rows in (32, 64, 128):
            assert ws(cg.Desc.make(B, 4096, 1000, 8, 2), rows, 1) > 0
            assert (ws(cg.Desc.make(B, 4096, 1000, 16, 2), rows, 1) > 0) == (rows >= (64 if B <= 8 else 128))
            assert (ws(cg.Desc.make(B, 4096, 1000, 8, 2, g=128), rows, 1) > 0) == (rows >= (32 if B <= 8 else 64))
            assert (ws(cg.Desc.make(B, 4096, 1000, 8, 2, g=64), rows, 1) > 0) == (rows >= (32 if B <= 8 else 128))
            assert ws(cg.Desc.make(B, 4096, 1000, 4, 1, g=128), rows, 1) > 0
            assert ws(cg.Desc.make(B, 4096, 1000, 4, 1, g=32), rows, 1) > 0
    for v, m, g, ok in ((8, 2, 128, True), (8, 2, 32, True), (8, 2, 16, False), (4, 1, 32, True), (4, 1, 16, False), (16, 2, 64, True), (16, 2, 32, False),
                        (4, 2, -1, True), (4, 3, -1, False), (16, 4, -1, True)):
        assert (ws(cg.Desc.make(4, 4096, 1000, v, m, g=g), 128, 1) > 0) == ok, (v, m, g)
    assert ws(cg.Desc.make(2, 512, 65536 * 128, 8, 1), 128, 1) == 0     # more blocks than a grid has


@pytest.mark.parametrize("v,m,g", [(8, 2, -1), (4, 1, 128), (8, 1, -1), (8, 3, -1), (16, 4, -1), (8, 2, 128), (8, 2, 32), (4, 4, -1)])
def test_default_plan_asks_for_no_more_workspace(v, m, g):
    for B in (1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 64, 70, 500, 5000, 65535):
        for K, N in ((512, 512), (2048, 2048), (8192, 1024), (4096, 4096), (14336, 4096), (8192, 28672), (28672, 8192), (1024, 1)):
            d = cg.Desc.make(B, K, N, v, m, g=g)
            p = cg.codegemm_default_plan(d)
            q = cg.Plan.from_buffer_copy(p)
            q.centroid_rows = q.centroid_splits = 0
            assert cg.codegemm_workspace_bytes(d, p) == cg.codegemm_workspace_bytes(d) <= cg.codegemm_workspace_bytes(d, q), (B, K, N)


def test_default_plan_keeps_the_other_kernels_where_they_win():
    plan = lambda B, K, N, v, m, g=-1: cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, g=g))
    assert plan(1, 8192, 28672, 8, 2).centroid_rows == 0 and plan(1, 2048, 2048, 8, 2).centroid_rows == 0
    assert plan(1, 8192, 8192, 16, 4).centroid_rows == 0
    assert (plan(1, 4096, 4096, 8, 2).centroid_rows, plan(1, 4096, 4096, 8, 2).centroid_splits) == (32, 1)
    fp32 = lambda B, K, N, v, m: cg.codegemm_default_plan(cg.Desc.make(B, K, N, v, m, y_fp32=True))
    assert fp32(1, 4096, 4096, 8, 2).centroid_rows == 0 and fp32(1, 4096, 4096, 8, 1).centroid_rows == 32
    assert fp32(4, 8192, 8192, 16, 4).centroid_rows == 0 and fp32(16, 8192, 8192, 16, 2).centroid_rows == 128
    assert plan(4, 8192, 8192, 8, 2, 16).centroid_rows == 0             # groups smaller than an MFMA's contraction
    assert plan(16, 2048, 2048, 8, 2, 32).centroid_rows == 0 and plan(16, 2048, 2048, 8, 1, 32).centroid_rows != 0
    assert plan(2, 8192, 8192, 16, 4, 64).centroid_rows == 0 and plan(4, 8192, 8192, 16, 4, 64).centroid_rows != 0
    for B in (2, 8, 32, 500):
        assert plan(B, 8192, 28672, 8, 2).centroid_rows != 0
    assert plan(2, 512, (1 << 24), 8, 1).centroid_rows == 0             # more blocks than a grid has
