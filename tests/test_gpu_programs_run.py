"""That the MFMA programs of the direct-load and unaligned-row tests do run:
every program, stage count and split that the compiler's resource report says
fits the bound machine, on aligned and on unaligned rows, and no other.  Its
operands have infinities of both signs around them, and a product holds one in
a row of A and one in a column of B at the ragged end of K."""
import numpy as np
import pytest
import torch

import oracle.enumerate as oe
import oracle.matmul as om
from paper_1801_04348_amd import pk
from tests import inputs, test_gpu_dma, test_gpu_unaligned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


@pytest.fixture(scope="module")
def described(table):
    return pk.pk_case_table_describe(table)


def points(dtype):
    return sorted(set(test_gpu_dma.POINTS[dtype]) | set(test_gpu_unaligned.POINTS[dtype]))


def forms(described, dtype, point, stage):
    """The compiled kernels of a program: by variant bits (0, 4: twin, 16: split)."""
    code = {"f32": pk.PK_F32, "bf16": pk.PK_BF16}[dtype]
    return {e["variant"] & ~1: e for e in described["instances"]
            if e["family"] == pk.PK_FAMILY_MFMA and e["dtype"] == code and not e["variant"] & (2 | 8) and
            (e["variant"] & 1) == stage and tuple(e[k] for k in ("bm", "bn", "bk", "wm", "wn")) == point}


def expected(described, dtype, point, stage, ks):
    m, f = described["machine"], forms(described, dtype, point, stage)
    regs = max(oe.regs_per_block(e["vgpr"], e["agpr"], e["threads"]) for e in f.values())
    fits = regs <= m["regs_block"] and f[0]["lds_bytes"] <= m["lds_block"] and f[0]["threads"] <= m["max_threads_block"]
    return fits and (ks == 0 or 16 in f)


def operand(shape, dtype, seed, lead):
    """(host values, device view `lead` elements past alignment, infinities around its rows)."""
    x = inputs.small_int_f32(shape, seed=seed)
    ld = -(-shape[1] // 8) * 8 + 16
    buf = torch.full((shape[0] + 2, ld), float("inf"), dtype=torch.float32)
    buf[:, ::2] = -float("inf")
    buf[1:-1, 8 + lead:8 + lead + shape[1]] = x
    dev = (inputs.bf16_bits(buf) if dtype == "bf16" else buf).cuda()[1:-1, 8 + lead:8 + lead + shape[1]]
    return (inputs.bf16_bits(x) if dtype == "bf16" else x), dev


def runs(table, dtype, point, stage, ks, a, b, C):
    bm, bn, bk, wm, wn = point
    p = pk.params(family=pk.PK_FAMILY_MFMA, variant=stage, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn, ks=ks)
    try:
        pk.pk_matmul(table, p, dtype, a, b, C)
    except pk.PkError as e:
        assert e.code in (pk.PK_ERR_NO_FEASIBLE_BRANCH, pk.PK_ERR_INVALID_ARG)
        return False
    torch.cuda.synchronize()
    return True


@pytest.mark.parametrize("lead", [0, 1, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_what_fits_runs(table, described, dtype, lead):
    ran = {}
    for point in points(dtype):
        bm, bn, bk = point[:3]
        M, N, K = bm + 6, bn + 7, 5 * bk - 3
        (ah, a), (bh, b) = operand((M, K), dtype, 1, lead), operand((K, N), dtype, 2, lead)
        ref = om.matmul(ah, bh, dtype)
        for stage in (0, 1):
            for ks in (0, 2):
                C = torch.full((M, N), float("nan"), device="cuda")
                ran[point, stage, ks] = runs(table, dtype, point, stage, ks, a, b, C)
                if ran[point, stage, ks]:
                    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), (point, stage, ks)
    assert ran == {(p, s, k): expected(described, dtype, p, s, k) for p, s, k in ran}
    for point in points(dtype):
        assert ran[point, 0, 0] or ran[point, 1, 0], point


@pytest.mark.parametrize("lead", [0, 1, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinities_stay_in_their_rows(table, described, dtype, lead):
    """In row 3 of A and column 5 of B, at the last of a ragged K: they reach
    that row and that column only, through the shifts and masks too."""
    M, N, ran = 70, 77, 0
    one = (lambda v: inputs.bf16_bits(torch.tensor([[v]])).item()) if dtype == "bf16" else (lambda v: v)
    for K in (103, 106):
        (ah, a), (bh, b) = operand((M, K), dtype, 3, lead), operand((K, N), dtype, 4, lead)
        ref = om.matmul(ah, bh, dtype)
        a[3, K - 1], b[K - 1, 5] = one(float("inf")), one(-float("inf"))
        rows, cols = np.arange(M) != 3, np.arange(N) != 5
        for point in points(dtype):
            for stage in (0, 1):
                C = torch.zeros((M, N), device="cuda")
                if not runs(table, dtype, point, stage, 0, a, b, C):
                    continue
                ran += 1
                got = C.cpu().numpy().astype(np.float64)
                assert np.array_equal(got[np.ix_(rows, cols)], ref[np.ix_(rows, cols)]), (K, point, stage)
                # an infinity, or NaN where the other operand's value is zero
                assert not np.isfinite(got[3]).any() and not np.isfinite(got[:, 5]).any(), (K, point, stage)
    assert ran == 2 * sum(expected(described, dtype, p, s, 0) for p in points(dtype) for s in (0, 1)) > 0


def test_deep_buffers_under_capture(table):
    """Launches that add LDS for a third and fourth buffer, recorded in a graph
    whose programs have not run before, replayed among other work."""
    M, N, K = 200, 300, 1003
    (ah, a), (bh, b) = operand((M, K), "bf16", 5, 0), operand((K, N), "bf16", 6, 0)
    ref = om.matmul(ah, bh, "bf16")
    ps = [pk.params(family=pk.PK_FAMILY_MFMA, variant=s, bm=bm, bn=bn, bk=64, wm=2, wn=2)
          for bm, bn in ((64, 128), (128, 64)) for s in (0, 1)]
    outs = [torch.zeros((M, N), device="cuda") for _ in ps]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for p, C in zip(ps, outs):
            pk.pk_matmul(table, p, "bf16", a, b, C)
    for _ in range(3):
        for C in outs:
            C.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for p, C in zip(ps, outs):
            assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), p
