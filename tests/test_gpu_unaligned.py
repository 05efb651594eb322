"""Products whose rows are not aligned for 16-byte loads: the MFMA programs'
twins read such rows in 16-byte chunks at element alignment, shifting the
chunks that would cross the end of K or of N.  Every remainder of K and N
modulo a chunk, rows shorter than a chunk, edge and interior tiles, shares of
K and the grouped kernels, on small-integer operands (every sum exact in
float32, so the result must equal the oracle's bit for bit) whose surroundings
hold NaN."""
import sys

import numpy as np
import pytest
import torch

import oracle.matmul as om
from paper_1801_04348_amd import pk
from tests import inputs

pytestmark = pytest.mark.gpu

# one small tile, one of several chunks per work-item, and the largest that has a twin in every form
POINTS = {"f32": [(64, 64, 32, 2, 2), (128, 128, 32, 2, 2), (128, 256, 32, 2, 4), (256, 128, 16, 4, 2)],
          "bf16": [(64, 64, 64, 2, 2), (128, 128, 64, 2, 2), (256, 128, 32, 2, 2)]}
TINY = [(70, 200, 5), (70, 3, 200), (5, 7, 9), (1, 1, 1), (65, 8, 8), (66, 4, 4), (9, 6, 2)]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


def operand(shape, dtype, seed, lead=1, extra=4):
    """(host values, device view off 16-byte alignment, NaN around its rows)."""
    x = inputs.small_int_f32(shape, seed=seed)
    buf = torch.full((shape[0], shape[1] + extra), float("nan"), dtype=torch.float32)
    buf[:, lead:lead + shape[1]] = x
    if dtype == "bf16":
        return inputs.bf16_bits(x), inputs.bf16_bits(buf).cuda()[:, lead:lead + shape[1]]
    return x, buf.cuda()[:, lead:lead + shape[1]]


def check(table, dtype, p, a, b, ref, what):
    C = torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    try:
        pk.pk_matmul(table, p, dtype, a, b, C)
    except pk.PkError as e:
        if e.code in (pk.PK_ERR_NO_FEASIBLE_BRANCH, pk.PK_ERR_INVALID_ARG) and p.variant >= 0:
            return  # the program does not fit this machine, or has no split form
        raise
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), what


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r", range(8))
def test_every_remainder(table, dtype, r):
    shapes = [(70, 129 + r, 65 + r), (261, 257 + (3 * r) % 8, 136 + (5 * r) % 8)]
    shapes += TINY if r == 0 else []
    for M, N, K in shapes:
        (ah, a), (bh, b) = operand((M, K), dtype, 10 + r), operand((K, N), dtype, 20 + r)
        ref = om.matmul(ah, bh, dtype)
        for (bm, bn, bk, wm, wn) in POINTS[dtype]:
            for stage in (0, pk.PK_MFMA_SINGLE):
                for ks in (0, 3):
                    p = pk.params(family=pk.PK_FAMILY_MFMA, variant=stage, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn, ks=ks)
                    check(table, dtype, p, a, b, ref, (M, N, K, bm, bn, bk, stage, ks))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_grouped_rows_packed(table, dtype):
    dims = [(70 + 9 * i, 60 + 11 * i, 40 + 13 * i) for i in range(16)] + TINY
    ops = [(operand((M, K), dtype, 3 * i, lead=0, extra=0), operand((K, N), dtype, 3 * i + 1, lead=1, extra=2))
           for i, (M, N, K) in enumerate(dims)]
    Cs = [torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda") for M, N, _ in dims]
    plan = pk.pk_grouped_plan_create(table, dtype, [a[1] for a, _ in ops], [b[1] for _, b in ops], Cs)
    say(dtype, plan.kernels())
    plan.run()
    torch.cuda.synchronize()
    for (a, b), C, d in zip(ops, Cs, dims):
        assert np.array_equal(C.cpu().numpy().astype(np.float64), om.matmul(a[0], b[0], dtype)), d


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
def test_choice_of_one_size_on_both_alignments(table, dtype):
    # pk_matmul's own choice is kept per size and alignment: calls of one size
    # on aligned and unaligned rows in turn each compute the product
    M, N, K = 256, 512, 264
    a = inputs.small_int_i32((M, K), seed=41)
    b = inputs.small_int_i32((K, N), seed=42)
    ref = om.matmul(a, b, "i32").astype(np.float64)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "i32": torch.int32}[dtype]
    for lead in (0, 1, 0, 1):
        views = []
        for x in (a, b):
            buf = torch.zeros((x.shape[0], x.shape[1] + 8), dtype=dt, device="cuda")
            buf[:, lead:lead + x.shape[1]] = x.to(dt).cuda()
            views.append(buf[:, lead:lead + x.shape[1]])
        C = torch.full((M, N), -1, dtype=torch.int32 if dtype == "i32" else torch.float32, device="cuda")
        pk.pk_matmul(table, None, dtype, views[0], views[1], C)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), lead


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("steps", range(1, 14))
def test_steps_around_the_pipeline(table, dtype, steps):
    """One to thirteen K steps, whole and ragged, in edge tiles: loads run up
    to four steps ahead through registers."""
    for bk in sorted({p[2] for p in POINTS[dtype]}):
        for K in (steps * bk, steps * bk - 3, steps * bk + 1):
            M, N = 67, 131
            (ah, a), (bh, b) = operand((M, K), dtype, steps), operand((K, N), dtype, 40 + steps)
            ref = om.matmul(ah, bh, dtype)
            for (bm, bn, pbk, wm, wn) in POINTS[dtype]:
                for stage in (0, pk.PK_MFMA_SINGLE):
                    for ks in (0, 2) if steps in (9, 13) else (0,):
                        p = pk.params(family=pk.PK_FAMILY_MFMA, variant=stage, bm=bm, bn=bn, bk=pbk, wm=wm, wn=wn, ks=ks)
                        check(table, dtype, p, a, b, ref, (M, N, K, bm, bn, pbk, stage, ks))
