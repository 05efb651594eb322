"""C += A B of the MFMA programs at the edges of their tiles: every program on
interior and ragged tiles, every element of C with a value of its own, and
nothing written around C.  Operands are small integers, so results are exact."""
import pytest
import torch

from paper_1801_04348_amd import pk
from tests import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


@pytest.fixture(scope="module")
def described(table):
    return pk.pk_case_table_describe(table)


def programs(described, dtype):
    code = {"f32": pk.PK_F32, "i32": pk.PK_I32, "bf16": pk.PK_BF16}[dtype]
    return sorted({tuple(e[k] for k in ("bm", "bn", "bk", "wm", "wn", "variant")) for e in described["instances"]
                   if e["family"] == pk.PK_FAMILY_MFMA and e["dtype"] == code and e["variant"] in (0, 1)})


# one row and column, a block of 32 less and more one, tiles less and more one, whole tiles
@pytest.mark.parametrize("rows", ["1", "31", "33", "bm - 1", "bm + 1", "2 * bm"])
@pytest.mark.parametrize("dtype", ["f32", "i32", "bf16"])
def test_every_program(table, described, dtype, rows):
    ran = 0
    for bm, bn, bk, wm, wn, stage in programs(described, dtype):
        M, N, K = eval(rows, {"bm": bm}), eval(rows, {"bm": bn}), bk + 3
        A, B = inputs.small_int_f32((M, K), seed=M), inputs.small_int_f32((K, N), seed=N + 1)
        start = torch.arange(M * N, dtype=torch.float32).reshape(M, N) % 8191
        ref = (A.double() @ B.double() + start.double())
        out = torch.int32 if dtype == "i32" else torch.float32
        cast = (lambda x: x.int()) if dtype == "i32" else inputs.bf16_bits if dtype == "bf16" else (lambda x: x)
        for pad in (0, 3):
            buf = torch.full((M + 2, N + 8), -77, dtype=out, device="cuda")
            C = buf[1:-1, 1 + pad:1 + pad + N]
            C.copy_(start.to(out))
            p = pk.params(family=pk.PK_FAMILY_MFMA, variant=stage, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn, ks=0)
            print("accumulate %s %dx%dx%d_w%dx%d stage %d on %dx%dx%d" % (dtype, bm, bn, bk, wm, wn, stage, M, N, K),
                  flush=True)
            try:
                pk.pk_matmul(table, p, dtype, cast(A).cuda(), cast(B).cuda(), C, accumulate=True)
            except pk.PkError as e:  # does not fit the bound machine
                assert e.code in (pk.PK_ERR_NO_FEASIBLE_BRANCH, pk.PK_ERR_INVALID_ARG)
                continue
            ran += 1
            got = buf.cpu()
            assert torch.equal(got[1:-1, 1 + pad:1 + pad + N].double(), ref)
            got[1:-1, 1 + pad:1 + pad + N] = -77
            assert (got == -77).all()
    assert ran >= 4
