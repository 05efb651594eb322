"""Products whose aligned rows lie megabytes apart, below and past the 4 GiB
that a tile's direct loads reach: the wide program or its twin, or, where the
program named has none, the CASE choice -- each the oracle's small-integer
result bit for bit, with NaN between the rows."""
import numpy as np
import pytest
import torch

import oracle.matmul as om
from paper_1801_04348_amd import pk
from tests import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


def spread(shape, dtype, ld, seed):
    """(host values, device view of row stride ld, NaN beside its rows)."""
    x = inputs.small_int_f32(shape, seed=seed)
    host = inputs.bf16_bits(x) if dtype == "bf16" else x
    buf = torch.empty(((shape[0] - 1) * ld + shape[1] + 8,), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                      device="cuda")
    around = buf.as_strided((shape[0], shape[1] + 8), (ld, 1))
    around.fill_(float("nan"))
    view = around[:, :shape[1]]
    view.copy_(x.to(buf.dtype))
    return host, view


# program (bm, bn, bk, wm, wn), stages, (M, N, K); rows that its tile reads at a time of A, of B
PROGRAMS = [("f32", (64, 64, 32, 2, 2), 0, (70, 72, 88), 64, 32),
            ("f32", (64, 64, 32, 2, 2), 1, (70, 72, 40), 64, 16),
            ("bf16", (128, 64, 64, 2, 2), 0, (130, 72, 136), 128, 64),
            ("bf16", (128, 256, 64, 2, 2), 1, (130, 264, 72), 128, 32),   # no twin
            ("bf16", (256, 128, 32, 2, 2), 1, (260, 136, 72), 256, 32)]   # loads through registers


@pytest.mark.parametrize("which", ["a", "b"])
@pytest.mark.parametrize("span", [2 ** 31 - 2 ** 20, 2 ** 31 + 2 ** 20, 2 ** 32 - 2 ** 20, 2 ** 32 + 2 ** 20])
def test_spans_of_a_tile(table, which, span):
    ran = 0
    for dtype, (bm, bn, bk, wm, wn), stage, (M, N, K), rows_a, rows_b in PROGRAMS:
        es = 2 if dtype == "bf16" else 4
        ld = span // es // ((rows_a if which == "a" else rows_b) - 1) // 8 * 8
        A, a = spread((M, K), dtype, ld if which == "a" else K + 8, 1)
        B, b = spread((K, N), dtype, ld if which == "b" else N + 8, 2)
        assert a.data_ptr() % 16 == 0 and b.data_ptr() % 16 == 0
        ref = om.matmul(A, B, dtype)
        p = pk.params(family=pk.PK_FAMILY_MFMA, variant=stage, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn)
        for params in (p, None):
            C = torch.full((M, N), float("nan"), device="cuda")
            try:
                pk.pk_matmul(table, params, dtype, a, b, C)
            except pk.PkError as e:
                if e.code != pk.PK_ERR_NO_FEASIBLE_BRANCH:
                    raise
                continue
            torch.cuda.synchronize()
            ran += params is not None
            assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), (dtype, bm, bn, bk, stage, ld)
        C = torch.full((M, N), float("nan"), device="cuda")
        pk.pk_grouped_plan_create(table, dtype, [a], [b], [C]).run()
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), ("grouped", dtype, ld)
        del a, b
        torch.cuda.empty_cache()
    assert ran >= 3


def test_one_row_of_any_stride(table):
    A, a = spread((1, 96), "f32", 1 << 20, 1)
    a = a.as_strided((1, 96), (1 << 40, 1))
    B, b = spread((96, 64), "f32", 72, 2)
    C = torch.full((1, 64), float("nan"), device="cuda")
    pk.pk_matmul(table, None, "f32", a, b, C)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy().astype(np.float64), om.matmul(A, B, "f32"))
