"""Products whose rows are aligned for 16-byte loads: the wide MFMA programs
copy them straight to LDS, in a cycle of two to four buffers of K steps.  K of
one step's part, of whole steps fewer and more than the buffers, and ragged
ones; tiles at the edges of M and N; shares of K; accumulation; operands whose
surroundings hold NaN and values of both infinities' sign.  Small-integer
operands: every sum is exact in float32, so results equal the oracle's bit
for bit."""
import numpy as np
import pytest
import torch

import oracle.matmul as om
from paper_1801_04348_amd import pk
from tests import inputs

pytestmark = pytest.mark.gpu

# (bm, bn, bk, wm, wn): tiles of two, three and four buffers, and the two
# orders in which the largest split their step
POINTS = {"f32": [(64, 64, 32, 2, 2), (128, 64, 32, 2, 2), (128, 256, 32, 2, 4), (256, 128, 16, 4, 2)],
          "bf16": [(64, 64, 64, 2, 2), (64, 128, 64, 2, 2), (128, 128, 64, 2, 2), (128, 256, 32, 2, 2),
                   (128, 256, 64, 2, 2), (256, 128, 32, 2, 2), (256, 128, 64, 2, 2)]}


@pytest.fixture(scope="module")
def table():
    return pk.pk_case_table_build(0)


def operand(shape, dtype, seed):
    """(host values, device view on 16-byte alignment, NaN around its rows)."""
    x = inputs.small_int_f32(shape, seed=seed)
    ld = -(-shape[1] // 8) * 8 + 8
    buf = torch.full((shape[0] + 2, ld + 8), float("nan"), dtype=torch.float32)
    buf[1:-1, 8:8 + shape[1]] = x
    dev = (inputs.bf16_bits(buf) if dtype == "bf16" else buf).cuda()[1:-1, 8:8 + shape[1]]
    assert dev.data_ptr() % 16 == 0
    return (inputs.bf16_bits(x) if dtype == "bf16" else x), dev


def run(table, dtype, point, variant, ks, a, b, C, accumulate=False):
    bm, bn, bk, wm, wn = point
    p = pk.params(family=pk.PK_FAMILY_MFMA, variant=variant, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn, ks=ks)
    try:
        pk.pk_matmul(table, p, dtype, a, b, C, accumulate=accumulate)
    except pk.PkError as e:
        if e.code in (pk.PK_ERR_NO_FEASIBLE_BRANCH, pk.PK_ERR_INVALID_ARG):
            return False  # the program does not fit this machine, or has no split form
        raise
    torch.cuda.synchronize()
    return True


def cases():
    return [(d, pt) for d in POINTS for pt in POINTS[d]]


@pytest.mark.parametrize("dtype,point", cases())
def test_steps_and_edges(table, dtype, point):
    bm, bn, bk = point[:3]
    # part of a step; whole steps around the buffers' number; ragged ends
    for i, K in enumerate((1, bk // 2 - 3, bk // 2, bk - 1, bk, bk + 5, 2 * bk, 3 * bk - 7, 4 * bk, 5 * bk + bk // 2, 7 * bk + 1)):
        M, N = [(bm + 3, 2 * bn - 5), (1, 3), (2 * bm, bn), (bm - 1, bn + 1)][i % 4]
        A, a = operand((M, K), dtype, 2 * i)
        B, b = operand((K, N), dtype, 2 * i + 1)
        ref = om.matmul(A, B, dtype)
        for variant in (0, 1):
            for ks in (0, 2):
                out = torch.full((M + 1, N + 3), float("nan"), device="cuda")
                C = out[:M, :N]
                if not run(table, dtype, point, variant, ks, a, b, C):
                    continue
                got = out.cpu().numpy()
                assert np.array_equal(got[:M, :N].astype(np.float64), ref), (M, N, K, variant, ks)
                assert np.isnan(got[M:]).all() and np.isnan(got[:, N:]).all()
                C.copy_(torch.ones_like(C))
                run(table, dtype, point, variant, ks, a, b, C, accumulate=True)
                assert np.array_equal(C.cpu().numpy().astype(np.float64), ref + 1), (M, N, K, variant, ks)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinities_stay_in_their_rows(table, dtype):
    """An infinity in row 3 of A and one in column 5 of B reach that row and
    that column only, over a ragged last step."""
    M, N, K = 70, 72, 104
    A, a = operand((M, K), dtype, 1)
    B, b = operand((K, N), dtype, 2)
    A, B = A.clone(), B.clone()
    inf = torch.tensor(float("inf"))
    a[3, K - 1] = inf if dtype == "f32" else inputs.bf16_bits(inf.reshape(1, 1)).item()
    b[K - 1, 5] = -inf if dtype == "f32" else inputs.bf16_bits(-inf.reshape(1, 1)).item()
    ref = om.matmul(A, B, dtype)
    C = torch.empty((M, N), device="cuda")
    for point in POINTS[dtype]:
        if not run(table, dtype, point, 0, 0, a, b, C):
            continue
        got = C.cpu().numpy().astype(np.float64)
        rows, cols = np.arange(M) != 3, np.arange(N) != 5
        assert np.array_equal(got[np.ix_(rows, cols)], ref[np.ix_(rows, cols)]), point
        # +-inf, or NaN where the other operand's value is zero
        assert not np.isfinite(got[3]).any() and not np.isfinite(got[:, 5]).any()
