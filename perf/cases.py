"""Performance cases: the calls a user of this library makes, over the sizes
they are made at.

Every case goes through the Python binding's public entry points with no
program parameters given, i.e. with the case table's own (CASE) choice, which
is what a program that has not tuned anything calls.  Sizes are those of the
benchmark, the side benchmarks and the tests (products of order 256 to 8192,
the sweep's 1000 and 3000, groups of products of 16 to 512, transposition of
order 2^14, the Jacobi vector of 2^15 + 2 points, division by a polynomial of
degree 2^15) and odd ones of the same ranges.
"""
import math
import random

import numpy as np
import torch

from paper_1801_04348_amd import pk

MODULUS = 2147483647  # the side benchmark's prime, 2^31 - 1
_tables = {}


def _table():
    """The bound case table, built once per process as a program does."""
    if "t" not in _tables:
        torch.cuda.init()
        _tables["t"] = pk.pk_case_table_build(0)
    return _tables["t"]


def listed():
    return [
        # the smallest call: one product of order 256, where the latency of
        # choosing and launching counts (the float32 parity size)
        dict(name="f32_256", kind="matmul", dtype="f32", M=256, N=256, K=256, pad=0, accumulate=False),
        # packed operands of odd sizes: rows not aligned for wide loads
        dict(name="f32_odd", kind="matmul", dtype="f32", M=1531, N=777, K=1201, pad=0, accumulate=False),
        # one of the sweep's large products, with a ragged edge along N
        dict(name="f32_8192x3000x4096", kind="matmul", dtype="f32", M=8192, N=3000, K=4096, pad=0, accumulate=False),
        # the dense bfloat16 product
        dict(name="bf16_4096", kind="matmul", dtype="bf16", M=4096, N=4096, K=4096, pad=0, accumulate=False),
        # bfloat16, packed operands of odd sizes
        dict(name="bf16_odd", kind="matmul", dtype="bf16", M=1021, N=3001, K=2047, pad=0, accumulate=False),
        # the wrapping int32 product of the parity configurations
        dict(name="i32_1024", kind="matmul", dtype="i32", M=1024, N=1024, K=1024, pad=0, accumulate=False),
        # many uneven products through a plan that the program keeps: rows
        # padded to 8 elements, as the benchmark lays them out ...
        dict(name="grouped_f32_4096", kind="grouped", dtype="f32", G=4096, lo=16, hi=512, dims_seed=0, pad=8),
        # ... and packed tightly, as they come when nobody pads them
        dict(name="grouped_bf16_packed", kind="grouped", dtype="bf16", G=1024, lo=16, hi=512, dims_seed=1, pad=0),
        # transposition of order 2^14 (the paper's Table 3)
        dict(name="transpose_16384", kind="transpose", dtype="f32", M=16384, N=16384),
        # addition of two matrices of odd sizes
        dict(name="madd_odd", kind="madd", dtype="f32", M=3001, N=4999),
        # four time steps on the paper's vector (Table 2): launches count
        dict(name="jacobi_32770", kind="jacobi", dtype="i32", N=2 ** 15 + 2, steps=4),
        # one division, the largest of the paper's Table 4
        dict(name="polydiv_32768", kind="polydiv", M=2 ** 15, K=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["matmul"] * 6 + ["grouped"] * 2 + ["transpose", "madd", "jacobi", "polydiv"])
    if kind == "matmul":
        dtype = rng.choice(["f32", "bf16", "i32"])
        most = {"f32": 1.9e11, "bf16": 2.5e11, "i32": 2.0e10}[dtype]  # below the largest listed product's time
        while True:
            M, N, K = (_log_int(rng, 64, 8192) for _ in range(3))
            if rng.random() < 0.4:  # rows of whole 16-byte chunks, as model dimensions usually are
                N, K = max(64, N // 8 * 8), max(64, K // 8 * 8)
            if 2.0 * M * N * K <= most:
                break
        return dict(kind=kind, dtype=dtype, M=M, N=N, K=K, pad=rng.choice([0, 0, 8]),
                    accumulate=rng.random() < 0.25)
    if kind == "grouped":
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), G=_log_int(rng, 32, 3000), lo=16,
                    hi=_log_int(rng, 64, 512), dims_seed=rng.randrange(1 << 20), pad=rng.choice([0, 8]))
    if kind in ("transpose", "madd"):
        return dict(kind=kind, dtype=rng.choice(["f32", "i32"]), M=_log_int(rng, 256, 14000),
                    N=_log_int(rng, 256, 14000))
    if kind == "jacobi":
        return dict(kind=kind, dtype=rng.choice(["f32", "i32"]), N=_log_int(rng, 2 ** 12, 2 ** 26),
                    steps=rng.randint(1, 31))
    return dict(kind=kind, M=_log_int(rng, 2 ** 9, 2 ** 16), K=_log_int(rng, 16, 1000))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _values(n, dtype, g):
    """n operand values: float32 uniform on [-1, 1), bfloat16 rounded from
    them, int32 over the whole range (sums wrap)."""
    if dtype == "i32":
        return torch.randint(-2 ** 31, 2 ** 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    x = torch.rand((n,), generator=g, device="cuda", dtype=torch.float32).mul_(2.0).sub_(1.0)
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _out_dtype(dtype):
    return torch.int32 if dtype == "i32" else torch.float32


def _rows(cols, pad):
    """Row stride of a matrix of `cols` columns (rows padded to `pad` elements, or packed)."""
    return -(-cols // pad) * pad if pad else cols


def _group_dims(case):
    r = random.Random(case["dims_seed"])
    return [tuple(_log_int(r, case["lo"], case["hi"]) for _ in range(3)) for _ in range(case["G"])]


def _group_views(case, flat_a, flat_b, flat_c):
    """The products' matrices: consecutive in three buffers, rows padded as
    the case says, each matrix starting at a multiple of 8 elements where
    rows are padded and right behind the one before otherwise."""
    As, Bs, Cs, at = [], [], [], [0, 0, 0]
    for M, N, K in _group_dims(case):
        for i, (flat, out, r, c) in enumerate(((flat_a, As, M, K), (flat_b, Bs, K, N), (flat_c, Cs, M, N))):
            ld = _rows(c, case["pad"])
            if flat is not None:
                out.append(flat[at[i]:at[i] + r * ld].view(r, ld)[:, :c])
            at[i] += r * ld
    return As, Bs, Cs, at


def _group_inputs(case, seed):
    na, nb, nc = _group_views(case, None, None, None)[3]
    g = _gen(seed)
    return _values(na, case["dtype"], g), _values(nb, case["dtype"], g), nc


def _matmul_inputs(case, seed):
    M, N, K, dt = case["M"], case["N"], case["K"], case["dtype"]
    g = _gen(seed)
    lda, ldb, ldc = _rows(K, case["pad"]), _rows(N, case["pad"]), _rows(N, case["pad"])
    A = _values(M * lda, dt, g).view(M, lda)[:, :K]
    B = _values(K * ldb, dt, g).view(K, ldb)[:, :N]
    if case["accumulate"]:
        C = _values(M * ldc, "i32" if dt == "i32" else "f32", g).view(M, ldc)[:, :N]
    else:
        C = torch.zeros((M, ldc), dtype=_out_dtype(dt), device="cuda")[:, :N]
    return A, B, C


def _residues(n, g):
    return torch.randint(0, MODULUS, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def prepare(case, seed):
    s = {"case": case, "table": _table()}
    kind = case["kind"]
    if kind == "matmul":
        s["A"], s["B"], s["C"] = _matmul_inputs(case, seed)
    elif kind == "grouped":
        a, b, nc = _group_inputs(case, seed)
        s["out"] = torch.zeros((nc,), dtype=torch.float32, device="cuda")
        As, Bs, Cs, _ = _group_views(case, a, b, s["out"])
        s["plan"] = pk.pk_grouped_plan_create(s["table"], case["dtype"], As, Bs, Cs)
    elif kind in ("transpose", "madd"):
        g = _gen(seed)
        M, N = case["M"], case["N"]
        s["A"] = _values(M * N, case["dtype"], g).view(M, N)
        if kind == "madd":
            s["B"] = _values(M * N, case["dtype"], g).view(M, N)
        s["C"] = torch.zeros((N, M) if kind == "transpose" else (M, N), dtype=_out_dtype(case["dtype"]), device="cuda")
    elif kind == "jacobi":
        s["a"] = _values(2 * case["N"], case["dtype"], _gen(seed))
    else:
        g = _gen(seed)
        s["dividend"] = _residues(case["M"] + case["K"], g)
        s["b"] = _residues(case["M"], g)
        s["a"] = torch.empty_like(s["dividend"])
    return s


def run(s):
    case, t = s["case"], s["table"]
    kind = case["kind"]
    if kind == "matmul":
        pk.pk_matmul(t, None, case["dtype"], s["A"], s["B"], s["C"], accumulate=case["accumulate"])
        return s["C"]
    if kind == "grouped":
        s["plan"].run()
        return s["out"]
    if kind == "transpose":
        pk.pk_transpose(t, None, case["dtype"], s["A"], s["C"])
        return s["C"]
    if kind == "madd":
        pk.pk_madd(t, None, case["dtype"], s["A"], s["B"], s["C"])
        return s["C"]
    if kind == "jacobi":
        pk.pk_jacobi1d(t, None, case["dtype"], s["a"], case["steps"])
        return s["a"]
    s["a"].copy_(s["dividend"])  # the division works in place: each one gets its dividend
    pk.pk_polydiv(t, None, s["a"], s["b"], MODULUS)
    return s["a"]


def work(case):
    kind = case["kind"]
    if kind == "matmul":
        M, N, K = case["M"], case["N"], case["K"]
        es = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": es * (M * K + K * N) + 4 * M * N * (2 if case["accumulate"] else 1), "flops": 2 * M * N * K}
    if kind == "grouped":
        es = 2 if case["dtype"] == "bf16" else 4
        d = np.array(_group_dims(case), dtype=np.float64)
        M, N, K = d[:, 0], d[:, 1], d[:, 2]
        return {"bytes": float((es * (M * K + K * N) + 4 * M * N).sum()), "flops": float((2 * M * N * K).sum())}
    if kind == "transpose":
        return {"bytes": 8 * case["M"] * case["N"], "flops": 0}
    if kind == "madd":
        return {"bytes": 12 * case["M"] * case["N"], "flops": case["M"] * case["N"]}
    if kind == "jacobi":  # the vector read once; one half's interior written, or both
        n = case["N"] - 2
        return {"bytes": (12 if case["steps"] > 1 else 8) * n, "flops": 3 * n * case["steps"]}
    # the dividend and the divisor read, the remainder and the zeros above it written
    return {"bytes": 4 * (2 * (case["M"] + case["K"]) + case["M"]), "flops": 2 * case["M"] * case["K"]}


def _wrapped_product(A, B):
    """A B modulo 2^32 for int32 A, B, exactly: 16-bit halves in float64,
    whose sums of K products stay below 2^53."""
    def halves(X):
        u = X.to(torch.int64) & 0xffffffff
        return (u & 0xffff).double(), (u >> 16).double()
    (al, ah), (bl, bh) = halves(A), halves(B)
    low = (al @ bl).to(torch.int64)
    mid = ((ah @ bl).to(torch.int64) + (al @ bh).to(torch.int64)) & 0xffff
    return (low + (mid << 16)) & 0xffffffff


def _as_int32(x):
    """int32 values of int64 residues modulo 2^32."""
    x = x & 0xffffffff
    return torch.where(x >= 2 ** 31, x - 2 ** 32, x).to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    if kind == "matmul":
        A, B, C = _matmul_inputs(case, seed)
        if case["dtype"] == "i32":
            p = _wrapped_product(A, B)
            return _as_int32(p + C.to(torch.int64) if case["accumulate"] else p)
        p = A.double() @ B.double()
        return p + C.double() if case["accumulate"] else p
    if kind == "grouped":
        a, b, nc = _group_inputs(case, seed)
        out = torch.zeros((nc,), dtype=torch.float64, device="cuda")
        As, Bs, Cs, _ = _group_views(case, a.double(), b.double(), out)
        for A, B, C in zip(As, Bs, Cs):
            C.copy_(A @ B)
        return out
    if kind in ("transpose", "madd"):
        g = _gen(seed)
        A = _values(case["M"] * case["N"], case["dtype"], g).view(case["M"], case["N"])
        if kind == "transpose":
            return A.t().contiguous() if case["dtype"] == "i32" else A.t().double()
        B = _values(case["M"] * case["N"], case["dtype"], g).view(case["M"], case["N"])
        return A.double() + B.double() if case["dtype"] == "f32" else _as_int32(A.to(torch.int64) + B.to(torch.int64))
    if kind == "jacobi" and case["dtype"] == "f32":
        a = _values(2 * case["N"], "f32", _gen(seed)).double().view(2, case["N"])
        for t in range(case["steps"]):
            src, dst = a[t % 2], a[(t + 1) % 2]
            dst[1:-1] = (src[:-2] + src[1:-1] + src[2:]) / 3.0
        return a.reshape(-1)
    return None  # whole numbers of a recurrence
