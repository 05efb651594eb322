"""Host rules of a product's launch that no entry point shows, called in the
library itself by a small program compiled here (no GPU)."""
import os
import subprocess

import pytest

from paper_1801_04348_amd import build
from tests import machines

PRELUDE = r"""
#include <cstdio>
#include <cstring>
#include "select.hpp"
using namespace pk;
static pk_machine machine() {
    pk_machine m{};
    %s
    return m;
}
"""


def run(tmp_path, body, machine):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    sets = "\n".join('std::strcpy(m.%s, "%s");' % (k, v) if isinstance(v, str) else "m.%s = %d;" % (k, v)
                     for k, v in machine.as_dict().items())
    src, exe = str(tmp_path / "rules.cpp"), str(tmp_path / "rules")
    with open(src, "w") as f:
        f.write(PRELUDE % sets + body)
    cmd = [build.HIPCC] + build.COMMON + [src, "-o", exe, "-L" + build.PKG, "-l:" + os.path.basename(build.LIB), "-Wl,-rpath," + build.PKG]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stderr[-4000:]
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=60)
    assert p.returncode == 0, p.stderr[-2000:]
    return [x.split() for x in p.stdout.splitlines()]


DEPTHS = r"""
int main() {
    const pk_machine m = machine();
    for (const auto &e : registry()) {
        if (e.family != PK_FAMILY_MFMA || (e.variant & (PK_MFMA_GROUPED | PK_MFMA_ELEMENT)) || e.dtype == PK_I32) continue;
        int extra = -1;
        const int depth = dma_depth(m, e, 1, 1000, &extra);
        std::printf("%s %d %d %d\n", e.name, depth, extra, e.lds_bytes);
    }
}
"""


def test_no_lds_is_added_to_programs_that_load_through_registers(tmp_path):
    """The programs of 1024 work-items, and the single-stage bfloat16 ones of
    K tile 32 (half a step is less than one group of products), load through
    registers: they read no third buffer, so a launch adds no LDS for one."""
    rows = run(tmp_path, DEPTHS, machines.gfx950())
    registers = [r for r in rows if "_w4x4" in r[0] or ("bf16" in r[0] and "x32_w" in r[0] and "_st1" in r[0])]
    direct = [r for r in rows if r not in registers]
    assert len(registers) >= 6 and any(int(r[1]) == 4 for r in direct)
    assert all(r[1:3] == ["2", "0"] for r in registers), registers


def test_added_lds_fits_the_hardware_whatever_the_descriptor_says(tmp_path):
    """A table may be bound to the descriptor of a machine with more LDS than
    gfx950's 160 KiB a workgroup: every program's launch stays within those."""
    rows = run(tmp_path, DEPTHS, machines.variant(lds_block=1 << 20, lds_cu=1 << 20))
    assert any(int(r[2]) > 0 for r in rows)
    assert all(int(r[2]) + int(r[3]) <= 160 * 1024 for r in rows), [r for r in rows if int(r[2]) + int(r[3]) > 160 * 1024]


WIDE = r"""
int main() {
    // reads "M K lda ldb" lines' worth of a fixed list; operands at aligned addresses
    const int64_t cases[][4] = {%s};
    for (const auto &e : registry()) {
        if (e.family != PK_FAMILY_MFMA || (e.variant & (PK_MFMA_GROUPED | PK_MFMA_ELEMENT | PK_MFMA_SPLIT)) || e.dtype == PK_I32)
            continue;
        std::printf("%%s %%d %%d %%d", e.name, e.tile_m, e.bk, e.dtype == PK_BF16 ? 2 : 4);
        for (const auto &c : cases)
            std::printf(" %%d", (int)wide_rows(e, c[0], c[1], (void *)4096, c[2], (void *)8192, c[3]));
        std::printf("\n");
    }
}
"""


def test_row_strides_that_direct_loads_reach(tmp_path):
    """A program that loads straight to LDS is wide while the last byte of a
    tile's rows lies within 32 bits of its first, whatever the matrix's other
    rows; one that loads through registers, on any stride."""
    cases = [(M, K, lda, ldb) for M in (1, 2, 64, 100, 256, 5000) for K in (1, 20, 64, 5000)
             for lda, ldb in ((8192, 8192), (1 << 40, 64), (64, 1 << 40), (4000000, 4000000), (17000000, 64),
                              (34000000, 64), (64, 34000000), (64, 69000000), (128000000, 128000000))]
    body = WIDE % ", ".join("{%dLL, %dLL, %dLL, %dLL}" % c for c in cases)
    rows = run(tmp_path, body, machines.gfx950())
    assert len(rows) >= 40
    for name, bm, bk, es, *wide in rows:
        bm, bk, es = int(bm), int(bk), int(es)
        buffer = bk // 2 if name.endswith("_st1") else bk
        registers = "_w4x4" in name or (es == 2 and bk == 32 and name.endswith("_st1"))
        for (M, K, lda, ldb), w in zip(cases, wide):
            span = max((min(M, bm) - 1) * lda, (min(K, buffer) - 1) * ldb) * es
            assert int(w) == (registers or span + 4096 <= 2 ** 32), (name, M, K, lda, ldb)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_choice_on_long_aligned_rows(dtype):
    """Rows of 9 to 30 MB that direct loads reach change nothing in the choice
    (operand addresses are not read): it is that of short ones."""
    from paper_1801_04348_amd import pk
    import ctypes
    tbl = pk.pk_case_table_build(-1, machines.gfx950())
    es = 2 if dtype == "bf16" else 4

    def pick(M, N, K, lda, ldb):
        out = pk.pk_params()
        pk._check(pk.lib().pk_select_operands(tbl.handle, pk._dt(dtype), ctypes.c_void_p(4096), lda,
                                              ctypes.c_void_p(8192), ldb, M, N, K, pk.PK_POLICY_CASE,
                                              ctypes.byref(out)))
        return out.as_dict() if hasattr(out, "as_dict") else bytes(out)

    for M, N, K in [(1, 64, 512), (64, 64, 4096), (100, 1000, 300), (1000, 256, 512), (2048, 2048, 1024), (4096, 640, 2048)]:
        for mb in (9, 16):
            ld = mb * 1000000 // es // 8 * 8
            assert pick(M, N, K, ld, ld) == pick(M, N, K, max(K, 8) // 8 * 8 + 8, N // 8 * 8 + 8), (M, N, K, mb)


@pytest.mark.parametrize("dtype,M,N,K", [
    ("i32", 59, 8140, 2164), ("i32", 6, 4744, 5632), ("i32", 25, 4256, 2640), ("i32", 23, 2336, 7816),
    ("i32", 3, 2936, 4336), ("i32", 6943, 27, 6782), ("i32", 3213, 9, 6520), ("i32", 53, 1008, 4614),
    ("f32", 8141, 6355, 15), ("f32", 7692, 6808, 18), ("f32", 3616, 3576, 4), ("f32", 1224, 6884, 21)])
def test_thin_products_run_on_the_matrix_cores(dtype, M, N, K):
    """Products with a dimension below 64 whose fastest VALU program takes 1.3
    to 4 times the fastest MFMA program's time (timed on gfx950)."""
    from paper_1801_04348_amd import pk
    tbl = pk.pk_case_table_build(-1, machines.variant(regs_block=65536, regs_cu=65536, max_blocks_cu=2))
    assert pk.pk_select(tbl, dtype, M, N, K).family == pk.PK_FAMILY_MFMA


@pytest.mark.parametrize("dtype,M,N,K", [
    ("f32", 179, 2, 1), ("f32", 31, 123, 1), ("f32", 5, 9, 3), ("f32", 67, 25, 8), ("f32", 2071, 4, 1),
    ("f32", 1307, 13, 13), ("i32", 1922, 8, 48), ("i32", 434, 16, 48), ("i32", 70, 36, 43)])
def test_smallest_products_run_on_valu_programs(dtype, M, N, K):
    """Products of a few loads a lane, whose fastest MFMA program takes 1.3 to
    1.6 times the fastest VALU program's time (timed on gfx950 in a graph)."""
    from paper_1801_04348_amd import pk
    tbl = pk.pk_case_table_build(-1, machines.variant(regs_block=65536, regs_cu=65536, max_blocks_cu=2))
    assert pk.pk_select(tbl, dtype, M, N, K).family != pk.PK_FAMILY_MFMA
