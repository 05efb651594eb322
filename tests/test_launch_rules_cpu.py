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
