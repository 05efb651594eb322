"""What the compiler makes of the kernels that load straight to LDS: facts
their inline assembly and their LDS addresses rely on, read from the code of
small instances compiled here (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_1801_04348_amd import build

KERNELS = """
#include "kernels/mfma.hpp"
extern "C" __global__ void __launch_bounds__(256) deep_bf16(pkk::MmArgs a) { pkk::mfma_bf16<64, 64, 64, 2, 2, 2>(a); }
extern "C" __global__ void __launch_bounds__(256) two_f32(pkk::MmArgs a) { pkk::mfma_f32<64, 64, 32, 2, 2, 2>(a); }
"""


def device_code(tmp_path, *flags, source=KERNELS):
    """The compiler's text output for `source`, with the build's own flags."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, out = str(tmp_path / "kernels.hip"), str(tmp_path / "kernels.out")
    with open(src, "w") as f:
        f.write(source)
    cmd = [build.HIPCC] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S", *flags, src, "-o", out]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert p.returncode == 0, p.stderr[-4000:]
    with open(out) as f:
        return f.read()


def test_direct_loads_read_a_base_the_scalar_unit_wrote(tmp_path):
    """A load right behind a vector instruction that wrote its scalar base
    would read the old value, and the compiler puts no wait inside inline
    assembly: the base is a copy made between the write of m0 and the load."""
    lines = [x.split(";")[0].strip() for x in device_code(tmp_path).splitlines()]
    loads = [i for i, x in enumerate(lines) if x.startswith("global_load_lds_dwordx4")]
    assert len(loads) >= 8
    for i in loads:
        base = re.search(r"(s\[\d+:\d+\])$", lines[i]).group(1)
        assert lines[i - 1].startswith("s_mov_b64 " + base + ","), lines[i - 2:i + 1]
        assert lines[i - 2].startswith("s_mov_b32 m0,"), lines[i - 2:i + 1]


def test_direct_loads_say_that_they_write_m0(tmp_path):
    asm = re.findall(r'asm sideeffect "[^"]*global_load_lds_dwordx4[^"]*", "([^"]*)"',
                     device_code(tmp_path, "-emit-llvm"))
    assert asm and all("~{m0}" in c for c in asm)


def test_no_address_past_the_end_of_an_lds_object(tmp_path):
    """The third and fourth buffers of K steps lie in LDS that the launch adds
    behind the kernel's own array: not addressed from that array, of which
    they are out of bounds."""
    ir = device_code(tmp_path, "-emit-llvm")
    size = {n: int(b) for n, b in re.findall(r"^(@\S+) = .*addrspace\(3\) global \[(\d+) x i8\]", ir, re.M)}
    assert len(size) == 2
    reached = [(n, int(off)) for n, off in re.findall(r"addrspace\(3\) (@\w+), i32 (\d+)", ir) if n in size]
    assert reached and all(off < size[n] for n, off in reached), max(off for _, off in reached)


@pytest.mark.parametrize("kernel", [
    "mfma_f32<64, 64, 32, 2, 2, 2>", "mfma_bf16<64, 64, 64, 2, 2, 2>", "mfma_bf16<256, 128, 32, 2, 2, 2>"])
def test_accumulation_loads_several_rows_at_once(tmp_path, kernel):
    """C += A B reads C ahead of its stores: a load per row behind the row
    before's store would take a trip to memory for each."""
    code = device_code(tmp_path, source="""
#include "kernels/mfma.hpp"
extern "C" __global__ void __launch_bounds__(256) k(pkk::MmArgs a) { pkk::%s(a); }
""" % kernel)
    # single words are loaded from C alone; (a batch's last may stand out of line)
    ops = re.findall(r"^\s+(global_load_dword|global_store_dword|s_waitcnt vmcnt)\b", code, re.M)
    runs = re.findall("L+", "".join("L" if o == "global_load_dword" else "." for o in ops))
    assert max(map(len, runs)) >= 3
