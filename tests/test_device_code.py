"""Checks of the gfx950 code in the built library, read as assembly on the CPU."""
import os
import re
import subprocess

import pytest

from paper_2410_02425_amd import build

LLVM = "/opt/rocm/llvm/bin"


def gfx950_listing(name, tmp_path):
    """Instructions of a built object's gfx950 code, one string each."""
    obj, tool = os.path.join(build.BUILD, name + ".o"), os.path.join(LLVM, "llvm-objdump")
    if not (os.path.exists(obj) and os.path.exists(tool)):
        pytest.skip("no built object or no disassembler here")
    host = tmp_path / (name + ".o")
    host.write_bytes(open(obj, "rb").read())
    subprocess.run([tool, "--offloading", host.name], cwd=tmp_path, check=True, capture_output=True)
    code = [f for f in os.listdir(tmp_path) if f.startswith(name) and f.endswith("gfx950")]
    assert len(code) == 1, code
    text = subprocess.run([tool, "-d", "--no-show-raw-insn", "--no-leading-addr", code[0]], cwd=tmp_path, check=True,
                          capture_output=True, text=True).stdout
    return [line.split("//")[0].strip() for line in text.splitlines() if line.startswith("\t")]


def sgprs(operand):
    """The scalar registers that an operand names."""
    m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", operand.strip())
    if not m:
        return set()
    lo = int(m.group(1) or m.group(2))
    return set(range(lo, int(m.group(3) or lo) + 1))


@pytest.mark.parametrize("name", ["gemm", "attention"])
def test_loads_into_lds_keep_their_wait_states(name, tmp_path):
    """A load into LDS takes its LDS address from M0 and its base from scalar
    registers.  One wait state stands between a scalar write of M0 and the load,
    five between a vector instruction's write of the base and the load (an
    instruction counts one, s_nop n counts n + 1).  The compiler keeps both for
    loads of its own, but not for those in asm blocks."""
    code = gfx950_listing(name, tmp_path)
    loads = [i for i, ins in enumerate(code) if ins.startswith("global_load_lds")]
    assert len(loads) > 50
    for i in loads:
        base = sgprs(code[i].split(",")[-1].split()[0])
        waits, j = 0, i - 1
        while waits < 5 and j >= 0:
            op, _, args = code[j].partition(" ")
            dst = args.split(",")[0]
            assert waits >= 1 or dst != "m0", (i, code[j], code[i])
            assert not (op.startswith("v_") and sgprs(dst) & base), (i, waits, code[j], code[i])
            waits += int(args, 0) + 1 if op == "s_nop" else 1
            j -= 1
