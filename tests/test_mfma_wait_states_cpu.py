"""Wait states before the matrix instruction that is written as inline assembly.

A matrix instruction may read a vector register no earlier than 2 wait states
after a vector instruction wrote it.  The compiler keeps this distance for its
builtins but does not look into inline assembly, and a schedule that breaks it
may still give exact results.  So the device code of the built library is
disassembled and the instructions before each one are checked.
"""

import os
import re
import subprocess

import pytest

from paper_1503_06189_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin")
if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
    LLVM = "/opt/rocm/llvm/bin"
OPCODE = "v_mfma_f32_16x16x128_f8f6f4"
WAIT_STATES = 2


def _registers(operand):
    """Vector registers of an operand, as a set of numbers."""
    m = re.match(r"v\[(\d+):(\d+)\]$", operand) or re.match(r"v(\d+)()$", operand)
    return set(range(int(m[1]), int(m[2] or m[1]) + 1)) if m else set()


def _parse(line):
    text = line.split("//")[0].strip()
    op, _, rest = text.partition(" ")
    return op, [x.split()[0] for x in rest.split(", ") if x.strip()]


def violations(lines):
    """(reads, number of them that come too early) of OPCODE in a disassembly."""
    code = [_parse(x) for x in lines if x.startswith("\t")]
    found, early = 0, []
    for k, (op, args) in enumerate(code):
        if op != OPCODE:
            continue
        found += 1
        reads = set().union(*(_registers(a) for a in args[1:4]))
        waited, j = 0, k - 1
        while waited < WAIT_STATES and j >= 0:
            prev, p = code[j]
            if prev == "s_nop":
                waited += int(p[0], 0) + 1
            else:
                if prev.startswith("v_") and not prev.startswith("v_mfma"):
                    wrote = _registers(p[0])
                    if "swap" in prev:
                        wrote |= _registers(p[1])
                    if wrote & reads:
                        early.append((k, prev, p))
                if prev.startswith(("s_branch", "s_cbranch")):
                    # other paths may join here: only the s_nop covers them all
                    early.append((k, prev, p))
                waited += 1
            j -= 1
    return found, early


def test_checker_sees_an_early_read():
    ok = ["\tv_mov_b32_e32 v107, v108", "\ts_nop 1", f"\t{OPCODE} v[104:107], v[96:99], v[44:49], v[104:107] cbsz:4 blgp:2"]
    assert violations(ok) == (1, [])
    assert len(violations([ok[0], ok[2]])[1]) == 1
    assert len(violations([ok[0], "\ts_nop 0", ok[2]])[1]) == 1
    assert violations(["\tv_mov_b32_e32 v1, v108", ok[2]]) == (1, [])


def test_no_source_is_written_just_before(tmp_path):
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build()
    run = lambda tool, *a: subprocess.run([os.path.join(LLVM, tool), *a], check=True,
                                          capture_output=True, text=True).stdout
    fat, obj = str(tmp_path / "fatbin"), str(tmp_path / "device.o")
    run("llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", build.LIB, str(tmp_path / "copy.so"))
    run("clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
        f"--input={fat}", f"--output={obj}")
    found, early = violations(run("llvm-objdump", "-d", "--no-show-raw-insn", obj).splitlines())
    assert found > 0
    assert early == [], early[:5]
