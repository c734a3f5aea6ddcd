"""The rules of plan.hpp that choose a kernel, at the sizes they were measured
at.  The header is compiled for the host."""

import os
import shutil
import subprocess

import pytest

from paper_1503_06189_amd import build

CXX = shutil.which("g++") or shutil.which("c++")


def evaluate(tmp_path, expressions):
    """The C++ expressions' values as integers, in order."""
    if CXX is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    lines = "".join(f'    printf("%lld\\n", (long long)({e}));\n' for e in expressions)
    src.write_text('#include <stdio.h>\n#include "plan.hpp"\nusing namespace xe;\n'
                   f"int main() {{\n{lines}}}\n")
    subprocess.run([CXX, "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [int(x) for x in out.split()]


# (inputs, channels, wide kernel): each side of the line, and sizes that bursts
# of flags cost the unit kernel up to twice as much
WIDE = [(16, 400, 0), (128, 4000, 0), (129, 128, 0), (129, 129, 1), (256, 64, 0), (256, 128, 0),
        (256, 129, 1), (256, 400, 1), (257, 56, 0), (257, 57, 1), (512, 32, 0), (512, 33, 1),
        (513, 5, 0), (513, 6, 1), (1000, 2, 0), (1000, 3, 1)]


def test_flag_counts(tmp_path):
    got = evaluate(tmp_path, [f"use_wide_flags({F}, {-(-N // 128)}, 256)" for N, F, _ in WIDE])
    assert got == [w for _, _, w in WIDE]


# (halves geometry, inputs, 4-byte aligned rows, longest chunk of the int8
# kernel in steps); frames of 25 to 40 steps were slower on the 6-bit kernel
SHORT = [(1, 64, 1, 64), (1, 127, 0, 64), (0, 100, 1, 40), (0, 132, 1, 40), (0, 130, 0, 40),
         (0, 192, 1, 40), (0, 193, 0, 32), (0, 250, 0, 32), (0, 256, 1, 32), (0, 257, 0, 24),
         (0, 260, 1, 40), (0, 384, 1, 40), (0, 388, 1, 32), (0, 512, 1, 32), (0, 512, 0, 24),
         (0, 576, 1, 40), (0, 580, 1, 32), (0, 768, 1, 32), (0, 772, 1, 24), (0, 1024, 1, 24),
         (0, 2048, 1, 24)]


def test_short_chunks(tmp_path):
    got = evaluate(tmp_path, [f"short_steps({s}, {N}, {a})" for s, N, a, _ in SHORT])
    assert got == [n for _, _, _, n in SHORT]
