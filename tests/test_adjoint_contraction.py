"""Multiply-adds of the adjoint kernels are fused only where the source says so.

The one-kernel and the two-kernel form of a reversed stage promise the same bits
though the compiler sees the same expressions in different surroundings.  That
holds by construction only if no multiplication leaves the front end marked as
free to fuse with an addition of another statement: those the front end fuses
itself, within one expression, become fmuladd and are the same in every kernel."""
import os
import re
import subprocess

from paper_2106_07694_amd import build

def test_no_multiplication_of_the_adjoint_is_free_to_fuse(tmp_path):
    out = str(tmp_path / "adjoint.ll")
    subprocess.run([build.HIPCC, *build.COMMON, "-x", "hip", "--cuda-device-only", "-S", "-emit-llvm", "-Xclang",
                    "-disable-llvm-passes", os.path.join(build.CSRC, "adjoint.hip"), "-o", out],
                   check=True, capture_output=True)
    where, free, fused = "", set(), 0
    for line in open(out):
        m = re.match(r"define .*?@(\w+)\(", line)
        where = m.group(1) if m else where
        if re.search(r"= fmul\b.*\bcontract\b", line):
            free.add(where)
        fused += "@llvm.fmuladd" in line
    assert fused > 0
    assert not free, sorted(free)
