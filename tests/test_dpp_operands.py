"""Registers of the multiply-adds with a broadcast operand (csrc/tridiag.h): several instructions in one statement of inline
assembly, so none of its results may share a register with an operand that a later one still reads, also where the compiler
knows that both hold the same value before.  Read off the assembly of a kernel in which they do; nothing runs."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_02561_amd", "csrc")
SOURCE = """
#include "tridiag.h"
__global__ void four(const double* in, double* out) {
    const double v = in[threadIdx.x];
    double a = v, b = v, c = v, d = v;
    solar::fmac_bcast64<3>(a, b, c, d, v, v);
    out[threadIdx.x] = (a + b) + (c + d);
}
__global__ void sum(const double* in, double* out) {
    const double v = in[threadIdx.x], w = in[threadIdx.x + 64];
    double p = v;
    solar::fmac_bcast64_sum<3>(p, w, w, v, v, v);
    out[threadIdx.x] = p;
}
__global__ void sum_x(const double* in, double* out) {
    const double v = in[threadIdx.x], w = in[threadIdx.x + 64];
    double p = v;
    solar::fmac_bcast64_sum<3>(p, v, w, w, w, w);
    out[threadIdx.x] = p;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_results_do_not_overlap_later_operands(tmp_path):
    src, asm = tmp_path / "operands.hip", tmp_path / "operands.s"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-S", "-I", CSRC,
                    str(src), "-o", str(asm)], check=True, capture_output=True)
    blocks = re.findall(r"#ASMSTART\n(.*?)#ASMEND", asm.read_text(), re.S)
    groups = [re.findall(r"v_fmac_f64_dpp (\S+), (\S+), (\S+) ", b) for b in blocks]
    groups = [g for g in groups if g]
    assert [len(g) for g in groups] == [4, 4, 4]
    for g in groups:
        for i, (dst, _, _) in enumerate(g):
            later = {o for _, x, y in g[i + 1:] for o in (x, y)}
            assert dst not in later, g
