"""The inline-asm blocks of row_bcast.h and cn_stencil.h write some operands
before they have read all the others.  Compiled (no GPU) with an input that
holds the same value as such an operand -- a row passed as halo and as chunk
row, a chain's start among its states -- a block must still name a register
pair for each operand: two in one pair would read the overwritten value."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_05395_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

KERNEL = """#include "cn_stencil.h"
using namespace bb;
__global__ void block(double *p, const double *z, StencilRhs<1, true> w3, StencilRhs<2, true> w5)
{
    double v[16], c[8];
    for (int t = 0; t < 16; ++t) v[t] = p[t * 64 + threadIdx.x];
    for (int t = 0; t < 8; ++t) c[t] = z[t * 64 + threadIdx.x];
    %s
    for (int t = 0; t < 16; ++t) p[t * 64 + threadIdx.x] = v[t];
}
"""
SPLIT = "double e[4], g[4], m1[1] = {c[0]}, m2[4] = {c[0], c[1], c[2], c[3]};" \
        "for (int t = 0; t < 4; ++t) { e[t] = v[t]; g[t] = v[4 + t]; }"
JOIN = "for (int t = 0; t < 4; ++t) { v[t] = e[t]; v[4 + t] = g[t]; }"
# statement, vector operands of the block (its temporaries included)
BLOCKS = {
    "ends1": ("double e = v[3], o = c[2]; rows8_ends<0, 16>(v, e, o, c[0], c[1]); v[0] = e; v[1] = o;", 12),
    "ends2": ("double e = v[3], o = v[7], f = c[4], q = c[5];"
              "rows8_ends<0, 16>(v, e, o, f, q, c[0], c[1], c[2], c[3]); v[0] = e + o; v[1] = f + q;", 16),
    "forward1": ("rows8_forward<0, 16>(v, v[7], c[0], c[1]);", 13),
    "forward2": ("rows8_forward<0, 16>(v, v[7], v[6], c[0], c[1], c[2]);", 15),
    "backward1": ("rows8_backward<0, 16>(v, v[0], c[0]);", 10),
    "backward2": ("rows8_backward<0, 16>(v, v[0], v[1], c[0], c[1]);", 12),
    "correct1": ("rows8_correct<0, 16>(v, v[3], c[0]);", 10),
    "correct2": ("rows8_correct<0, 16>(v, v[3], v[5], c[0], c[1]);", 12),
    "up1": (SPLIT + "chain4<1, true, 0>(e, g, m1, e[3], 0.0);" + JOIN, 6),
    "down2": (SPLIT + "chain4<2, false, 4>(e, g, m2, e[0], g[0]);" + JOIN, 14),
    "stencil1": ("double s = c[0]; stencil_rows8(v, v[0], s, w3.w); v[8] = s;", 14),
    "stencil2": ("double s = c[0], u = c[1]; stencil_rows8(v, v[0], v[1], s, u, w5.w); v[8] = s; v[9] = u;", 16),
}


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)), reason="no hipcc")
@pytest.mark.parametrize("name", sorted(BLOCKS))
def test_each_operand_has_its_own_registers(tmp_path, name):
    stmt, operands = BLOCKS[name]
    src, out = tmp_path / "block.hip", tmp_path / "block.s"
    src.write_text(KERNEL % stmt)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    "-x", "hip", "--offload-device-only", "-S", str(src), "-o", str(out)],
                   check=True, capture_output=True)
    blocks = re.findall(r"#ASMSTART\n(.*?)#ASMEND", out.read_text(), re.S)
    block = [b for b in blocks if "v_fma" in b or "v_fmac" in b]
    assert len(block) == 1
    assert len(set(re.findall(r"v\[\d+:\d+\]", block[0]))) == operands
