"""The wait state between a scalar write of m0 and the LDS copy that reads it.

gfx950 needs one between the two (the compiler supplies it for its own
copies, but not inside an asm string).  The copy helpers of gemm_common.h are
compiled in a kernel of their own and every copy of the listing is checked; no
other source issues such copies from inline assembly.
"""
import glob
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_00512_amd", "csrc")

KERNEL = """
#include "gemm_common.h"
namespace lstmss {
__global__ void copies(const char *p, int n, int *out) {
    __shared__ int a[1024];
    const int lane = threadIdx.x;
    dma16(p + 16 * lane, (lds_void_t *)&a[0]);
    dma4(p + 4 * lane, (lds_void_t *)&a[256 * n]);
    dma16_buf(buf_rsrc(p, ~0u), 16 * lane, 0, (lds_void_t *)&a[512]);
    dma16_buf(buf_rsrc(p + 64, ~0u), 16 * lane, n, (lds_void_t *)&a[768]);
    __builtin_amdgcn_s_waitcnt(0);
    lds_barrier();
    out[lane] = a[lane];
}
}
"""


def unprotected(asm):
    """(copies, copies that follow a write of m0 at once) of a listing."""
    copies, bad, prev = 0, [], ""
    for line in asm.splitlines():
        ins = line.split(";")[0].strip()
        if not ins or ins.startswith(".") or ins.endswith(":"):
            continue
        if re.match(r"(global|buffer|scratch)_load", ins) and re.search(r"\blds\b|_lds_", ins):
            copies += 1
            if re.match(r"s_\w+ m0,", prev):
                bad.append(ins)
        prev = ins
    return copies, bad


def test_checker():
    m0, cp = "s_mov_b32 m0, s1\n", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds\n"
    assert unprotected(m0 + cp)[1] and not unprotected(m0 + "s_nop 0\n" + cp)[1]


def test_copies_wait_for_m0(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, out = tmp_path / "copies.hip", tmp_path / "copies.s"
    src.write_text(KERNEL)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", CSRC, "-S",
                    "--cuda-device-only", str(src), "-o", str(out)], check=True, capture_output=True)
    copies, bad = unprotected(out.read_text())
    assert copies == 4 and not bad, bad


def test_no_other_asm_copies():
    for f in glob.glob(os.path.join(CSRC, "*")):
        text = re.sub(r"//[^\n]*", "", open(f).read())
        for ins in re.findall(r'asm\s+volatile\s*\((.*?)\);', text, re.S):
            if "lds" in ins.split(":")[0]:
                assert os.path.basename(f) == "gemm_common.h", (f, ins)
