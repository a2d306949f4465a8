"""Registers of the fp32 weight-gradient kernels: the main loop of an instance
whose registers spill to scratch memory waits for them every stage (the 128-row
groups of a 75 % selection lost a tenth of the backward call that way).  The
compiled code of every instance is listed and no block with matrix instructions
may read or write scratch memory.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_00512_amd", "csrc")


def spilling(asm):
    """(kernels, the scratch accesses of their blocks with bf16 matrix instructions)."""
    found, name, block, mfma, scratch = {}, None, None, 0, 0

    def end():
        if name and mfma:
            found[name] = found.get(name, 0) + scratch
    for line in asm.splitlines():
        ins = line.split(";")[0].strip()
        label = re.match(r"(\w+|\.LBB\w+):$", ins)
        if label:
            end()
            mfma = scratch = 0
            if not label.group(1).startswith(".L"):
                name = label.group(1)
        mfma += ins.startswith("v_mfma_f32_32x32x16_bf16")
        scratch += ins.startswith("scratch_")
    end()
    return found


def test_checker():
    k = "_Zk:\n.LBB0_1:\n%s v_mfma_f32_32x32x16_bf16 a, b\n.LBB0_2:\n scratch_load_dword v1\n"
    assert spilling(k % "") == {"_Zk": 0} and spilling(k % " scratch_load_dword v2\n") == {"_Zk": 1}


def test_no_scratch_in_the_main_loop(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "w.s"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-S",
                    "--cuda-device-only", os.path.join(CSRC, "wgrad_f32.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    found = spilling(out.read_text())
    assert len(found) == len(set(found)) >= 30
    bad = {k: n for k, n in found.items() if n}
    assert not bad, bad
