"""Builds the library's kernels and host driver for the CPU stand-in of the
device (devsim.cpp): the sources as they are, but for the few constructs that a
host compiler cannot take (inline assembly, LDS declarations)."""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(os.path.dirname(HERE)))
CSRC = os.path.join(ROOT, "paper_1806_00512_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def host_source(text):
    text = re.sub(r"extern __shared__[^;]*\bsmem\[\];", "unsigned char *smem = sim::dynamic_lds();", text)
    text = re.sub(r"^(\s*)(__shared__ [^;]*?(\w+)(?:\[[^;]*\])?);",
                  r"\1\2; sim::lds(&\3, sizeof(\3));", text, flags=re.M)
    text = re.sub(r'asm volatile\("s_mov_b32 m0[^"]*(global_load_lds_dword|buffer_load_dword)(x4)?[^;]*?\);',
                  lambda m: "(void)lds; " + (
                      "sim::copy_rsrc((const int *)&rsrc, voff, soff, (void *)lds_dst, 16);"
                      if m[1].startswith("buffer") else
                      "sim::copy(gsrc, (void *)lds_dst, %d);" % (16 if m[2] else 4)), text)
    text = re.sub(r"__builtin_amdgcn_readfirstlane\(\(int\)\(uintptr_t\)lds_dst\)", "0", text)
    text = re.sub(r'asm volatile\("s_waitcnt lgkmcnt\(0\)\\n\\ts_barrier" ::: "memory"\);',
                  "sim::barrier();", text)
    text = re.sub(r'asm volatile\("(s_waitcnt lgkmcnt\(0\))?" ::: "memory"\);', "sim::wave_sync();", text)
    assert "asm volatile" not in re.sub(r"//[^\n]*", "", text)
    return text


def build(out, sources, sanitize=True, opt=("-O1",)):
    """out: a folder; opt: optimisation levels of the sources (the last one
    holds for the rest); returns the path of the shared library built in it."""
    src = os.path.join(out, "paper_1806_00512_amd", "csrc")
    os.makedirs(src, exist_ok=True)
    for f in os.listdir(CSRC):
        with open(os.path.join(CSRC, f)) as g:
            text = g.read()
        with open(os.path.join(src, f), "w") as g:
            g.write(host_source(text))
    inc = os.path.join(out, "include")
    if not os.path.exists(inc):
        os.symlink(os.path.join(ROOT, "include"), inc)
    flags = [CLANG, "-x", "c++", "-std=c++17", "-g1", "-fPIC", "-ffp-contract=off", "-w",
             "-fno-strict-aliasing", "-I" + HERE, "-I" + inc]
    if sanitize:
        flags += ["-fsanitize=address", "-fno-omit-frame-pointer", "-shared-libasan"]
    jobs, objs = [], []
    for i, f in enumerate(sources + [os.path.join(HERE, "devsim.cpp")]):
        obj = os.path.join(out, os.path.basename(f) + ".o")
        objs.append(obj)
        level = "-O1" if i == len(sources) else opt[min(i, len(opt) - 1)]
        jobs.append(subprocess.Popen(flags + [level, "-c", os.path.join(src, f), "-o", obj]))
    if any([j.wait() for j in jobs]):
        raise RuntimeError("build failed")
    lib = os.path.join(out, "liblstmss_devsim.so")
    subprocess.run([CLANG, "-shared", "-o", lib] + objs + (["-fsanitize=address", "-shared-libasan"] if sanitize else []),
                   check=True)
    return lib


ALL = ["lstmss_api.cpp", "cell.hip", "gemm1.hip", "gemm1_big.hip", "gemm1_f32.hip", "wgrad_f32.hip",
       "wgrad_bf16.hip", "gemm.hip", "train.hip", "bidir.hip"]

if __name__ == "__main__":
    print(build(sys.argv[1], ALL))
