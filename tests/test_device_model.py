"""The product kernels themselves, run on the CPU (tests/hipsim/device): the
sources are built by the host compiler against a stand-in for the device
language, in which a work-item is a fiber, wavefront operations are rendezvous
of 64 of them, LDS starts out as garbage and copies into LDS land only when a
wait requires it (or, in a second run with the wavefronts in the opposite order,
at once).  With the address sanitizer on every operand, result and LDS array
an access out of bounds, a missing wait or barrier, or a barrier that not every
wavefront reaches fails here, as does a wrong sum.

Every tile and mode of the bf16 large-tile products and the fp32 products and
weight gradient, with rows, columns and contraction lengths that end inside a
tile, one, two and more stages, and refills of the gathered-row table.  The
sums are those of the fp32 accumulators: relative errors of some 1e-7.
"""
import json
import os
import shutil
import subprocess
import sys

import pytest

DEVICE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hipsim", "device")
CLANG = "/opt/rocm/llvm/bin/clang++"

BIG = [
    dict(mode="dense", tm=256, tn=256, M=264, N=136, rows=128),
    dict(mode="dense", tm=128, tn=256, M=136, m_begin=8, N=264, rows=256, splitk=2, steps=2),
    dict(mode="gather", tm=256, tn=256, M=72, N=136, rows=2560, kept=2176),   # table refill
    dict(mode="gather", tm=128, tn=256, M=72, N=136, rows=256, kept=192, steps=2),
    dict(mode="sel", tm=128, tn=256, M=136, m_begin=64, N=136, rows=768, splitk=2),
    dict(mode="sel", tm=256, tn=256, M=72, m_begin=8, N=136, rows=512, P=16),
    dict(mode="rowa", tm=128, tn=256, M=130, N=136, rows=192, kcol0=64, splitk=3),
    dict(mode="rowa", tm=256, tn=256, M=70, N=264, rows=320),
    dict(mode="rowa", tm=128, tn=256, M=70, N=136, rows=256),
]
F32 = [
    dict(mode="dense", tm=128, tn=128, M=136, m_begin=5, N=130, rows=75),
    dict(mode="gather", tm=128, tn=32, M=60, N=31, rows=3000, kept=2304),     # table refill
    dict(mode="gather", tm=64, tn=64, M=66, N=66, rows=80, kept=52, steps=2),
    dict(mode="sel", tm=64, tn=64, M=90, m_begin=21, ldw=91, N=68, rows=192, splitk=2),
    dict(mode="sel", tm=128, tn=128, M=90, m_begin=20, N=68, rows=256, P=16),
    dict(mode="rowa", tm=128, tn=128, M=70, N=130, rows=131, kcol0=13, splitk=2),
    dict(mode="rowa", tm=64, tn=64, M=70, N=66, rows=72),
    dict(mode="rowa", tm=128, tn=32, M=130, N=20, rows=140, kcol0=2, splitk=3),
    dict(mode="fine", tm=0, tn=0, M=100, m_begin=64, N=96, rows=128, kept=1, splitk=2),
]
COARSE, FINE = dict(P=4, R=8), dict(P=4, R=8, S=0)
WGRAD = [
    dict(T=2, B=20, I=30, H=33, S=4, **COARSE),
    dict(T=3, B=18, I=66, H=70, S=6, cut=1, **COARSE),           # two launches
    dict(T=1, B=33, I=40, H=66, S=0, **COARSE),
    dict(T=2, B=40, I=20, H=32, P=16, R=8, S=4),
    dict(T=2, B=64, I=40, H=32, fine=1, **FINE),
    # a removed block of an infinite feature stays out of the fp32 recomputation
    dict(T=2, B=64, I=40, H=32, fine=1, infs=[[0, 3, 40], [1, 7, 2]], **FINE),
]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(CLANG) or shutil.which("ld") is None or not os.path.isdir(DEVICE):
        pytest.skip("no host clang++, or a tree without the stand-in's sources")
    sys.path.insert(0, DEVICE)
    import build as devbuild
    return devbuild.build(str(tmp_path_factory.mktemp("devsim")),
                          ["gemm1_big.hip", "gemm1.hip", "gemm1_f32.hip", "wgrad_f32.hip", "wgrad_bf16.hip"],
                          opt=("-O1", "-O0"))


def run(lib, cases):
    asan = subprocess.run([CLANG, "-print-file-name=libclang_rt.asan-x86_64.so"],
                          capture_output=True, text=True, check=True).stdout.strip()
    env = dict(os.environ, LD_PRELOAD=asan, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    r = subprocess.run([sys.executable, os.path.join(DEVICE, "products.py"), lib], env=env, text=True,
                       input="".join(json.dumps(c) + "\n" for c in cases), capture_output=True, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    out = [json.loads(l[3:]) for l in r.stdout.splitlines() if l.startswith("ok ")]
    assert len(out) == len(cases)
    for c, o in zip(cases, out):
        assert o.get("out", 0) <= 1e-6 and o.get("dW", 0) <= 1e-6, (c, o)


def test_large_tile_products(lib):
    run(lib, [dict(c, bf16=True) for c in BIG])


def test_f32_products(lib):
    run(lib, [dict(c, bf16=False) for c in F32])


def test_f32_weight_gradient(lib):
    run(lib, [dict(c, bf16=False) for c in WGRAD])


# operands near either end of fp32's range (the products are far from both):
# all 24 bits count (2^-118, and denormal values), and those that scaling or its
# sums take to infinity are computed again
@pytest.mark.parametrize("scale,wscale", [(2.0 ** -118, 2.0 ** 40), (2.0 ** 30, 2.0 ** -118),
                                          (2.0 ** -134, 2.0 ** 60), (2.0 ** 104, 2.0 ** -90),
                                          (2.0 ** 45, 2.0 ** 45), (2.0 ** -130, 2.0 ** 110)])
def test_f32_range(lib, scale, wscale):
    run(lib, [dict(c, bf16=False, scale=scale, wscale=wscale) for c in (F32[2], F32[6], WGRAD[1], WGRAD[2])])


def test_model_sees_mistakes(lib):
    # a result one row short, and a table entry past W: planted in the arguments
    for bad in (dict(F32[0], bf16=False, short=1), dict(F32[2], bf16=False, wild=1)):
        with pytest.raises(AssertionError, match="AddressSanitizer"):
            run(lib, [bad])
