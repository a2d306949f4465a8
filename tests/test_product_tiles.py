"""The tile each product of the large-tile tests is meant to take, from the
library's own rule (host code, no GPU)."""
import ctypes

import pytest

import paper_1806_00512_amd.lstmss as lstmss
from test_gpu_gemm_big import CASES


def tile(columns, rows, launches):
    lib = ctypes.CDLL(lstmss.LIB_PATH)
    tm, tn = ctypes.c_int(0), ctypes.c_int(0)
    # gemm1_tile(bf16, N, rows, steps * splits, &tm, &tn)
    lib._ZN6lstmss10gemm1_tileEbillPiS0_(True, columns, ctypes.c_long(rows), ctypes.c_long(launches),
                                         ctypes.byref(tm), ctypes.byref(tn))
    return tm.value, tn.value


@pytest.mark.parametrize("T,B,I,H,sp,product,want", CASES)
def test_tile(T, B, I, H, sp, product, want):
    per128 = -(-4 * H // 128) * -(-B // 128)
    rows, launches, k = {
        "input projection": (4 * H, T, I),
        "recurrent": (4 * H, min(-(-768 // per128), H // 128), H),
        "dh": (H, min(-(-512 // (-(-H // 128) * -(-B // 128))), 16), 4 * H * (1 - sp)),
        "input gradient": (I, T, 4 * H * (1 - sp)),
    }[product]
    # large tiles need whole 64-row stages and 16-byte aligned rows
    assert k % 64 == 0 and B % 8 == 0 and (I + H) % 8 == 0 and I % 8 == 0
    assert tile(B, rows, launches) == want


def test_all_large_tiles_are_covered():
    got = {(c[5], c[6]) for c in CASES}
    assert {t for _, t in got} >= {(256, 256), (128, 256)}
    # the gathered input gradient with refills of the row table, on both tiles
    for t in ((256, 256), (128, 256)):
        assert any(c[5] == "input gradient" and c[6] == t and c[4] > 0 and 4 * c[3] * (1 - c[4]) > 2048
                   for c in CASES)
