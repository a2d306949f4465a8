// Row grouping of the coarse structure's weight gradient, shared by the fp32
// and bf16 kernels (wgrad_f32.hip, wgrad_bf16.hip).
#pragma once

#include "gemm_common.h"

namespace lstmss {

namespace {

constexpr int WG_ATMAX = 4;

// Temporary tiles (kept rows per group / 32) and accumulator tiles (original
// rows per group / 32) of the sparse weight-gradient kernel.  (Grouping four
// regions of 24 kept rows into three exactly filled tiles needs 224
// accumulator registers, one wavefront per SIMD: measured 1.14-1.3x slower
// than the 24-of-32 tiles at 25 % sparsity.)
inline void wgrad_tiles(int P, int R, int S, int *greg, int *tt, int *at) {
    const int kr = (R - S) * P, rp = R * P;
    *greg = kr <= 32 ? max(1, 32 / kr) : 1;
    *tt = (*greg * kr + 31) / 32;
    *at = (*greg * rp + 31) / 32;
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

} // namespace

} // namespace lstmss
