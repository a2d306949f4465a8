// fp32 products on the bf16 matrix instructions: every fp32 operand x, times
// 2^24, is the exact sum of three bf16 values, 2^24 x = hi + mid + lo (8
// significant bits each), and a product of two operands is the six partial
// products of relative size above 2^-27:
//   x y ~ lo hi' + hi lo' + mid mid' + mid hi' + hi mid' + hi hi',
// each formed exactly by the bf16 MFMA and added in fp32.  A 32 x 32 x 16
// block takes six bf16 MFMAs (6 x 32 cycles) in place of eight fp32 ones
// (8 x 64 cycles).
//
// The power of two is there for small operands: the last bit of an fp32 value
// is 2^-149 at the least, bf16 ends at 2^-133 (2^-126 without denormals), so an
// unscaled lo or mid plane would lose bits of every |x| below 2^-110 (a value
// of 2^-120 kept 14 of its 24 bits).  2^24 brings the last bit to 2^-125.  Results
// are scaled back by 2^-48, exactly; sums from 2^80 on and operands from 2^104 on
// become infinite on the way and take the recomputation below.
//
// Rounding (measured on random products of 2048 terms): the fp32 MFMA leaves a
// relative error of 8.1e-7; six partial products into one accumulator 6.9e-7,
// with a mean of -1e-7 of the results' size, because the bits of a small
// product below a large accumulator's are cut off towards minus infinity; the
// five small partial products in an accumulator of their own 2.7e-7 with no
// mean (below 3e-9).  Products that feed the recurrence use two accumulators
// (split_mma2): a mean would add up over the steps and over the batch.  The
// weight gradient uses one (split_mma) for the sums of one step, whose signs it
// alternates: a mean would add up over a training run's updates.
//
// The operands are split once, on their way from registers into LDS, where
// each plane holds 16-byte pieces of 8 consecutive k of one row (or column):
// piece (kg, r) at index kg * ROWS + slot(r).  A fragment read (lane l: row
// l % 32, k = 8 (l / 32) + 0..7) touches 512 contiguous bytes per half-wave.
//
// An infinite operand (or one that is infinite once scaled) makes products
// of infinity and zero, i.e. NaN, where fp32 has an infinity; the kernels
// therefore check their accumulators and recompute a wavefront's tile with the
// fp32 MFMA whenever one is not finite.
#pragma once

#include "gemm_common.h"

namespace lstmss {

namespace {

// bf16 pair (x in the low half), round to nearest even.
__device__ __forceinline__ uint32_t cvt_pk_bf16(float x, float y) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

constexpr float SPLIT_SCALE = 0x1p24f;    // of either operand
constexpr float SPLIT_UNSCALE = 0x1p-48f; // of a product of the two

// The three planes of a pair of values times `scale`.
__device__ __forceinline__ void split2(float x, float y, float scale, uint32_t &h, uint32_t &m,
                                       uint32_t &l) {
    x *= scale;
    y *= scale;
    h = cvt_pk_bf16(x, y);
    const float rx = x - __uint_as_float(h << 16), ry = y - __uint_as_float(h & 0xffff0000u);
    m = cvt_pk_bf16(rx, ry);
    const float sx = rx - __uint_as_float(m << 16), sy = ry - __uint_as_float(m & 0xffff0000u);
    l = cvt_pk_bf16(sx, sy);
}

// Splits 8 values of consecutive k into the piece at dst of each plane
// (planes `stride` pieces apart: hi, mid, lo).
__device__ __forceinline__ void split_store(uint4 *dst, int stride, const float *v,
                                            float scale = SPLIT_SCALE) {
    uint4 h, m, l;
    split2(v[0], v[1], scale, h.x, m.x, l.x);
    split2(v[2], v[3], scale, h.y, m.y, l.y);
    split2(v[4], v[5], scale, h.z, m.z, l.z);
    split2(v[6], v[7], scale, h.w, m.w, l.w);
    dst[0] = h;
    dst[stride] = m;
    dst[2 * stride] = l;
}

__device__ __forceinline__ f32x16 mfma_bf(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Planes of the six partial products, smallest first.
constexpr int SPLIT_A[6] = {2, 0, 1, 1, 0, 0};
constexpr int SPLIT_B[6] = {0, 2, 1, 0, 1, 0};

// acc[i][j] += A_i B_j for MT x NT fragments (planes first); consecutive
// MFMAs go to different accumulators.
template <int MT, int NT>
__device__ __forceinline__ void split_mma(f32x16 (&acc)[MT][NT], const uint4 (&av)[3][MT],
                                          const uint4 (&bv)[3][NT]) {
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[i][j] = mfma_bf(av[SPLIT_A[p]][i], bv[SPLIT_B[p]][j], acc[i][j]);
}

// The same with the five small partial products in `low`.
template <int MT, int NT>
__device__ __forceinline__ void split_mma2(f32x16 (&acc)[MT][NT], f32x16 (&low)[MT][NT],
                                           const uint4 (&av)[3][MT], const uint4 (&bv)[3][NT]) {
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                f32x16 &c = p == 5 ? acc[i][j] : low[i][j];
                c = mfma_bf(av[SPLIT_A[p]][i], bv[SPLIT_B[p]][j], c);
            }
}

// 0 when v is finite, else NaN (0 * v).
__device__ __forceinline__ float nonfinite(f32x16 c) {
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        s += c[v] * 0.f;
    return s;
}

} // namespace

} // namespace lstmss
