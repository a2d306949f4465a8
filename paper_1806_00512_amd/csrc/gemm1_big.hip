// Data-gradient and forward products of bf16 storage on large tiles.
//
// Paper: the gate gradient feeds every weight and data gradient product of
// the LSTM backward pass (section 3); the kept slices are a dense matrix plus
// an offset index array, so the products run as dense block GEMMs that read
// the kept rows of W through the index (section 3 after Fig. 2, section 4).
#include "gemm_common.h"
#include "select.h"

namespace lstmss {

namespace {

// --------------------------------------------------------------------------
// part[z][m][n] = sum over k in split z of W[row(k)][m] G[k][n], row(k) =
// idx[k/P]*P + k%P (GATHER), the row selected in this launch (SEL) or k; ROWA:
// sum over k of W[m][kcol0 + k] G[k][n].
//
// What bounds the 128 x 128-tile kernel (gemm1_kernel) on these products is
// LDS: its wavefronts of 32 x 64 read 1.5 KB per MFMA, 192 bytes per clock and
// CU at the full MFMA rate where 8-byte transposed reads deliver about 100, and
// its two stages are drained at every barrier.  Here eight wavefronts share a
// 256 x 256 tile (128 x 64 each, 0.75 KB per MFMA) or a 128 x 256 one (64 x 64
// each, 1 KB), the k-steps alternate between two operand register sets,
// and the copies of 64-row stages go to two (256 x 256) or three LDS buffers,
// each awaited by its count so that later ones stay in flight.
//
// Stages are laid out as gemm1_kernel's (rows of k with permuted 16-byte
// pieces, read through ds_read_b64_tr_b16; ROWA's first operand in 128-byte
// lines of k) and every accumulator takes the same MFMAs in the same order, so
// both kernels give the same bits.
//
// Measured at H = I = 4096, B = 256, T = 100 (us, before -> after): input
// projection 3.4 TFLOP on 256 x 256 tiles 4900 -> 3250, recurrent product (192
// tiles, three splits) 53 -> 43; input gradient, 96 steps on 256 x 256 tiles and 4
// on 128 x 128, dense 4100 -> 3070, 50 % gathered 2200 -> 1630; dh product on 128 x
// 256 tiles, dense 55 -> 47, 50 % with the selection 40 -> 36 (its kept rows of W
// alone are 67 MB).
// --------------------------------------------------------------------------
enum GBMode { GB_DENSE = 0, GB_GATHER = 1, GB_SEL = 2, GB_ROWA = 3 };

template <int TM, int TN, int MODE>
__global__ __launch_bounds__(512, 2) void gemm1_big_kernel(Gemm1Args a) {
    constexpr bool GATHER = MODE == GB_GATHER, SEL = MODE == GB_SEL, ROWA = MODE == GB_ROWA;
    constexpr int NTH = 512, NW = 8, TK = 64;
    constexpr int NS = TM + TN > 384 ? 2 : 3;               // LDS stages
    constexpr int WM = TM + TN > 384 ? 2 : TM / 64, WN = NW / WM;
    constexpr int MT = TM / WM / 32, NT = TN / WN / 32;     // MFMA tiles per wavefront
    constexpr int NIA = TK * TM / 512 / NW, NIB = TK * TN / 512 / NW;  // 1 KB copies per wavefront
    constexpr int TAB = GATHER || SEL ? GEMM1_KC_MAX : 1;
    __shared__ __align__(16) uint16_t sA[NS][TK * TM];
    __shared__ __align__(16) uint16_t sB[NS][TK * TN];
    // rows of W (SEL: of the staging matrix too) of the split's k, a ring
    // refilled half by half (SEL: the split fits)
    __shared__ int srow[TAB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM, half = lane >> 5;
    // one step: consecutive work-groups take the splits of one tile, so that
    // an XCD (work-groups are dealt to the eight in turn) reads few splits' rows
    // of G; batched steps: tiles of one step, so that it reads few columns of W
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if (a.steps == 1) {
        const int l = bx + gridDim.x * (by + gridDim.y * bz);
        const int r = l / gridDim.z;
        bz = l - r * gridDim.z;
        by = r / gridDim.x;
        bx = r - by * gridDim.x;
    }
    const int mm0 = bx * TM, n0 = by * TN;
    const int step = bz / a.splitk, split = bz - step * a.splitk;
    const int kb = split * (int)a.k_chunk;
    const int ke = min((int)a.Kp, kb + (int)a.k_chunk);
    const int M = a.M, N = a.N, ldw = (int)a.ldw, P = a.P;
    const bf16_t *W = (const bf16_t *)a.W;
    const bf16_t *G = (const bf16_t *)a.Gc + step * a.gc_step;
    const int32_t *idx = a.idx + (GATHER ? step * a.idx_step : 0);
    const int nst = (ke - kb) / TK;  // whole stages

    auto fill_rows = [&](int p0, int n) {
        const int p1 = min(ke - kb, p0 + n);
        for (int i = p0 + tid; i < p1; i += NTH) {
            const int k = kb + i;
            srow[i & (TAB - 1)] = idx[k / P] * P + k % P;
        }
    };
    if constexpr (GATHER)
        fill_rows(0, TAB);
    if constexpr (SEL) {
        // coarse selection of the split's regions from the chunk sums of
        // squares, with the routines of the select kernel; scratch in the
        // stage buffers (free until the first stage) as in gemm1_kernel
        const int R = a.sel_R, S = a.sel_S, kr = P * (R - S), nch = a.sel_nch;
        const long s_lo = (long)(kb / kr) * R;
        const long s_hi = ke == a.Kp ? a.sel_nslices : min(a.sel_nslices, (long)(ke / kr) * R);
        const int gs = (64 / R) * R;  // whole regions per wavefront
        const int ng = (int)((s_hi - s_lo + gs - 1) / gs);
        const bool write_idx = bx == 0 && by == 0;
        const int L = P * nch, rsb = 64 * L * (int)sizeof(double);
        const int na = (int)(sizeof(sA) / rsb);
        const int nact = L < 16 ? 0 : min(NW, na + (int)(sizeof(sB) / rsb));
        const bool pow2 = (L & (L - 1)) == 0;
        const int lg = __builtin_ctz(L);
        auto pos = [&](int j, int e) { return j * L + (pow2 ? e ^ (j & (L - 1)) : e); };
        const int gstep = nact > 0 ? nact : NW;
        for (int g = wave; wave < gstep && g < ng; g += gstep) {
            const long j0 = s_lo + (long)g * gs;
            const int nsl = (int)min((long)gs, s_hi - j0);
            SliceSel sl;
            if (nact > 0) {
                double *sq = (double *)(wave < na ? (char *)&sA[0][0] + wave * rsb
                                                  : (char *)&sB[0][0] + (wave - na) * rsb);
                const double *src = a.sel_sq + j0 * P * nch;
                const int n = nsl * L;
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the previous group's reads
                for (int x0 = 0; x0 < n; x0 += 8 * 64) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int x = x0 + u * 64 + lane;
                        v[u] = x < n ? src[x] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int x = x0 + u * 64 + lane;
                        const int j = pow2 ? x >> lg : x / L;
                        if (x < n)
                            sq[pos(j, x - j * L)] = v[u];
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the wavefront's writes landed
                double scv = 0.0;
                if (lane < nsl) {
                    for (int p = 0; p < P; ++p) {
                        double rs = sq[pos(lane, p * nch)];
                        for (int c = 1; c < nch; ++c)
                            rs = rs + sq[pos(lane, p * nch + c)];
                        scv = p == 0 ? rs : scv + rs;
                    }
                }
                sl = rank_slices(scv, j0, nsl, R, S, a.sel_nslices);
            } else {
                sl = select_slices(a.sel_sq, nch, j0, nsl, P, R, S, a.sel_nslices);
            }
            if (sl.slot >= 0) {
                const int j = (int)(j0 + lane);
                for (int p = 0; p < P; ++p)
                    srow[sl.slot * P + p - kb] = j * P + p;
                if (write_idx)
                    a.sel_idx[sl.slot] = j;
            }
        }
    }

    // copies: instruction q = wave + 8 i fills elements [512 q, 512 q + 512) of a
    // stage's operand, lane j its 8 elements from 8 j on.  Columns past M or N
    // are clamped to the last whole piece of the row (never stored).
    uint32_t va[NIA], vb[NIB];  // byte offset from the stage's first row (gathered: in the row)
    int ka[NIA], kbr[NIB];      // row within the stage
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
        const int off = (wave + NW * i) * 512 + lane * 8;
        if constexpr (ROWA) {
            const int ml = off / TK, pc = (off - ml * TK) / 8;
            va[i] = 2u * ((uint32_t)min(mm0 + ml, M - 1) * ldw + a.kcol0 + ((pc ^ g1_swzr(ml)) * 8));
            ka[i] = 0;
        } else {
            const int kl = off / TM, pc = (off - kl * TM) / 8;
            const int m = min(a.m_lo + mm0 + (pc ^ g1_swz16(kl)) * 8, (M - 1) & ~7);
            va[i] = 2u * ((GATHER || SEL ? 0u : (uint32_t)kl * ldw) + m);
            ka[i] = kl;
        }
    }
#pragma unroll
    for (int i = 0; i < NIB; ++i) {
        const int off = (wave + NW * i) * 512 + lane * 8;
        const int kl = off / TN, pc = (off - kl * TN) / 8;
        const int n = min(n0 + (pc ^ g1_swz16(kl)) * 8, N - 8);
        vb[i] = 2u * ((SEL ? 0u : (uint32_t)kl * N) + n);
        kbr[i] = kl;
    }
    // table entries of the stage to be copied next, read ahead of its copies
    uint32_t oa[NIA], ob[NIB];
    auto look = [&](int s) __attribute__((always_inline)) {
        if constexpr (GATHER || SEL)
#pragma unroll
            for (int i = 0; i < NIA; ++i)
                oa[i] = (uint32_t)srow[(s * TK + ka[i]) & (TAB - 1)];
        if constexpr (SEL)
#pragma unroll
            for (int i = 0; i < NIB; ++i)
                ob[i] = (uint32_t)srow[(s * TK + kbr[i]) & (TAB - 1)];
    };
    auto load = [&](int s) __attribute__((always_inline)) {
        const int buf = s % NS, k0 = kb + s * TK;
        const i32x4 rw = buf_rsrc(W + (GATHER || SEL ? 0L : ROWA ? (long)k0 : (long)k0 * ldw), ~0u);
        const i32x4 rg = buf_rsrc(G + (SEL ? 0L : (long)k0 * N), ~0u);
#pragma unroll
        for (int i = 0; i < NIA; ++i)
            dma16_buf(rw, (int)(GATHER || SEL ? oa[i] * (2u * ldw) + va[i] : va[i]), 0,
                      (lds_void_t *)&sA[buf][(wave + NW * i) * 512]);
#pragma unroll
        for (int i = 0; i < NIB; ++i)
            dma16_buf(rg, (int)(SEL ? ob[i] * (2u * N) + vb[i] : vb[i]), 0,
                      (lds_void_t *)&sB[buf][(wave + NW * i) * 512]);
    };
    auto wait_stages = [&](int n) __attribute__((always_inline)) {  // n stages may be in flight
        if (NS > 2 && n >= 2)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS > 2 ? 2 : 0) * (NIA + NIB)));
        else if (n >= 1)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(NIA + NIB));
        else
            __builtin_amdgcn_s_waitcnt(0);
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = 0.f;
    const int mw = wm * MT * 32, nw = wn * NT * 32;  // wavefront tile origin

    // this lane's element offsets of its operand reads within a k-step: for
    // the transposed reads lane s of a group of 16 points at row s / 4, columns
    // 4 (s % 4) .. + 3 (rows 4 further down and further k-steps: constants)
    const int g = lane >> 4, sl = lane & 15;
    const int kl0 = 8 * (g >> 1) + (sl >> 2);
    int ao[MT], asw[MT], bo[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = ROWA ? mw + i * 32 + (lane & 31) : mw + i * 32 + 16 * (g & 1) + 4 * (sl & 3);
        ao[i] = ROWA ? m * TK : kl0 * TM + (((m >> 3) ^ g1_swz16(kl0)) << 3) + (m & 7);
        asw[i] = g1_swzr(m);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int n = nw + j * 32 + 16 * (g & 1) + 4 * (sl & 3);
        bo[j] = kl0 * TN + (((n >> 3) ^ g1_swz16(kl0)) << 3) + (n & 7);
    }
    auto trd = [](const uint16_t *p, int next4) __attribute__((always_inline)) {
        const g1_s16x4 lo = __builtin_bit_cast(
            g1_s16x4, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((g1_lds_bf16x4 *)(p)));
        const g1_s16x4 hi = __builtin_bit_cast(
            g1_s16x4, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((g1_lds_bf16x4 *)(p + next4)));
        return __builtin_bit_cast(u16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // operands of k-step s of buffer buf into register set st
    u16x8 fa[2][MT], fb[2][NT];
    auto rd = [&](int buf, int s, auto setc) __attribute__((always_inline)) {
        constexpr int st = decltype(setc)::value;
        const uint16_t *pa = &sA[buf][0], *pb = &sB[buf][0];
#pragma unroll
        for (int i = 0; i < MT; ++i)
            fa[st][i] = ROWA ? *(const u16x8 *)(pa + ao[i] + (((2 * s + half) ^ asw[i]) << 3))
                             : trd(pa + ao[i] + s * 16 * TM, 4 * TM);
#pragma unroll
        for (int j = 0; j < NT; ++j)
            fb[st][j] = trd(pb + bo[j] + s * 16 * TN, 4 * TN);
    };
    auto mma = [&](auto setc) __attribute__((always_inline)) {
        constexpr int st = decltype(setc)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[i][j] = mfma32x32x16bf(fa[st][i], fb[st][j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};

    __syncthreads();  // the row table is written, the selection's scratch is free
#pragma unroll
    for (int c = 0; c < NS; ++c)
        if (c < nst) {
            look(c);
            load(c);
        }
    if (nst > 0) {
        wait_stages(min(NS - 1, nst - 1));
        lds_barrier();
        rd(0, 0, S0);
        rd(0, 1, S1);
    }
    // Iteration it multiplies stage it (k-steps 0 and 1 already in registers)
    // and, before its last k-step, meets the other wavefronts once stage it + 1
    // has landed: stage it's buffer then takes stage it + NS.
    for (int it = 0; it + 1 < nst; ++it) {
        const int buf = it % NS;
        mma(S0);
        rd(buf, 2, S0);
        mma(S1);
        rd(buf, 3, S1);
        if (it + NS < nst)
            look(it + NS);
        mma(S0);
        wait_stages(min(NS - 2, nst - 2 - it));
        lds_barrier();
        if (it + NS < nst)
            load(it + NS);
        if constexpr (GATHER) {
            // every wavefront has read the entries up to stage it + NS: a used
            // half of the ring takes the positions TAB / 2 ahead
            const int pos = (it + NS + 1) * TK;
            if ((pos & (TAB / 2 - 1)) == 0 && kb + pos + TAB / 2 < ke)
                fill_rows(pos + TAB / 2, TAB / 2);
        }
        const int nb = (it + 1) % NS;
        rd(nb, 0, S0);
        mma(S1);
        rd(nb, 1, S1);
    }
    if (nst > 0) {  // the last stage
        const int buf = (nst - 1) % NS;
        mma(S0);
        rd(buf, 2, S0);
        mma(S1);
        rd(buf, 3, S1);
        mma(S0);
        mma(S1);
    }

    // SEL: the split's kept rows are shared out over its m-tiles, each
    // work-group copying its share (its columns) to the compacted matrix; the
    // first pieces are loaded before the partial sums are stored
    constexpr int PPR = TN / 8;  // 16-byte pieces per tile row
    constexpr int CPB = SEL ? 2 : 1;
    uint4 cbuf[CPB];
    int c_r0 = 0, c_np = 0;
    if constexpr (SEL) {
        const int nr = ke - kb, nmt = (int)gridDim.x;
        c_r0 = (int)((long)nr * bx / nmt);
        c_np = ((int)((long)nr * (bx + 1) / nmt) - c_r0) * PPR;
#pragma unroll
        for (int i = 0; i < CPB; ++i) {
            const int e = tid + i * NTH;
            const int k = c_r0 + e / PPR, n = n0 + (e % PPR) * 8;
            cbuf[i] = make_uint4(0, 0, 0, 0);
            if (e < c_np && n < N)
                cbuf[i] = *(const uint4 *)(G + (long)srow[k] * N + n);
        }
    }
    float *out = a.part + step * a.out_step + split * a.part_stride;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int n = n0 + nw + j * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = a.m_lo + mm0 + mw + i * 32 + acc_row(lane, v);
                if (m >= a.m_begin && m < M && n < N)
                    out[(long)(m - a.out_row0) * N + n] = acc[i][j][v];
            }
        }
    if constexpr (SEL) {
        bf16_t *gc = (bf16_t *)a.sel_gc;
#pragma unroll
        for (int i = 0; i < CPB; ++i) {
            const int e = tid + i * NTH;
            const int k = c_r0 + e / PPR, n = n0 + (e % PPR) * 8;
            if (e < c_np && n < N)
                *(uint4 *)(gc + (long)(kb + k) * N + n) = cbuf[i];
        }
        for (int e = tid + CPB * NTH; e < c_np; e += NTH) {
            const int k = c_r0 + e / PPR, n = n0 + (e % PPR) * 8;
            if (n < N)
                *(uint4 *)(gc + (long)(kb + k) * N + n) = *(const uint4 *)(G + (long)srow[k] * N + n);
        }
    }
}

template <int TM, int TN>
void launch_tile(dim3 grid, const Gemm1Args &a, bool rowa, hipStream_t s) {
    if (rowa)
        hipLaunchKernelGGL((gemm1_big_kernel<TM, TN, GB_ROWA>), grid, dim3(512), 0, s, a);
    else if (a.sel_sq)
        hipLaunchKernelGGL((gemm1_big_kernel<TM, TN, GB_SEL>), grid, dim3(512), 0, s, a);
    else if (a.idx)
        hipLaunchKernelGGL((gemm1_big_kernel<TM, TN, GB_GATHER>), grid, dim3(512), 0, s, a);
    else
        hipLaunchKernelGGL((gemm1_big_kernel<TM, TN, GB_DENSE>), grid, dim3(512), 0, s, a);
}

} // namespace

// Arguments checked by the caller (gemm1.hip): 16-byte aligned operands and
// rows, whole 64-row stages, m_lo set.
void launch_gemm1_big(dim3 grid, const Gemm1Args &a, int TM, int TN, bool rowa, hipStream_t s) {
    if (TM == 256 && TN == 256)
        launch_tile<256, 256>(grid, a, rowa, s);
    else
        launch_tile<128, 256>(grid, a, rowa, s);
}

} // namespace lstmss
