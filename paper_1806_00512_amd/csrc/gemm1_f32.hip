// Data-gradient product on the compacted gate gradient and the forward
// products, fp32 storage, on bf16 matrix instructions (split.h).
//
// Paper: the gate gradient feeds every weight and data gradient product of
// the LSTM backward pass (section 3); after sparsifying, the kept slices are
// a dense matrix plus an offset index array, so the products run as dense
// block GEMMs that read the kept rows of W through the index (section 3 after
// Fig. 2, section 4).
#include "select.h"
#include "split.h"

namespace lstmss {

namespace {

// --------------------------------------------------------------------------
// part[z][m][n] = sum over k in split z of W[row(k)][m] G[k][n], row(k) =
// idx[k/P]*P + k%P (GATHER) or k; ROWA: sum over k of W[m][kcol0 + k] G[k][n]
// (forward products).
//
// Work-group tile TM x TN, WM x WN wavefronts of MT x NT MFMA tiles, stages of
// TK = 8 KG rows.  A thread loads 8 consecutive k of two columns (or, ROWA, 8
// consecutive k of one row of W and of one column of G), splits them and
// stores one 16-byte piece per column and plane.  The MFMAs of stage s run from
// registers, which then take the operands of s + 1 from one LDS buffer; s + 2 is
// split and written to the other (whose operands were read during s - 1) and
// the global loads of the next NRAW stages are outstanding.  One barrier per
// stage.
//
// SEL: the coarse selection of one step inside its dh product.  Every
// work-group ranks the slices of its split's regions (whole regions: the
// split length is a multiple of P (R - S) kept rows) from the element
// kernel's chunk sums of squares, with the same wavefront routines as the
// select kernel, and gathers the rows of both operands through the result:
// W rows and the staging matrix's rows (Gc).  The split's work-groups share
// out the copy of its kept rows to the compacted matrix (after their
// product, from the staging matrix); those of tile (0, 0) also write the
// split's slots of the offset index.
// FN: the fine structure with 32-row slices and 32-column blocks on the
// masked matrix, TN = 32 (a work-group's columns are one block): the
// work-group gathers the rows of the slices that keep its block and skips the
// others, W rows and gate-gradient rows alike (their products are exactly
// zero, so the result is bit-identical to multiplying them).
// --------------------------------------------------------------------------
enum G1Mode { G1_DENSE = 0, G1_GATHER = 1, G1_SEL = 2, G1_FN = 3, G1_ROWA = 4 };

// V: width of the loads: pairs of columns (ROWA: 2 k of a row) as 8 bytes (1) or
// one by one (0); 2, ROWA only: 4 k of a row as 16 bytes
template <int TM, int TN, int WM, int WN, int KG, int MODE, int V>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm1_split_kernel(Gemm1Args a) {
    constexpr bool GATHER = MODE == G1_GATHER, SEL = MODE == G1_SEL, FN = MODE == G1_FN,
                   ROWA = MODE == G1_ROWA;
    constexpr int NTH = WM * WN * 64, TK = 8 * KG;
    constexpr int MT = TM / WM / 32, NT = TN / WN / 32;
    // staging units: pairs of columns x 8 k (ROWA: single rows / columns x 8 k)
    constexpr int UA = TM / (ROWA ? 1 : 2) * KG, UB = TN / (ROWA ? 1 : 2) * KG;
    static_assert(ROWA ? (UA <= NTH && UB <= NTH) : UA + UB <= NTH, "one unit per thread");
    static_assert(UA % 64 == 0, "a wavefront stages one operand");
    constexpr int TAB = SEL || GATHER ? GEMM1_KC_MAX : 1;
    __shared__ uint4 sA[2][3][KG][TM];
    __shared__ uint4 sB[2][3][KG][TN];
    // element offsets of the gathered rows of W (GATHER: a ring refilled half
    // by half) and, SEL, of the staging matrix
    __shared__ __align__(16) int srow[TAB];
    __shared__ __align__(16) int sgrow[SEL ? TAB : 1];
    __shared__ int slist[FN ? FINE_MAX_SLICES : 1];
    __shared__ int s_nact;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM, half = lane >> 5;
    const int mm0 = blockIdx.x * TM, n0 = blockIdx.y * TN;
    const int step = blockIdx.z / a.splitk, split = blockIdx.z - step * a.splitk;
    const int kb = split * (int)a.k_chunk;
    const int ke0 = min((int)a.Kp, kb + (int)a.k_chunk);
    const int M = a.M, N = a.N, ldw = (int)a.ldw, P = a.P;
    const float *__restrict__ W = (const float *)a.W;
    const float *__restrict__ G = (const float *)a.Gc + step * a.gc_step;
    const int32_t *__restrict__ idx = a.idx + (GATHER ? step * a.idx_step : 0);

    int ke = ke0;
    if constexpr (FN) {
        // slices of [kb, ke0) that keep this work-group's column block, in
        // ascending order (one wavefront compacts them with ballots)
        if (tid < 64) {
            const int32_t *fi = a.fidx + step * a.fidx_step;
            const int c = n0 >> 5, s_end = ke0 >> 5;
            int base = 0;
            for (int sb = kb >> 5; sb < s_end; sb += 64) {
                const int sl = sb + tid;
                bool kept = false;
                if (sl < s_end) {
                    const int32_t *e = fi + (long)sl * a.fkept;
                    for (int q = 0; q < a.fkept; ++q)
                        kept |= e[q] == c;
                }
                const uint64_t m = __ballot(kept);
                if (kept)
                    slist[base + __popcll(m & ((1ull << tid) - 1ull))] = sl;
                base += __popcll(m);
            }
            if (tid == 0)
                s_nact = base;
        }
        __syncthreads();
        ke = kb + s_nact * 32;
    }
    // table entries of positions [p0, p0 + n) of the split
    auto fill_rows = [&](int p0, int n) {
        const int p1 = min(ke - kb, p0 + n);
        for (int i = p0 + tid; i < p1; i += NTH) {
            const int k = kb + i;
            srow[i & (TAB - 1)] = (idx[k / P] * P + k % P) * ldw;
        }
    };
    if constexpr (GATHER)
        fill_rows(0, TAB);
    if constexpr (SEL) {
        const int R = a.sel_R, S = a.sel_S, kr = P * (R - S), nch = a.sel_nch;
        const long s_lo = (long)(kb / kr) * R;
        const long s_hi = ke0 == a.Kp ? a.sel_nslices : min(a.sel_nslices, (long)(ke0 / kr) * R);
        const int gs = (64 / R) * R;  // whole regions per wavefront
        const int ng = (int)((s_hi - s_lo + gs - 1) / gs);
        const bool write_idx = blockIdx.x == 0 && blockIdx.y == 0;
        // A group's chunk sums (L per slice) are one contiguous run: a
        // wavefront reads it coalesced into its own region of the plane
        // buffers (free until the first stage), lane j's slice at row j,
        // its entries permuted by j when L is a power of two so that the
        // lanes' reads of one entry fall on distinct banks; then each lane
        // folds its slice as select_slices does.  With fewer than 16 entries
        // per slice (measured faster so), or without room for a region, the
        // lanes read their slices directly.
        constexpr int NW = WM * WN;
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
                double *sq = (double *)(wave < na ? (char *)&sA[0][0][0][0] + wave * rsb
                                                  : (char *)&sB[0][0][0][0] + (wave - na) * rsb);
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
                for (int p = 0; p < P; ++p) {
                    srow[sl.slot * P + p - kb] = (j * P + p) * ldw;
                    sgrow[sl.slot * P + p - kb] = (j * P + p) * N;
                }
                if (write_idx)
                    a.sel_idx[sl.slot] = j;
            }
        }
    }
    // slot of row / column r in its plane: the lanes of a 16-lane group of
    // piece stores fall on distinct banks
    auto slot = [](int r, int kg) { return ROWA ? r ^ ((kg * (16 / KG)) & 15) : r ^ ((r >> 4) & 1); };
    auto slotB = [](int r) { return ROWA ? r : r ^ ((r >> 4) & 1); };

    // this thread's staging units
    const bool isa = wave * 64 < UA;                       // (ROWA: stages rows of W)
    const bool isb = ROWA ? tid < UB : !isa && tid < UA + UB;
    const int ua = ROWA || isa ? tid : 0, ub = ROWA ? tid : isb ? tid - UA : 0;
    const int kga = ROWA ? ua % KG : ua / (TM / 2), ma = ROWA ? ua / KG : (ua % (TM / 2)) * 2;
    const int kgb = ub / (ROWA ? TN : TN / 2), nb = ROWA ? ub % TN : (ub % (TN / 2)) * 2;
    const int kg = isa ? kga : kgb;                        // (not ROWA)
    // columns past M or N are clamped to valid ones (never stored)
    constexpr int ALIGN = V > 0 && !ROWA ? ~1 : ~0;
    const int mcol = min((ROWA ? 0 : a.m_lo) + mm0 + ma, (M - 1) & ALIGN);
    const int ncol = min(n0 + nb, (N - 1) & ALIGN);
    // not ROWA: operand, row length and columns of this wavefront's unit
    const float *__restrict__ src = isa ? W : G;
    const int ld = isa ? ldw : N;
    const uint32_t col = isa ? mcol : ncol;
    const uint32_t dcol1 = col + 1 < (uint32_t)ld ? 1 : 0;  // second column (V = 0)
    // element offset of the unit within 8 KG rows that follow each other
    const uint32_t vofs = ROWA ? 8 * kgb * N + ncol : 8 * kg * ld + col;
    const int *tab = isa || !SEL ? srow : sgrow;

    // stages of global loads in flight (128 x 128 tiles have registers for two)
    constexpr int NRAW = TN == 128 ? 2 : 4;
    float r[NRAW][2][8];
    const int nst = (ke - kb + TK - 1) / TK;
    int p_ld = 0;  // position of the next stage to load
    auto load_stage = [&](auto setc, auto wholec) __attribute__((always_inline)) {
        constexpr int st = decltype(setc)::value;
        constexpr bool whole = decltype(wholec)::value;  // the stage ends inside the split
        const int pos = p_ld;
        if constexpr (ROWA) {
            if (UA == NTH || isa) {
                const float *p = W + (long)mcol * ldw + a.kcol0 + kb + pos + 8 * kga;
                if (V > 0 && whole) {
                    typedef float fv __attribute__((ext_vector_type(V == 2 ? 4 : 2)));
#pragma unroll
                    for (int j = 0; j < 8; j += V == 2 ? 4 : 2) {
                        const fv u = *(const fv *)(p + j);
#pragma unroll
                        for (int e = 0; e < (V == 2 ? 4 : 2); ++e)
                            r[st][0][j + e] = u[e];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        r[st][0][j] = whole || kb + pos + 8 * kga + j < ke ? p[j] : 0.f;
                }
            }
            if (UB == NTH || isb) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (whole) {
                        r[st][1][j] = (G + (long)(kb + pos + j) * N)[vofs];
                    } else {
                        const int k = kb + pos + 8 * kgb + j;
                        const float v = G[(long)min(k, ke - 1) * N + ncol];
                        r[st][1][j] = k < ke ? v : 0.f;
                    }
                }
            }
        } else {
            // rows of this wavefront's operand that follow each other start at
            // k0 (FN: a stage lies in one kept slice)
            const int k0 = FN ? __builtin_amdgcn_readfirstlane(slist[pos >> 5]) * 32 + (pos & 31) : kb + pos;
            uint32_t off[8];
            if (GATHER || SEL) {
                const uint4 u = *(const uint4 *)&tab[(pos + 8 * kg) & (TAB - 1)];
                const uint4 v = *(const uint4 *)&tab[(pos + 8 * kg + 4) & (TAB - 1)];
                off[0] = u.x; off[1] = u.y; off[2] = u.z; off[3] = u.w;
                off[4] = v.x; off[5] = v.y; off[6] = v.z; off[7] = v.w;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool in = whole || kb + pos + 8 * kg + j < ke;
                const float *p;
                if (SEL)
                    p = src + (in ? off[j] : 0) + col;
                else if (GATHER)
                    p = src + (!in ? 0 : isa ? off[j] : (uint32_t)((k0 + 8 * kg + j) * ld)) + col;
                else if (whole)
                    p = src + (long)(k0 + j) * ld + vofs;
                else
                    p = src + (in ? (uint32_t)((k0 + 8 * kg + j) * ld) : 0u) + col;
                float2 t;
                if (V > 0) {
                    t = *(const float2 *)p;
                } else {
                    t.x = p[0];
                    t.y = p[dcol1];
                }
                r[st][0][j] = in ? t.x : 0.f;
                r[st][1][j] = in ? t.y : 0.f;
            }
        }
        p_ld += TK;
    };
    auto load = [&](auto setc, auto allc) __attribute__((always_inline)) {
        if (decltype(allc)::value || FN || kb + p_ld + TK <= ke)
            load_stage(setc, std::true_type());
        else
            load_stage(setc, std::false_type());
    };
    auto stash = [&](auto setc, auto bufc) __attribute__((always_inline)) {
        constexpr int st = decltype(setc)::value, buf = decltype(bufc)::value;
        if constexpr (ROWA) {
            if (UA == NTH || isa)
                split_store(&sA[buf][0][kga][slot(ma, kga)], KG * TM, r[st][0]);
            if (UB == NTH || isb)
                split_store(&sB[buf][0][kgb][slotB(nb)], KG * TN, r[st][1]);
        } else {
            uint4 *d = isa ? &sA[buf][0][kga][slot(ma, kga)] : &sB[buf][0][kgb][slotB(nb)];
            uint4 *d1 = isa ? &sA[buf][0][kga][slot(ma + 1, kga)] : &sB[buf][0][kgb][slotB(nb + 1)];
            const int stride = isa ? KG * TM : KG * TN;
            if (UA + UB == NTH || isa || isb) {
                split_store(d, stride, r[st][0]);
                split_store(d1, stride, r[st][1]);
            }
        }
    };

    f32x16 acc[MT][NT], low[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = low[i][j][v] = 0.f;
    const int mw = wm * MT * 32, nw = wn * NT * 32;  // wavefront tile origin

    // operands of the 16-row k-steps of a stage in registers
    constexpr int KS = KG / 2;
    uint4 av[KS][3][MT], bv[KS][3][NT];
    auto read = [&](auto bufc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int q = 2 * ks + half;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    av[ks][p][i] = sA[buf][p][q][slot(mw + i * 32 + (lane & 31), q)];
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    bv[ks][p][j] = sB[buf][p][q][slotB(nw + j * 32 + (lane & 31))];
            }
        }
    };
    // stage s (s mod 4 static): its MFMAs, the operands of s + 1, the pieces of
    // s + 2 and the loads of s + 2 + NRAW (`all`: these stages exist)
    auto stage = [&](auto qc, int s, auto allc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        constexpr bool all = decltype(allc)::value;
        constexpr std::integral_constant<int, q & 1> B0{};
        constexpr std::integral_constant<int, (q & 1) ^ 1> B1{};
        constexpr std::integral_constant<int, (q + 2) % NRAW> RS{};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            split_mma2<MT, NT>(acc, low, av[ks], bv[ks]);
        if (all || s + 1 < nst)
            read(B1);
        if (all || s + 2 < nst)
            stash(RS, B0);
        if (all || s + 2 + NRAW < nst)
            load(RS, allc);
        if constexpr (GATHER && q == 3) {
            // the half of the ring whose positions are all loaded takes the
            // positions from TAB / 2 ahead on
            const int pos = (s + 1) * TK;
            if ((pos & (TAB / 2 - 1)) == 0 && kb + pos + TAB / 2 < ke)
                fill_rows(pos + TAB / 2, TAB / 2);
        }
        lds_barrier();
    };
    constexpr std::integral_constant<int, 0> Q0{};
    constexpr std::integral_constant<int, 1> Q1{};
    constexpr std::integral_constant<int, 2> Q2{};
    constexpr std::integral_constant<int, 3> Q3{};
    __syncthreads();
    if (nst > 0) {  // FN: a block no slice of the range keeps has no stages
        load(Q0, std::false_type());
        if (1 < nst)
            load(Q1, std::false_type());
        if constexpr (NRAW == 4) {
            if (2 < nst)
                load(Q2, std::false_type());
            if (3 < nst)
                load(Q3, std::false_type());
        }
        stash(Q0, Q0);
        if (NRAW < nst)
            load(Q0, std::false_type());
        if (1 < nst)
            stash(Q1, Q1);
        if (NRAW + 1 < nst)
            load(Q1, std::false_type());
        lds_barrier();
        read(Q0);
        lds_barrier();
        int s = 0;
        for (; s + 3 + 2 + NRAW + 1 < nst; s += 4) {  // (never loads the last stage)
            stage(Q0, s, std::true_type());
            stage(Q1, s + 1, std::true_type());
            stage(Q2, s + 2, std::true_type());
            stage(Q3, s + 3, std::true_type());
        }
        for (; s < nst; s += 4) {
            stage(Q0, s, std::false_type());
            if (s + 1 < nst)
                stage(Q1, s + 1, std::false_type());
            if (s + 2 < nst)
                stage(Q2, s + 2, std::false_type());
            if (s + 3 < nst)
                stage(Q3, s + 3, std::false_type());
        }
    }

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] += low[i][j][v];

    // an accumulator that is not finite: the tile again on the fp32 MFMA
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            bad += nonfinite(acc[i][j]);
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] *= SPLIT_UNSCALE;
        }
    if (__builtin_expect(__ballot(bad != bad) != 0, 0)) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc[i][j][v] = 0.f;
        for (int k = kb + half; k - half < ke; k += 2) {
            const bool in = k < ke;
            const int kk = in ? k : ke - 1;
            const int fr = FN ? slist[(kk - kb) >> 5] * 32 + ((kk - kb) & 31) : kk;
            const int wo = GATHER ? (idx[kk / P] * P + kk % P) * ldw : SEL ? srow[kk - kb] : fr * ldw;
            const int go = SEL ? sgrow[kk - kb] : fr * N;
            float av[MT], bv[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int m = min((ROWA ? 0 : a.m_lo) + mm0 + mw + i * 32 + (lane & 31), M - 1);
                const float v = ROWA ? W[(long)m * ldw + a.kcol0 + kk] : W[(long)wo + m];
                av[i] = in ? v : 0.f;
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int n = min(n0 + nw + j * 32 + (lane & 31), N - 1);
                const float v = G[(long)go + n];
                bv[j] = in ? v : 0.f;
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = mfma32x32x2(av[i], bv[j], acc[i][j]);
        }
    }

    // SEL: compacted rows.  The split's rows are shared out over its
    // m-tiles, each work-group copying its share (its columns) from the
    // staging matrix after its product, so that no stage waits for these
    // stores; the first pieces are loaded before the partial sums are
    // stored, so that waiting for them does not wait for those stores.
    constexpr int PPR = TN / 4;  // 16-byte pieces per tile row
    constexpr int CPB = SEL ? 2 : 1;
    uint4 cbuf[CPB];
    int c_r0 = 0, c_np = 0;
    if constexpr (SEL) {
        const int nr = ke0 - kb, nmt = (int)gridDim.x;
        c_r0 = (int)((long)nr * blockIdx.x / nmt);
        c_np = ((int)((long)nr * (blockIdx.x + 1) / nmt) - c_r0) * PPR;
#pragma unroll
        for (int i = 0; i < CPB; ++i) {
            const int e = tid + i * NTH;
            const int k = kb + c_r0 + e / PPR, n = n0 + (e % PPR) * 4;
            cbuf[i] = make_uint4(0, 0, 0, 0);
            if (e < c_np && n < N)
                cbuf[i] = *(const uint4 *)(G + sgrow[k - kb] + n);
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
        float *gc = (float *)a.sel_gc;
#pragma unroll
        for (int i = 0; i < CPB; ++i) {
            const int e = tid + i * NTH;
            const int k = kb + c_r0 + e / PPR, n = n0 + (e % PPR) * 4;
            if (e < c_np && n < N)
                *(uint4 *)(gc + (long)k * N + n) = cbuf[i];
        }
        for (int e = tid + CPB * NTH; e < c_np; e += NTH) {
            const int k = kb + c_r0 + e / PPR, n = n0 + (e % PPR) * 4;
            if (n < N)
                *(uint4 *)(gc + (long)k * N + n) = *(const uint4 *)(G + sgrow[k - kb] + n);
        }
    }
}

template <int TM, int TN, int WM, int WN, int KG>
hipError_t launch_tile(dim3 grid, const Gemm1Args &a, int mode, int v, hipStream_t s) {
    const dim3 block(WM * WN * 64);
#define LSTMSS_G1S(MODE, V) \
    hipLaunchKernelGGL((gemm1_split_kernel<TM, TN, WM, WN, KG, MODE, V>), grid, block, 0, s, a)
#define LSTMSS_G1V(MODE) do { if (v) LSTMSS_G1S(MODE, 1); else LSTMSS_G1S(MODE, 0); } while (0)
    switch (mode) {
    case G1_DENSE: LSTMSS_G1V(G1_DENSE); break;
    case G1_GATHER: LSTMSS_G1V(G1_GATHER); break;
    case G1_SEL: if constexpr (TN != 32) { LSTMSS_G1V(G1_SEL); break; } else return hipErrorInvalidValue;
    case G1_FN: if constexpr (TN == 32) { LSTMSS_G1V(G1_FN); break; } else return hipErrorInvalidValue;
    default: if (v == 2) LSTMSS_G1S(G1_ROWA, 2); else LSTMSS_G1V(G1_ROWA); break;
    }
#undef LSTMSS_G1V
#undef LSTMSS_G1S
    return hipGetLastError();
}

hipError_t launch(dim3 grid, const Gemm1Args &a, int TM, int TN, int mode, int v, hipStream_t s) {
    if (TN == 32)
        return launch_tile<128, 32, 4, 1, 2>(grid, a, mode, v, s);
    if (TN == 64)
        return launch_tile<64, 64, 2, 2, 4>(grid, a, mode, v, s);
    return launch_tile<128, 128, 2, 2, 2>(grid, a, mode, v, s);
}

bool tile_ok(int TM, int TN) {
    return (TN == 32 && TM == 128) || (TN == 64 && TM == 64) || (TN == 128 && TM == 128);
}

// Launch configuration of a data-gradient product (sets a.m_lo).
struct G1Plan {
    int TM, TN, mode, v;
    dim3 grid;
};

hipError_t g1_plan(Gemm1Args &a, G1Plan *pl) {
    if (a.k_chunk % GEMM1_TK != 0 || a.splitk < 1 || a.steps < 1)
        return hipErrorInvalidValue;
    // fine fast path: no gather, whole 32-row slices, 32-column blocks, the
    // slices of one split fit the work-group's table
    if (a.fidx && (a.idx || a.sel_sq || a.P != 32 || a.fkept < 1 || a.fkept > 64 ||
                   a.N % 32 != 0 || ceil_div(a.k_chunk, 32) > FINE_MAX_SLICES))
        return hipErrorInvalidValue;
    // pairs of columns load as 8 bytes; the tile origin is rounded down to
    // a pair and rows below m_begin are not stored
    const bool vec = a.ldw % 2 == 0 && a.N % 2 == 0 && ((uintptr_t)a.W & 7) == 0 &&
                     ((uintptr_t)a.Gc & 7) == 0;
    a.m_lo = vec ? a.m_begin / 2 * 2 : a.m_begin;
    pl->v = vec ? 1 : 0;
    const long z = (long)a.splitk * a.steps;
    gemm1_tile(false, a.N, a.M - a.m_lo, z, &pl->TM, &pl->TN);
    if (a.tm)
        pl->TM = a.tm;
    if (a.tn)
        pl->TN = a.tn;
    if (a.fidx) {  // one column block per work-group
        pl->TM = 128;
        pl->TN = 32;
    }
    if (!tile_ok(pl->TM, pl->TN))
        return hipErrorInvalidValue;
    pl->mode = a.fidx ? G1_FN : a.sel_sq ? G1_SEL : a.idx ? G1_GATHER : G1_DENSE;
    pl->grid = dim3((unsigned)ceil_div(a.M - a.m_lo, pl->TM), (unsigned)ceil_div(a.N, pl->TN), (unsigned)z);
    // selection inside the product: one step, splits of whole regions and whole
    // 32-row pieces whose gathered rows fit one table, rows copied in 16-byte
    // pieces (off with LSTMSS_OPT_GEMM_DMA, like the bf16 product's)
    if (a.sel_sq) {
        const int R = a.sel_R, S = a.sel_S;
        if (!a.dma || a.Kp % 32 != 0 || a.idx || pl->TN == 32 || a.steps != 1 || R < 1 || R > 64 || S < 1 || S >= R || a.P < 1 ||
            a.k_chunk > GEMM1_KC_MAX || a.k_chunk % ((long)a.P * (R - S)) != 0 || a.sel_nch < 1 ||
            !a.sel_gc || !a.sel_idx || a.N % 4 != 0 || (((uintptr_t)a.sel_gc) & 15) != 0 ||
            (((uintptr_t)a.Gc) & 15) != 0)
            return hipErrorInvalidValue;
    }
    return hipSuccess;
}

} // namespace

bool gemm1_f32_select_ok(Gemm1Args a) {
    G1Plan pl;
    return a.sel_sq && g1_plan(a, &pl) == hipSuccess;
}

hipError_t launch_gemm1_f32(Gemm1Args a, hipStream_t s) {
    G1Plan pl;
    const hipError_t e = g1_plan(a, &pl);
    if (e != hipSuccess)
        return e;
    return launch(pl.grid, a, pl.TM, pl.TN, pl.mode, pl.v, s);
}

hipError_t launch_gemm_fwd_f32(Gemm1Args a, hipStream_t s) {
    if (a.k_chunk % GEMM1_TK != 0 || a.splitk < 1 || a.steps < 1 || a.idx || a.m_begin != 0)
        return hipErrorInvalidValue;
    a.m_lo = 0;
    // W's rows load in pieces of consecutive k: 16 or 8 bytes where aligned
    const uintptr_t al = (uintptr_t)a.W | (uintptr_t)(4 * a.ldw) | (uintptr_t)(4L * a.kcol0);
    const int v = al % 16 == 0 ? 2 : al % 8 == 0 ? 1 : 0;
    int TM, TN;
    gemm1_tile(false, a.N, a.M, (long)a.splitk * a.steps, &TM, &TN);
    if (a.tm)
        TM = a.tm;
    if (a.tn)
        TN = a.tn;
    if (!tile_ok(TM, TN))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)ceil_div(a.M, TM), (unsigned)ceil_div(a.N, TN),
                    (unsigned)((long)a.splitk * a.steps));
    return launch(grid, a, TM, TN, G1_ROWA, v, s);
}

} // namespace lstmss
