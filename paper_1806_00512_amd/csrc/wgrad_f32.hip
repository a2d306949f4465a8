// Time-batched weight-gradient product on the compacted gate gradient, fp32
// storage, on bf16 matrix instructions (split.h); the storage-type dispatch of
// launch_wgrad.
//
// Paper: after sparsifying, the kept slices of the gate gradient are a dense
// matrix plus an offset index array, and the weight gradient
// dW[kept rows] += dG_c [x_t; h_{t-1}]^T runs on that matrix (section 3 after
// Fig. 2, section 4).
#include "split.h"
#include "wgrad.h"

namespace lstmss {

namespace {

// --------------------------------------------------------------------------
// Weight gradient of the steps of one launch, walked from the last down, so
// that dW is written (or, for a later launch of the same call, updated) once
// in a fixed summation order (deterministic, no atomics).
//
// Work-group: WR x WF wavefronts; wavefront (wr, wf) multiplies RT row tiles
// by FT feature tiles of 32.  Stages are batch chunks of 16 columns: a thread
// loads 8 consecutive columns of a row, splits them and stores one 16-byte
// piece per plane.  Four stages are in flight: while the MFMAs of stage s run
// from registers, the operands of s + 1 are read from one LDS buffer, s + 2
// is split and written to the other (whose operands were read during s - 1)
// and the global loads of s + 3 are outstanding.  A second stage of loads brought
// nothing and its registers spilled in the main loop of the 128-row groups and kept
// a third wavefront per SIMD out of others (H = I = 1024, B = 64, T = 35, us of the
// backward call: 75 % 878 -> 823, 25 % 1198 -> 1080; H = I = 2048, B = 128, T = 50 at
// 75 % 3476 -> 3002).  One barrier per stage.
//
// A step's products (at most SUM_STAGES stages of them) are summed in temporary
// tiles and added to the accumulators at once, and every other step's gate
// gradients are staged with the opposite sign and subtracted: the matrix unit
// cuts off the bits of a product below those of the sum, towards minus infinity,
// so one long sum has an error that grows with its length and a mean.  Relative
// error of dW and its mean, H = I = 2048, B = 128, T = 50, dense: one sum over all
// steps 1.21e-6, -2.2e-7; this 2.1e-7, 2e-10 (fp32 matrix instructions with a
// temporary tile per step 2.4e-7, 5e-11); H = I = 650, B = 20, T = 35: 4.3e-7, -3e-8;
// 1.3e-7, -7e-10 (1.35e-7, -6e-11).  The temporary tiles take the registers of
// 256 x 256 tiles of dW (dense call, H = 2048: 5.3 -> 5.9 ms).
//
// WG_DENSE: rows of dW are the MFMA's first operand (accumulator rows) and
// features its second (lanes).
// WG_FINE (fine structure with 32-row slices and 32-column blocks): a row
// tile is one slice and every chunk lies in one block, so the chunks of
// removed blocks skip their MFMAs (exact zeros, bit-identical).
// WG_ROUTE (coarse): wavefront row wr owns `greg` consecutive regions.  Every
// full region keeps exactly (R-S)*P rows, so at every step the group's kept
// rows are the same contiguous range of compacted rows (at most 32 RT).
// Features are the first operand and kept rows the second: the MFMAs
// accumulate a step's kept rows in temporary tiles whose lanes are kept rows;
// after the step each accumulator lane (an original row, ATN tiles) pulls its
// value from the temporary lane holding it (ds_bpermute across lanes of the
// same half), or nothing if its slice was dropped at that step.  The MFMA
// work is thus only the kept rows' (no zero-filled rows).
// --------------------------------------------------------------------------
enum WgKind { WG_DENSE = 0, WG_FINE = 1, WG_ROUTE = 2 };
// V: how batch columns load: 2: 16-byte pieces, B a multiple of 16; 1: 16-byte
// pieces, B a multiple of 4; 0: one by one
template <int WR, int WF, int RT, int FT, int ATN, int KIND, bool DBL, int V>
__global__ __launch_bounds__(WR * WF * 64, 2) void wgrad_split_kernel(WgradArgs a) {
    constexpr bool SPARSE = KIND == WG_ROUTE, FN = KIND == WG_FINE;
    constexpr int NTH = WR * WF * 64, KG = 2, TK = 8 * KG;
    constexpr int GROWS = RT * 32, NR = WR * GROWS, NF = WF * FT * 32;
    constexpr int RG = (NR * KG + NTH - 1) / NTH, RX = (NF * KG + NTH - 1) / NTH;
    __shared__ uint4 sG[2][3][KG][NR];
    __shared__ uint4 sX[2][3][KG][NF];
    // entry (kept slice number within the group) of each slice of the groups
    // at a step, -1 when dropped; written with the step's first stage (at most
    // three steps are between written and routed)
    constexpr int NSL = SPARSE ? 32 * ATN : 1;  // slices of a group (one row each at least)
    __shared__ int sinv[SPARSE ? 4 : 1][SPARSE ? WR : 1][NSL];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % WR, wf = wave / WR;
    const int I = a.I, H = a.H, B = a.B;
    const int NC = I + H, G4 = 4 * H;
    const int n0 = blockIdx.y * NF;
    const float *__restrict__ Gc = (const float *)a.Gc;
    const float *__restrict__ x = (const float *)a.x;
    const float *__restrict__ h = (const float *)a.h;

    // geometry of row group g: original rows [r0, r0 + rcount), compacted rows
    // [c0, c0 + ccount), kept-slice entries [q0, q0 + qcount), first slice j0
    const int rp = a.R * a.P, kr = (a.R - a.S) * a.P, ks = a.R - a.S;
    auto geom = [&](int g, int &r0, int &rcount, int &c0, int &ccount, int &q0, int &qcount,
                    int &j0) {
        if (SPARSE) {
            r0 = g * a.greg * rp;
            rcount = max(0, min(a.greg * rp, G4 - r0));
            c0 = g * a.greg * kr;
            ccount = max(0, min(a.greg * kr, a.Kp - c0));
            q0 = g * a.greg * ks;
            qcount = max(0, min(a.greg * ks, a.kept - q0));
            j0 = g * a.greg * a.R;
        } else {
            r0 = g * GROWS;
            rcount = max(0, min(GROWS, G4 - r0));
            c0 = r0;
            ccount = rcount;
            q0 = qcount = j0 = 0;
        }
    };
    int r0, rcount, c0, ccount, q0, qcount, j0;
    geom(blockIdx.x * WR + wr, r0, rcount, c0, ccount, q0, qcount, j0);
    // kept-slice entries and first slice of the group this wavefront loads the table of
    int lq0 = 0, lqc = 0, lj0 = 0;
    if (SPARSE && wave < WR) {
        int t0, t1, t2, t3;
        geom(blockIdx.x * WR + wave, t0, t1, t2, t3, lq0, lqc, lj0);
    }

    // staging units: 8 columns (k group kgu) of one row, fixed for the launch;
    // rows past the operands' ends are clamped to valid ones (they only feed
    // rows or columns that are never stored)
    uint32_t gofs[RG], xofs[RX];
    bool xisx[RX];
    auto slot = [](int r, int kg) { return r ^ (kg * 8); };
    const int kgu = tid % KG;  // the same for all of a thread's units
#pragma unroll
    for (int i = 0; i < RG; ++i) {
        const int rho = min((tid + i * NTH) / KG, NR - 1);
        const int k = rho / GROWS, lr = rho - k * GROWS;
        int t0, t1, lc0, lcc, t2, t3, t4;
        geom(blockIdx.x * WR + k, t0, t1, lc0, lcc, t2, t3, t4);
        gofs[i] = max(0, min(lc0 + min(lr, max(lcc - 1, 0)), (int)a.Kp - 1)) * B + 8 * kgu;
    }
#pragma unroll
    for (int i = 0; i < RX; ++i) {
        const int n = min(n0 + min((tid + i * NTH) / KG, NF - 1), NC - 1);
        xisx[i] = n < I;
        xofs[i] = (n < I ? n : n - I) * B + 8 * kgu;
    }
    // sign that step t's gate gradients are multiplied with
    auto sign = [](int t) { return t & 1 ? -1.f : 1.f; };
    // stages of the loads: step t_ld, first column b_ld; past the last stage the
    // loads repeat it (never multiplied)
    int t_ld = a.t_end - 1, b_ld = 0;
    float rg[RG][8], rx[RX][8];
    int ridx = -1;
    bool rfirst = false;      // the loaded stage is the first of its step
    float rsc = SPLIT_SCALE;  // scale and sign of its gate gradients
    auto load8 = [&](float (&r)[8], const float *p, int b) __attribute__((always_inline)) {
        if (V > 0) {  // B % 4 == 0: a piece of 4 is inside the row or past it
            float4 u = make_float4(0, 0, 0, 0), v = u;
            if (V == 2 || b < B)
                u = *(const float4 *)p;
            if (V == 2 || b + 4 < B)
                v = *(const float4 *)(p + 4);
            r[0] = u.x; r[1] = u.y; r[2] = u.z; r[3] = u.w;
            r[4] = v.x; r[5] = v.y; r[6] = v.z; r[7] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                r[j] = b + j < B ? p[j] : 0.f;
        }
    };
    auto load = [&]() __attribute__((always_inline)) {
        const float *Gt = Gc + (long)t_ld * a.Kp * B + b_ld;
        const float *xt = x + (long)t_ld * I * B + b_ld;
        const float *ht = h + (long)t_ld * H * B + b_ld;
#pragma unroll
        for (int i = 0; i < RG; ++i)
            if (NR * KG % NTH == 0 || tid + i * NTH < NR * KG)
                load8(rg[i], Gt + gofs[i], b_ld + 8 * kgu);
#pragma unroll
        for (int i = 0; i < RX; ++i)
            if (NF * KG % NTH == 0 || tid + i * NTH < NF * KG)
                load8(rx[i], (xisx[i] ? xt : ht) + xofs[i], b_ld + 8 * kgu);
        rfirst = b_ld == 0;
        rsc = sign(t_ld) * SPLIT_SCALE;
        // the step's kept-slice entries, from a clamped (always valid) position
        if (SPARSE && b_ld == 0 && wave < WR)
            ridx = a.idx[(long)t_ld * a.kept + (lqc > 0 ? lq0 + min(lane, lqc - 1) : 0)];
        b_ld += TK;
        if (b_ld >= B) {
            b_ld = 0;
            if (t_ld > a.t_begin)
                --t_ld;
        }
    };
    int step_st = 0;  // steps written to the table so far
    auto stash = [&](auto bufc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
#pragma unroll
        for (int i = 0; i < RG; ++i)
            if (NR * KG % NTH == 0 || tid + i * NTH < NR * KG)
                split_store(&sG[buf][0][kgu][slot((tid + i * NTH) / KG, kgu)], KG * NR, rg[i], rsc);
#pragma unroll
        for (int i = 0; i < RX; ++i)
            if (NF * KG % NTH == 0 || tid + i * NTH < NF * KG)
                split_store(&sX[buf][0][kgu][slot((tid + i * NTH) / KG, kgu)], KG * NF, rx[i]);
        if (SPARSE && rfirst) {
            if (wave < WR) {  // (one wavefront's LDS writes land in order)
                int *tab = sinv[step_st & 3][wave];
                for (int i = lane; i < NSL; i += 64)
                    tab[i] = -1;
                asm volatile("" ::: "memory");
                if (lane < lqc)
                    tab[ridx - lj0] = lane;
            }
            ++step_st;
        }
    };
    // FN: kept blocks of this wavefront's slices at step t
    uint64_t fmask[FN ? RT : 1] = {};
    auto block_masks = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const int sl = min((r0 >> 5) + i, (G4 >> 5) - 1);
            const int v = a.fidx[((long)t * (G4 >> 5) + sl) * a.fkept + min(lane, a.fkept - 1)];
            uint32_t lo = v < 32 ? 1u << v : 0u, hi = v >= 32 ? 1u << (v - 32) : 0u;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                lo |= __shfl_xor(lo, off, 64);
                hi |= __shfl_xor(hi, off, 64);
            }
            fmask[i] = ((uint64_t)__builtin_amdgcn_readfirstlane(hi) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane(lo);
        }
    };

    // accumulator tiles and a step's sums: dense [row tile][feature tile] both,
    // sparse [feature tile][original-row tile] and [feature tile][kept-row tile]
    constexpr int D0 = SPARSE ? FT : RT, D1 = SPARSE ? ATN : FT, E1 = SPARSE ? RT : FT;
    f32x16 acc[D0][D1], tmp[D0][E1];
    auto zero = [](f32x16 &c) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            c[v] = 0.f;
    };
    // row of dW and feature of register v of accumulator tile (i, j)
    auto dw_row = [&](int i, int j, int v) {
        return r0 + (SPARSE ? j * 32 + (lane & 31) : i * 32 + acc_row(lane, v));
    };
    auto dw_col = [&](int i, int j, int v) {
        return n0 + wf * FT * 32 + (SPARSE ? i * 32 + acc_row(lane, v) : j * 32 + (lane & 31));
    };
    // a later launch of the same call continues the sums of the earlier ones
    // from the stored dW (the same fp32 additions as one launch)
    auto init = [&](float scale) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D0; ++i)
#pragma unroll
            for (int j = 0; j < D1; ++j) {
                zero(acc[i][j]);
                if (a.accumulate) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int r = dw_row(i, j, v), f = dw_col(i, j, v);
                        const float w = a.dW[(long)min(r, G4 - 1) * NC + min(f, NC - 1)];
                        acc[i][j][v] = r < r0 + rcount && f < NC ? w * scale : 0.f;
                    }
                }
            }
    };
    auto zero_tmp = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D0; ++i)
#pragma unroll
            for (int j = 0; j < E1; ++j)
                zero(tmp[i][j]);
    };
    init(1.f / SPLIT_UNSCALE);
    zero_tmp();

    // sparse routing: accumulator lane at * 32 + lane (an original row) pulls
    // the temporary lane (kept row) that its slice's entry gives, or nothing
    // when its slice was dropped
    int rsp[ATN];  // slice within the group << 16 | row within the slice, -1: no row
    if constexpr (SPARSE) {
#pragma unroll
        for (int at = 0; at < ATN; ++at) {
            const int orow = r0 + at * 32 + (lane & 31);
            rsp[at] = at * 32 + (lane & 31) < rcount ? (orow / a.P - j0) << 16 | orow % a.P : -1;
        }
    }
    auto route = [&](int tl, float sg) __attribute__((always_inline)) {
        const int *tab = sinv[tl & 3][SPARSE ? wr : 0];
        int ent[ATN];
#pragma unroll
        for (int at = 0; at < ATN; ++at)
            ent[at] = rsp[at] >= 0 ? tab[rsp[at] >> 16] : -1;
#pragma unroll
        for (int at = 0; at < ATN; ++at) {
            const int src = ent[at] < 0 ? 0 : ent[at] * a.P + (rsp[at] & 0xffff);
            const int saddr = ((src & 31) + (lane & 32)) << 2;
            const int stile = src >> 5;
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) {
                // the permute of each temporary tile, blended by the tile
                // that holds the source (no array indexed by it)
                f32x16 w;
#pragma unroll
                for (int tt = 0; tt < RT; ++tt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float y = __int_as_float(
                            __builtin_amdgcn_ds_bpermute(saddr, __float_as_int(tmp[ft][tt][v])));
                        w[v] = tt == 0 ? y : (stile == tt ? y : w[v]);
                    }
#pragma unroll
                for (int v = 0; v < 16; ++v)  // dropped: nothing is added, even for inf/NaN
                    acc[ft][at][v] = fmaf(sg, ent[at] >= 0 ? w[v] : 0.f, acc[ft][at][v]);
            }
        }
    };

    // operands of a stage in registers (DBL: two sets, the next stage's read
    // during a stage's MFMAs; else one, read after them)
    uint4 gv[DBL ? 2 : 1][3][RT], xv[DBL ? 2 : 1][3][FT];
    auto read = [&](auto bufc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value, st = DBL ? buf : 0;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
                gv[st][p][i] = sG[buf][p][half][slot(wr * GROWS + i * 32 + (lane & 31), half)];
#pragma unroll
            for (int i = 0; i < FT; ++i)
                xv[st][p][i] = sX[buf][p][half][slot((wf * FT + i) * 32 + (lane & 31), half)];
        }
    };
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    constexpr int SUM_STAGES = 16;  // stages in one sum at most
    const int nbc = (B + TK - 1) / TK, nsteps = a.t_end - a.t_begin;
    load();
    stash(S0);
    load();
    stash(S1);
    load();
    if constexpr (FN)
        block_masks(a.t_end - 1);
    lds_barrier();
    read(S0);
    lds_barrier();
    int tl = 0, bc = 0;  // step (from the last) and chunk of the current stage
    auto stage = [&](auto pc) __attribute__((always_inline)) {
        constexpr int buf = decltype(pc)::value, st = DBL ? buf : 0;
        constexpr std::integral_constant<int, buf> P0{};
        constexpr std::integral_constant<int, 1 - buf> P1{};
        if (DBL)
            read(P1);
        if constexpr (SPARSE) {
            split_mma<FT, RT>(tmp, xv[st], gv[st]);
        } else if constexpr (FN) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
                if (!a.fskip || ((fmask[i] >> (bc * TK / 32)) & 1)) {
#pragma unroll
                    for (int p = 0; p < 6; ++p)
#pragma unroll
                        for (int j = 0; j < FT; ++j)
                            tmp[i][j] = mfma_bf(gv[st][SPLIT_A[p]][i], xv[st][SPLIT_B[p]][j], tmp[i][j]);
                }
        } else {
            split_mma<RT, FT>(tmp, gv[st], xv[st]);
        }
        ++bc;
        if (bc == nbc || (bc & (SUM_STAGES - 1)) == 0) {
            const float sg = sign(a.t_end - 1 - tl);
            if constexpr (SPARSE) {  // each kept row into its original row
                route(tl, sg);
            } else {
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < FT; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            acc[i][j][v] = fmaf(sg, tmp[i][j][v], acc[i][j][v]);
            }
            zero_tmp();
        }
        if (bc == nbc) {
            bc = 0;
            ++tl;
            if constexpr (FN)
                block_masks(max(a.t_end - 1 - tl, a.t_begin));
        }
        if (!DBL)
            read(P1);
        stash(P0);
        load();
        lds_barrier();
    };
    const int niters = nsteps * nbc;
    int it = 0;
    for (; it + 1 < niters; it += 2) {
        stage(S0);
        stage(S1);
    }
    if (it < niters)
        stage(S0);

    // an accumulator that is not finite: the tile again on the fp32 MFMA
    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < D0; ++i)
#pragma unroll
        for (int j = 0; j < D1; ++j) {
            bad += nonfinite(acc[i][j]);
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] *= SPLIT_UNSCALE;
        }
    if (__builtin_expect(__ballot(bad != bad) != 0, 0)) {
        init(1.f);
        for (int t = a.t_end - 1; t >= a.t_begin; --t) {
            const float *Gt = Gc + (long)t * a.Kp * B;
            const float *xt = x + (long)t * I * B, *ht = h + (long)t * H * B;
            auto feat = [&](int f, int b) {
                const int n = min(n0 + wf * FT * 32 + f, NC - 1);
                return n < I ? xt[(long)n * B + b] : ht[(long)(n - I) * B + b];
            };
            if constexpr (SPARSE) {
                for (int at = 0; at < ATN; ++at) {
                    const int row = r0 + at * 32 + (lane & 31);
                    const int js = row / a.P;
                    int slotr = -1;
                    if (row < r0 + rcount) {
                        const int e0 = q0 + (js - j0) / a.R * ks, e1 = min(e0 + ks, q0 + qcount);
                        for (int e = e0; e < e1; ++e)
                            if (a.idx[(long)t * a.kept + e] == js)
                                slotr = e * a.P + (row - js * a.P);
                    }
                    for (int ft = 0; ft < FT; ++ft) {
                        f32x16 c;
                        zero(c);
                        for (int b0 = 0; b0 < B; b0 += 2) {
                            const int b = b0 + half, bb = min(b, B - 1);
                            const float g = slotr >= 0 && b < B ? Gt[(long)slotr * B + bb] : 0.f;
                            const float f = feat(ft * 32 + (lane & 31), bb);
                            c = mfma32x32x2(b < B ? f : 0.f, g, c);
                        }
#pragma unroll
                        for (int i = 0; i < FT; ++i)  // (no array indexed by the loop variables)
#pragma unroll
                            for (int j = 0; j < ATN; ++j)
                                if (i == ft && j == at) {
#pragma unroll
                                    for (int v = 0; v < 16; ++v)
                                        acc[i][j][v] += slotr >= 0 ? c[v] : 0.f;
                                }
                    }
                }
            } else {
                if constexpr (FN)
                    block_masks(t);  // removed blocks stay out here too
                zero_tmp();
                for (int b0 = 0; b0 < B; b0 += 2) {
                    const int b = b0 + half, bb = min(b, B - 1);
                    float gv[RT], xv[FT];
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        const float g = Gt[(long)min(r0 + i * 32 + (lane & 31), G4 - 1) * B + bb];
                        gv[i] = b < B ? g : 0.f;
                    }
#pragma unroll
                    for (int j = 0; j < FT; ++j) {
                        const float f = feat(j * 32 + (lane & 31), bb);
                        xv[j] = b < B ? f : 0.f;
                    }
#pragma unroll
                    for (int i = 0; i < RT; ++i)
                        if (!FN || !a.fskip || ((fmask[FN ? i : 0] >> (b0 / 32)) & 1)) {
#pragma unroll
                            for (int j = 0; j < FT; ++j)
                                tmp[i][j] = mfma32x32x2(gv[i], xv[j], tmp[i][j]);
                        }
                }
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < FT; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            acc[i][j][v] += tmp[i][j][v];
            }
        }
    }

    // write the owned tile of dW
#pragma unroll
    for (int i = 0; i < D0; ++i)
#pragma unroll
        for (int j = 0; j < D1; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = dw_row(i, j, v), f = dw_col(i, j, v);
                if (r < r0 + rcount && f < NC)
                    a.dW[(long)r * NC + f] = acc[i][j][v];
            }
}

template <int WR, int WF, int RT, int FT, int ATN, int KIND, bool DBL>
hipError_t launch_split(const WgradArgs &a, long groups, int v, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div(groups, WR), (unsigned)ceil_div(a.I + a.H, WF * FT * 32));
    const dim3 block(WR * WF * 64);
    if (v == 2)
        hipLaunchKernelGGL((wgrad_split_kernel<WR, WF, RT, FT, ATN, KIND, DBL, 2>), grid, block, 0, s, a);
    else if (v == 1)
        hipLaunchKernelGGL((wgrad_split_kernel<WR, WF, RT, FT, ATN, KIND, DBL, 1>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((wgrad_split_kernel<WR, WF, RT, FT, ATN, KIND, DBL, 0>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_wgrad_f32(WgradArgs a, bool sparse, hipStream_t s) {
    const bool al = aligned16(a.Gc) && aligned16(a.x) && aligned16(a.h);
    const int v = !al || a.B % 4 != 0 ? 0 : a.B % 16 != 0 ? 1 : 2;
    const long G = 4L * a.H, NC = (long)a.I + a.H;
    // 128 x 256 tiles of dW (3/4 of the splitting per MFMA of 128 x 128) when they
    // still give every CU a work-group: H = I = 2048, B = 128, T = 50 (1024 tiles) the
    // dense call 5.8 vs 6.3 ms, H = I = 1024, B = 64, T = 35 (256 tiles) no difference
    const bool big = ceil_div(G, 128L) * ceil_div(NC, 256L) >= 256;
    if (a.fidx) {  // fine structure, 32-row slices x 32-column blocks
        if (sparse || a.B % 32 != 0 || a.fkept < 1 || a.fkept > 64 || G % 32 != 0)
            return hipErrorInvalidValue;
        return big ? launch_split<2, 4, 2, 2, 1, WG_FINE, false>(a, ceil_div(G, 64L), v, s)
                   : launch_split<2, 2, 2, 2, 1, WG_FINE, false>(a, ceil_div(G, 64L), v, s);
    }
    // sparsity 0 keeps every slice in order: the dense product, bit for bit
    if (!sparse || a.S == 0)
        return big ? launch_split<2, 4, 2, 2, 1, WG_DENSE, false>(a, ceil_div(G, 64L), v, s)
                   : launch_split<2, 2, 2, 2, 1, WG_DENSE, false>(a, ceil_div(G, 64L), v, s);
    if (!wgrad_supported(a.P, a.R, a.S))
        return hipErrorNotSupported;
    int tt = 1, at = 1;
    wgrad_tiles(a.P, a.R, a.S, &a.greg, &tt, &at);
    const long groups = ceil_div(ceil_div(G / a.P, a.R), a.greg);
    // four groups per work-group share each staged feature row (H = 2048 at
    // 50 %: 1.81 vs 1.92 ms) unless that leaves CUs idle (H = 650, B = 20:
    // 129 vs 104 us)
    const bool wide = ceil_div(groups, 4L) * ceil_div(NC, 128L) >= 256;
    if (tt == 1 && at <= 1)
        return wide ? launch_split<4, 2, 1, 2, 1, WG_ROUTE, true>(a, groups, v, s)
                    : launch_split<2, 2, 1, 2, 1, WG_ROUTE, true>(a, groups, v, s);
    if (tt == 1 && at <= 2)
        return wide ? launch_split<4, 2, 1, 2, 2, WG_ROUTE, true>(a, groups, v, s)
                    : launch_split<2, 2, 1, 2, 2, WG_ROUTE, true>(a, groups, v, s);
    if (tt == 1)
        return launch_split<2, 2, 1, 2, 4, WG_ROUTE, false>(a, groups, v, s);
    return at <= 2 ? launch_split<2, 2, 2, 1, 2, WG_ROUTE, false>(a, groups, v, s)
                   : launch_split<2, 2, 2, 1, 4, WG_ROUTE, false>(a, groups, v, s);
}

} // namespace

hipError_t launch_wgrad_bf16(WgradArgs a, bool sparse, hipStream_t s);  // wgrad_bf16.hip

bool wgrad_supported(int P, int R, int S) {
    int greg, tt, at;
    wgrad_tiles(P, R, S, &greg, &tt, &at);
    return tt <= 2 && at <= WG_ATMAX && (R - S) <= 64;
}

hipError_t launch_wgrad(WgradArgs a, bool sparse, bool bf16, hipStream_t s) {
    return bf16 ? launch_wgrad_bf16(a, sparse, s) : launch_wgrad_f32(a, sparse, s);
}

} // namespace lstmss
