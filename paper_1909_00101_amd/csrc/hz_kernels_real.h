// hz_kernels_real.h -- FP64 device bodies shared by the single-pair kernels
// (hz_real.hip) and the batched kernels (hz_batched.hip): the pivot Gram
// block of a block-column pair, the inner solve of one pivot block pair and
// the in-place block update of a row range.
#pragma once
#include "hz_device.h"
#include "hz_internal.h"

namespace hz {

// LDS (doubles) each body needs; the caller provides it, so one kernel can
// run several bodies over a single allocation.
// (gram: two regions for the waves' partial blocks with stride W2 + 2,
// which puts the 16 lanes of a tile row in distinct banks)
template <int W2> constexpr int gram_lds() { return 2 * W2 * (W2 + 2); }
template <int W2> constexpr int update_lds() { return W2 * (W2 + 1); }

// A pivot Gram block counts as numerically positive definite when every
// Cholesky pivot exceeds W2 * eps (eps = 2^-52) times that column's diagonal
// entry before the factorization: a smaller pivot is at the level of the
// factorization's own rounding errors (an exactly rank-deficient block, e.g.
// two equal columns, leaves pivots of either sign of about that size).
template <int W2> constexpr double PIV_REL() { return W2 * 2.220446049250313e-16; }
// Column stride of the inner solver's tiles in LDS: columns 16 bytes apart
// modulo the banks.
template <int W2> constexpr int inner_ld() { return W2 + 2; }
template <int W2> constexpr int inner_lds() { return 3 * W2 * inner_ld<W2>() + 128 + 16; }

// Device body: four waves form the Gram block of the block-column pair
// (p, q) of Y (m rows, ld m) over the 64-row chunks [c0, c1) and write it to
// out (column-major W2 x W2, lower tiles).  The MFMA operands come straight
// from global memory, no LDS in the loop: for X^T X both operands of a
// product hold the same kind of value (lane l: row k of the chunk's slab,
// column l % 16 of a 16-column tile), and which rows feed which k-step is
// free, so wave w takes rows 16w .. 16w + 15 of every chunk and lane group
// g = l / 16 loads rows 2g, 2g + 1 of each 8-row half as one 16-byte load:
// a column's 64 bytes are contiguous per load and every 128-byte line is
// used whole by one wave.  A wave's k-steps are, per chunk, rows
// 16w + 8h + 2g + j for (h, j) = (0,0), (0,1), (1,0), (1,1); the four
// waves' partial tiles are summed as (w0 + w1) + (w2 + w3) (tile, gram_lds
// doubles).  Further waves of a larger workgroup only take part in the
// barriers, so the sums do not depend on the workgroup size.
template <int W2>
__device__ __forceinline__ void gram_block(const double *__restrict__ Y, int64_t m, int p, int q,
                                           int64_t c0, int64_t c1, double *__restrict__ out,
                                           double *__restrict__ tile)
{
    constexpr int W = W2 / 2, NB = W2 / 16, NTL = NB * (NB + 1) / 2, PF = 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    d4 acc[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    const double *colp[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        const int cc = 16 * a + (lane & 15);
        const int gc = (cc < W) ? p * W + cc : q * W + (cc - W);
        colp[a] = Y + (int64_t)gc * m + 16 * wave + 2 * (lane >> 4);
    }
    d2 buf[PF][NB][2];
    auto load = [&](d2 (&b)[NB][2], int64_t c) {
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h) b[a][h] = *(const d2 *)(colp[a] + c * 64 + 8 * h);
    };
    auto mul = [&](const d2 (&b)[NB][2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                int t = 0;
#pragma unroll
                for (int a = 0; a < NB; ++a)
#pragma unroll
                    for (int b2 = 0; b2 <= a; ++b2, ++t)
                        acc[t] = mfma16(b[a][h][j], b[b2][h][j], acc[t]);
            }
    };
    // PF chunks in flight.  The main loop has no branch, so each chunk's
    // products wait only for that chunk's loads (a branch there made the
    // compiler wait for all of them); loads past the range are clamped to
    // its last chunk and left unused, and the remainder follows the loop.
    if (wave < 4 && c0 < c1) {
#pragma unroll
        for (int i = 0; i < PF; ++i) load(buf[i], c0 + i < c1 ? c0 + i : c1 - 1);
        int64_t c = c0;
        for (; c + PF <= c1; c += PF) {
#pragma unroll
            for (int i = 0; i < PF; ++i) {
                mul(buf[i]);
                load(buf[i], c + i + PF < c1 ? c + i + PF : c1 - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < PF - 1; ++i)
            if (c + i < c1) mul(buf[i]);
    }
    // Sum the waves' partial tiles pairwise, (w0 + w1) + (w2 + w3): waves 1
    // and 3 leave theirs in two LDS regions (tile reused, ld W2 + 2), wave 2
    // adds its own into the second, and wave 0 adds both regions to its own
    // and stores the lower tiles straight from its registers.  Element r of
    // tile (a, b) in lane l is entry (16a + 4r + l/16, 16b + l%16).
    constexpr int LDSUM = W2 + 2;
    double *const R0 = tile, *const R1 = tile + W2 * LDSUM;
    auto at = [&](int a, int b, int r) {
        return (16 * b + (lane & 15)) * LDSUM + 16 * a + 4 * r + (lane >> 4);
    };
    __syncthreads();                     // the caller's previous use of tile is over
    if (wave == 1 || wave == 3) {
        double *const R = (wave == 1) ? R0 : R1;
        int t = 0;
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b <= a; ++b, ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) R[at(a, b, r)] = acc[t][r];
    }
    __syncthreads();
    if (wave == 2) {
        int t = 0;
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b <= a; ++b, ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) R1[at(a, b, r)] = acc[t][r] + R1[at(a, b, r)];
    }
    __syncthreads();
    if (wave == 0) {
        int t = 0;
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b <= a; ++b, ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[(16 * b + (lane & 15)) * W2 + 16 * a + 4 * r + (lane >> 4)] =
                        (acc[t][r] + R0[at(a, b, r)]) + R1[at(a, b, r)];
    }
}

// The four pivot entries of a column pair (x, y) held as RPL rows per lane,
// summed over the lanes of its group (group_sum4): a_xx = f_x^T f_x, a_yy,
// a_xy, b_xy = g_x^T g_y (b_xx = b_yy = 1 after the prescaling, Section 2.1).
// Odd variants use the enhanced dot products of Appendix A.
template <int GW, int RPL, bool GEN>
__device__ __forceinline__ void pair_dots(const double (&fx)[RPL], const double (&fy)[RPL],
                                          const double (&gx)[RPL], const double (&gy)[RPL],
                                          int variant, double &axx, double &ayy, double &axy,
                                          double &bxy)
{
    axx = 0.0; ayy = 0.0; axy = 0.0; bxy = 0.0;
    if (GEN && (variant & 1)) {
        // the rounded-down products and their errors are summed apart
        double ex = 0.0, ey = 0.0, exy = 0.0, eb = 0.0;
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            edot_acc(fx[r], fx[r], axx, ex);
            edot_acc(fy[r], fy[r], ayy, ey);
            edot_acc(fx[r], fy[r], axy, exy);
            edot_acc(gx[r], gy[r], bxy, eb);
        }
        group_sum4<GW>(axx, ayy, axy, bxy);
        group_sum4<GW>(ex, ey, exy, eb);
        axx += ex;
        ayy += ey;
        axy += exy;
        bxy += eb;
    } else {
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            axx = fma(fx[r], fx[r], axx);
            ayy = fma(fy[r], fy[r], ayy);
            axy = fma(fx[r], fy[r], axy);
            bxy = fma(gx[r], gy[r], bxy);
        }
        group_sum4<GW>(axx, ayy, axy, bxy);
    }
}

// [x_i x_j] <- [x_i x_j] [[z11, z12], [z21, z22]] on RPL (even) rows per lane.
// In assembly so that both columns stay in their registers: written as
// expressions, x_i came out in fresh ones and was copied back, 24 moves to
// the 96 products of a step of 2w = 64.  Two rows are interleaved, which covers
// the latency of the products.
template <int RPL>
__device__ __forceinline__ void rotate_rows(double (&xi)[RPL], double (&xj)[RPL], double z11,
                                            double z21, double z12, double z22)
{
#pragma unroll
    for (int r = 0; r < RPL; r += 2) {
        double t, u;
        __asm__("v_mul_f64 %[t], %[a], %[z12]\n\t"
                "v_mul_f64 %[u], %[b], %[z12]\n\t"
                "v_mul_f64 %[a], %[a], %[z11]\n\t"
                "v_mul_f64 %[b], %[b], %[z11]\n\t"
                "v_fma_f64 %[a], %[c], %[z21], %[a]\n\t"
                "v_fma_f64 %[b], %[d], %[z21], %[b]\n\t"
                "v_fma_f64 %[c], %[c], %[z22], %[t]\n\t"
                "v_fma_f64 %[d], %[d], %[z22], %[u]"
                : [a] "+v"(xi[r]), [b] "+v"(xi[r + 1]), [c] "+v"(xj[r]), [d] "+v"(xj[r + 1]),
                  [t] "=&v"(t), [u] "=&v"(u)
                : [z11] "v"(z11), [z21] "v"(z21), [z12] "v"(z12), [z22] "v"(z22));
    }
}

// Phases 3 to 5 of the inner solver, with the columns in registers: F_hat,
// G_hat come as triangles in sF, sG (column-major); sF, sG, sZ (ld LDI) are
// overwritten.  A wave holds GW = 64 / LP lane groups laid side by side in
// each of its four 16-lane rows (the LP lanes of a group are strided by GW);
// a group holds a pair of columns, x for as long as the ordering lets it and
// y for one step.  GEN: any variant, with or without sorting; else variant
// 0, sorted.
//
// RING (HZ_ORD_RING).  Level by level (blocks of size 2h, h = W, W/2, ..., 1)
// group u of a block keeps column u of the block's first half as x for the
// whole level and meets every column of the second half once.  The y pass
// between the groups of a wave by lane exchanges inside the rows: one DPP
// move per word from a sub-step to the next, and a masked exchange from a
// level of h <= GW to the next one.  Only the sets of second-half columns of
// the wider levels, and the change from a wider level to the next, go
// through LDS, with one barrier each (six for 2w = 64 with 8 lanes).
//
// Round robin and modified modulus.  A step's pairs are those of the tables
// of hz_ordering; which group takes which pair follows from the step alone,
// and every column passes on through LDS, with one barrier per step.  For 2w =
// 64, where the LDS is what bounds a step, a group keeps its x (KEEP): at
// round-robin step k the kept columns are k, k - 1, ..., k - W + 1 (mod 2W -
// 1), at modified-modulus step k they are c, c - 1, ..., c - W + 1 (mod 2W) with
// c = k / 2, so that at most one group changes its x from a step to the next
// (from the lowest to the one above the highest) while the others pass only
// their y on; the steps of further sweeps go on from where the last one
// stopped.  That halves the LDS traffic for eight more selects and one
// wave's extra stores and loads: 68.5 against 84.4 us for an inner sweep at 2w
// = 64 with 16 lanes, but 20.4 against 19.9 at 2w = 32.
//
// Bound: the instructions of one or two waves per SIMD, about five cycles
// each from one wave, and in LDS the stores, 13 cycles of a compute unit for
// 64 lanes x 16 bytes.  With every column handed on through LDS after every
// step, the pivot sums taken one by one and the orderings read from a table,
// one inner sweep of 16 pivot pairs on which every pair rotates took, before
// and now: ring ordering 64.5 -> 46.4 us (2w = 64, 8 lanes) and 21.5 -> 14.2
// (2w = 32, 16 lanes); round robin 86.9 -> 68.5 (2w = 64, 16 lanes) and 25.5 ->
// 18.6 (2w = 32, 8 -> 16 lanes).
//
// The inner sweeps stop after one without big transformations, as the outer
// ones do (Section 2.5): small ones leave the block diagonal to working
// precision, and a further sweep only to see that there are none left cost an
// eighth of the inner sweeps of full-block solves (2048 x 630 94.2 -> 87.8 ms,
// the same errors against 64-bit references, also for sigma over twelve
// orders of magnitude).
template <int W2, int LP, int ORD, bool GEN>
__device__ __forceinline__ void pointwise_solve(double *__restrict__ sF, double *__restrict__ sG,
                                                double *__restrict__ sZ,
                                                unsigned *__restrict__ s_cnt, int inner_max,
                                                double tol, int sort, int variant,
                                                double *__restrict__ zt,
                                                unsigned long long *__restrict__ myc,
                                                unsigned long long *__restrict__ ph)
{
    constexpr int W = W2 / 2, NT = W * LP, RPL = W2 / LP, LDI = inner_ld<W2>();
    constexpr int GW = 64 / LP;              // groups per wave, and per 16-lane row
    constexpr int NWV = NT / 64;
    static_assert(GW == 4 || GW == 8 || GW == 16, "groups fill a 16-lane row");
    static_assert(W % GW == 0 && RPL % 2 == 0, "whole waves, rows in pairs");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane & (GW - 1), grp = wave * GW + g;
    // Rows of a lane's share of a column: pairs (16 bytes), placed for the
    // banks.  The columns of neighbouring groups lie 16 bytes apart modulo the
    // 256 bytes of the banks, and one cycle of a 16-byte load serves lanes 0-3,
    // 12-15, 20-23 and 24-27 (the next one 4-11, 16-19 and 28-31): sub takes
    // the places that GW columns leave, and the lowest bit of row, where a
    // column is long enough, the next 256 bytes -- 5.7 cycles for 64 lanes, 8.3
    // where the rows meet.
    const int row = lane >> 4, sub = (lane & 15) / GW;
    auto RI = [&](int k) {
        const int kk = k >> 1;
        const int pair = W2 == 64 ? (GW & 15) * sub + 16 * (row & 1) +
                                        (GW == 8 ? 4 * (row >> 1) + kk : (row >> 1) + 2 * kk)
                         : (GW == 8 && W2 == 32) ? row + 8 * sub + 4 * kk
                                                 : row + 4 * sub + (GW == 16 ? 4 : 0) * kk;
        return 2 * pair + (k & 1);
    };
    auto load = [&](const double *M, int c, double (&v)[RPL]) {
#pragma unroll
        for (int k = 0; k < RPL; k += 2) {
            const d2 p = *(const d2 *)(M + __umul24(c, LDI) + RI(k));
            v[k] = p[0];
            v[k + 1] = p[1];
        }
    };
    auto store = [&](double *M, int c, const double (&v)[RPL]) {
#pragma unroll
        for (int k = 0; k < RPL; k += 2) *(d2 *)(M + __umul24(c, LDI) + RI(k)) = d2{v[k], v[k + 1]};
    };
    double fx[RPL], gx[RPL], zx[RPL], fy[RPL], gy[RPL], zy[RPL];
    auto load_x = [&](int c) { load(sF, c, fx); load(sG, c, gx); load(sZ, c, zx); };
    auto load_y = [&](int c) { load(sF, c, fy); load(sG, c, gy); load(sZ, c, zy); };
    auto store_x = [&](int c) { store(sF, c, fx); store(sG, c, gx); store(sZ, c, zx); };
    auto store_y = [&](int c) { store(sF, c, fy); store(sG, c, gy); store(sZ, c, zy); };

    // the group's first columns
    constexpr bool RING = ORD == HZ_ORD_RING, MM = ORD == HZ_ORD_MM;
    constexpr bool KEEP = !RING && W2 == 64;
    int cx = grp, cy = W + grp;
    if (!RING) cy = MM ? (grp ? W2 - grp : W) : W2 - 1 - grp;
    if (KEEP) {
        cx = MM ? ((W2 - grp) & (W2 - 1)) : (grp ? W2 - 1 - grp : 0);
        cy = MM ? (grp ? grp : W) : (grp ? grp : W2 - 1);
    }

    // 3. prescale by 1/||g_c||
    load(sF, cx, fx);
    load(sG, cx, gx);
    load(sF, cy, fy);
    load(sG, cy, gy);
    {
        double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            a = fma(gx[k], gx[k], a);
            b = fma(gy[k], gy[k], b);
        }
        group_sum4<GW>(a, b, c, d);
        const double dx = rsqrt_nr(a), dy = rsqrt_nr(b);
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            fx[k] *= dx;
            gx[k] *= dx;
            zx[k] = (RI(k) == cx) ? dx : 0.0;
            fy[k] *= dy;
            gy[k] *= dy;
            zy[k] = (RI(k) == cy) ? dy : 0.0;
        }
    }
    if (ph && tid == 0) ph[3] = wall_clock64();

    // 4. inner sweeps
    const double tol2 = tol * tol;
    unsigned n_all = 0, n_big = 0, chg_any = 0;      // wave-uniform, per lane and not per group
    int nsw = 0;

    // One pointwise step on the group's pair (Section 2.1): the relative
    // orthogonality test, the 2x2 transformation, its classification (big
    // unless criterion C1, or C2 for variants 4 and 5, says small, Section
    // 2.5) and the sorting heuristic: the column with the smaller index gets
    // the larger transformed diagonal entry, which is b'' (or the larger
    // column of a pair that is orthogonal already).  first: x has the smaller
    // index (always, unless KEEP).  A pair that is left alone takes the
    // identity -- its x and a count as zero, which gives it exactly -- so that
    // the wave has one path; a wave in which every pair is left alone skips
    // it.  The lane masks are taken from plain comparisons, which cost one
    // instruction each.
    auto step = [&](bool first) {
        double axx, ayy, axy, bxy;
        pair_dots<GW, RPL, GEN>(fx, fy, gx, gy, variant, axx, ayy, axy, bxy);
        const bool orth_a = axy * axy < axx * ayy * tol2, orth_b = fabs(bxy) < tol;
        const bool lt = axx < ayy, gt = ayy < axx;
        const unsigned long long m_rot = ~(__builtin_amdgcn_ballot_w64(orth_a) &
                                           __builtin_amdgcn_ballot_w64(orth_b));
        // x is s, the smaller one (of equal ones, the one with the larger index),
        // and x gets b''; they change places where both or neither holds
        const bool xs = KEEP ? (first ? lt : !gt) : lt;
        const bool xb = (GEN && !sort) ? !xs : (KEEP ? first : true);
        const unsigned long long m_lt = __builtin_amdgcn_ballot_w64(lt),
                                 m_gt = __builtin_amdgcn_ballot_w64(gt);
        unsigned long long m_swap = m_lt;
        if (KEEP) {
            const unsigned long long m_first = __builtin_amdgcn_ballot_w64(first);
            m_swap = (m_first & m_lt) | (~m_first & m_gt);
        }
        if (GEN && !sort) m_swap = 0;
        if ((m_rot | m_swap) == 0) return;
        chg_any = 1;
        const bool orth = orth_a && orth_b;
        double rb, qb, rs, rr, t;
        hz_real_2x2_fast(axx, ayy, orth ? 0.0 : axy, orth ? 0.0 : bxy, orth, rb, qb, rs, rr, t);
        unsigned long long m_big;
        if (GEN && (variant & 4))                              // criterion C2
            m_big = __builtin_amdgcn_ballot_w64(rb * t != 1.0) |
                    __builtin_amdgcn_ballot_w64(rs * t != 1.0);
        else                                                   // criterion C1
            m_big = __builtin_amdgcn_ballot_w64(rb != 1.0) | __builtin_amdgcn_ballot_w64(rs != 1.0);
        n_all += (unsigned)__popcll(m_rot);
        n_big += (unsigned)__popcll(m_rot & m_big);
        // coefficients of x and y in b'' and s''
        const double bx = xs ? -qb : rb, by = xs ? rb : -qb;
        const double sx = xs ? rs : rr, sy = xs ? rr : rs;
        double z11 = bx, z21 = by, z12 = sx, z22 = sy;
        if (KEEP || GEN) {
            z11 = xb ? bx : sx;
            z21 = xb ? by : sy;
            z12 = xb ? sx : bx;
            z22 = xb ? sy : by;
        }
        rotate_rows<RPL>(fx, fy, z11, z21, z12, z22);
        rotate_rows<RPL>(gx, gy, z11, z21, z12, z22);
        rotate_rows<RPL>(zx, zy, z11, z21, z12, z22);
    };

    if constexpr (RING) {
        // the y of all groups by one lane exchange inside the rows
#define HZ_MOVE_Y(CTRL)                                                                        \
    _Pragma("unroll") for (int k = 0; k < RPL; ++k)                                            \
    {                                                                                          \
        fy[k] = dpp_d<CTRL>(fy[k]);                                                            \
        gy[k] = dpp_d<CTRL>(gy[k]);                                                            \
        zy[k] = dpp_d<CTRL>(zy[k]);                                                            \
    }
        // exchange of a level h <= GW with the next: groups with bit h/2 set
        // take their partner's y as x, the others their partner's x as y
        auto split = [&](int h, double (&x)[RPL], double (&y)[RPL]) {
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                const double a = x[k], b = y[k];
                if (h == 16) {
                    x[k] = dpp_into<0x128, 0xC>(a, b);       // row_ror:8
                    y[k] = dpp_into<0x128, 0x3>(b, a);
                } else if (h == 8) {
                    x[k] = dpp_into<0x114, 0xA>(a, b);       // row_shr:4
                    y[k] = dpp_into<0x104, 0x5>(b, a);       // row_shl:4
                } else if (h == 4) {
                    const double p = dpp_d<0x4E>(a), q = dpp_d<0x4E>(b);
                    x[k] = (lane & 2) ? q : a;
                    y[k] = (lane & 2) ? b : p;
                } else {
                    const double p = dpp_d<0xB1>(a), q = dpp_d<0xB1>(b);
                    x[k] = (lane & 1) ? q : a;
                    y[k] = (lane & 1) ? b : p;
                }
            }
        };
        for (;;) {
            const unsigned big0 = n_big;
            ++nsw;
            for (int h = W;; h >>= 1) {
                const int nset = (h > GW) ? h / GW : 1, ssz = (h > GW) ? GW : h;
                const int at = (grp & -h) * 2;                 // first column of the block
                const int ow = wave & (nset - 1);
                for (int p = 0;; ++p) {
                    // the offsets ring_off(0 .. ssz - 1) and back to 0, four at a time
                    for (int t = 0;;) {
                        step(true);
                        if (ssz == 1) break;
                        HZ_MOVE_Y(0xB1)                        // xor 1
                        step(true);
                        if (ssz == 2) {
                            HZ_MOVE_Y(0xB1)
                            break;
                        }
                        HZ_MOVE_Y(0x4E)                        // xor 2
                        step(true);
                        HZ_MOVE_Y(0xB1)
                        step(true);
                        t += 4;
                        if (ssz == 4) {
                            HZ_MOVE_Y(0x4E)
                        } else if (GW == 16 && ssz == 16 && (t & 7) == 0) {
                            HZ_MOVE_Y(0x128)                   // xor 8
                        } else {
                            HZ_MOVE_Y(0x141)                   // xor 7
                        }
                        if (t >= ssz) break;
                    }
                    if (p + 1 == nset) break;
                    if constexpr (GW < W) {
                        // the set to its place, the wave's next one from its place
                        store_y(at + h + GW * ((ow + p) & (nset - 1)) + g);
                        __syncthreads();
                        load_y(at + h + GW * ((ow + p + 1) & (nset - 1)) + g);
                    }
                }
                if (h == 1) break;
                if (h > GW) {
                    if constexpr (GW < W) {
                        const int hn = h >> 1, c = (grp & -hn) * 2 + (grp & (hn - 1));
                        store_x(at + (grp & (h - 1)));
                        store_y(at + h + GW * ((ow + nset - 1) & (nset - 1)) + g);
                        __syncthreads();
                        load_x(c);
                        load_y(c + hn);
                    }
                } else {
#define HZ_SPLIT(H) { split(H, fx, fy); split(H, gx, gy); split(H, zx, zy); }
                    if (h == 2) HZ_SPLIT(2)
                    else if (h == 4) HZ_SPLIT(4)
                    else if (GW >= 8 && h == 8) HZ_SPLIT(8)
                    else if (GW >= 16) HZ_SPLIT(16)
#undef HZ_SPLIT
                }
            }
            if (nsw >= inner_max) break;
            // stop after a sweep without big transformations; else back to the first level
            if (lane == 0) s_cnt[wave] = n_big - big0;
            store_x(2 * grp);
            store_y(2 * grp + 1);
            __syncthreads();
            unsigned any = 0;
            for (int w = 0; w < NWV; ++w) any |= s_cnt[w];
            if (__builtin_amdgcn_readfirstlane(any) == 0) break;
            load_x(grp);
            load_y(W + grp);
        }
        cx = 2 * grp;
        cy = 2 * grp + 1;
#undef HZ_MOVE_Y
    } else {
        constexpr int M = W2 - 1, ISTEPS = MM ? W2 : M;
        int kp = 0, kc = 0;      // step mod 2W - 1 (round robin) or 4W (modified modulus); c
        unsigned p = cx, q = cy; // !KEEP, round robin: the pair before it is ordered
        // both move on by one mod 2W - 1, but for the q = 2W - 1 of grp 0
        const unsigned qinc = grp ? 1 : 0, qmod = grp ? M : 1u << 31;
        int nx, ny;
        bool out = true, in = true;
        auto plan = [&]() {
            if constexpr (!KEEP && !MM) {
                p = min(p + 1, p + 1 - M);       // unsigned: the second wraps while p + 1 < M
                q = min(q + qinc, q + qinc - qmod);
                nx = min(p, q);
                ny = max(p, q);
                return;
            }
            const bool adv = !MM || (kp & 1);
            kp = MM ? (kp + 1) & (2 * W2 - 1) : (kp + 1 < M ? kp + 1 : 0);
            int pos = grp;
            if (KEEP) {
                const bool mine = adv && ((W - 1 - kc) & (W - 1)) / GW == wave;
                out = mine && ((kc + grp) & (W - 1)) == W - 1;
                if (adv) ++kc;
                pos = (kc + grp) & (W - 1);
                in = mine && pos == 0;
            }
            int x, y;
            if (MM) {
                x = ((kp >> 1) - pos) & (W2 - 1);
                y = (kp - x) & (W2 - 1);
                y = (y == x) ? x ^ W : y;
            } else {
                x = kp - pos;
                x += (x < 0) ? M : 0;
                y = kp + pos;
                y -= (y >= M) ? M : 0;
                y = (pos == 0) ? M : y;
            }
            nx = KEEP ? x : min(x, y);
            ny = KEEP ? y : max(x, y);
        };
        auto leave = [&]() {
            store_y(cy);
            if (!KEEP || out) store_x(cx);
        };
        auto enter = [&]() {
            cx = nx;
            cy = ny;
            load_y(cy);
            if (!KEEP || in) load_x(cx);
        };
        for (;;) {
            const unsigned big0 = n_big;
            ++nsw;
            for (int st = 1; st < ISTEPS; ++st) {
                plan();
                step(cx < cy);
                leave();
                __syncthreads();
                enter();
            }
            step(cx < cy);
            if (nsw >= inner_max) break;
            // stop after a sweep without big transformations
            plan();
            leave();
            if (lane == 0) s_cnt[wave] = n_big - big0;
            __syncthreads();
            unsigned any = 0;
            for (int w = 0; w < NWV; ++w) any |= s_cnt[w];
            if (__builtin_amdgcn_readfirstlane(any) == 0) break;
            enter();
        }
    }
    if (ph && tid == 0) ph[4] = wall_clock64();

    // 5. Theta rescale and write Z_tilde (column-major W2 x W2); the identity
    // when nothing was transformed or swapped.
    __syncthreads();                         // s_cnt free
    if (lane == 0) {
        s_cnt[3 * wave] = n_all / LP;
        s_cnt[3 * wave + 1] = n_big / LP;
        s_cnt[3 * wave + 2] = chg_any;
    }
    __syncthreads();
    unsigned ta = 0, tb = 0, tc = 0;
    for (int w = 0; w < NWV; ++w) {
        ta += s_cnt[3 * w];
        tb += s_cnt[3 * w + 1];
        tc |= s_cnt[3 * w + 2];
    }
    const bool changed = __builtin_amdgcn_readfirstlane(tc) != 0;
    double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        a = fma(gx[k], gx[k], fma(fx[k], fx[k], a));
        b = fma(gy[k], gy[k], fma(fy[k], fy[k], b));
    }
    group_sum4<GW>(a, b, c, d);
    const double tx = rsqrt_nr(a), ty = rsqrt_nr(b);
    auto unit = [](bool p) { return p ? 1.0 : 0.0; };
#pragma unroll
    for (int k = 0; k < RPL; k += 2) {
        const int r = RI(k);
        *(d2 *)(zt + cx * W2 + r) = changed ? d2{zx[k] * tx, zx[k + 1] * tx}
                                            : d2{unit(r == cx), unit(r + 1 == cx)};
        *(d2 *)(zt + cy * W2 + r) = changed ? d2{zy[k] * ty, zy[k + 1] * ty}
                                            : d2{unit(r == cy), unit(r + 1 == cy)};
    }
    if (tid == 0) {
        myc[0] = ta;
        myc[1] = tb;
        myc[2] = (unsigned long long)nsw;
        myc[3] = changed ? 0ull : 1ull;
        if (ph) ph[5] = wall_clock64();
    }
}

// Device body: the workgroup (NT threads) solves the block pair whose Gram
// blocks are pa (F) and pb (G) (column-major W2 x W2, lower triangles),
// writes Z_tilde to zt, the counters (transformations, big ones, inner
// sweeps) to myc[0..2] and to myc[3] whether Z_tilde is the identity, and
// on a non-positive pivot sets FLAG_CHOL in status[ST_FLAGS] and failcode
// into status[ST_FAILPAIR] (minimum kept).  When no pair of the block was
// transformed or swapped, Z_tilde is the diagonal Theta-scaled prescale,
// which only renormalizes columns that already have ||f_j||^2 + ||g_j||^2 =
// 1 up to rounding; it is then set to I exactly and myc[3] = 1, so the
// block update may be skipped (Section 2.5).
template <int W2, int LP, int ORD, bool GEN>
__device__ __forceinline__ void inner_solve(
    const double *__restrict__ pa, const double *__restrict__ pb, int nsplit, size_t sstride,
    int inner_max, double tol, int sort, int variant, double *__restrict__ zt,
    unsigned long long *__restrict__ myc, int *__restrict__ status, int failcode, unsigned long long *__restrict__ ph, double *__restrict__ lds)
{
    constexpr int NT = (W2 / 2) * LP;
    constexpr int LDI = inner_ld<W2>();
    static_assert(NT >= 64, "bad inner geometry");
    double *const sF = lds;
    double *const sG = lds + W2 * LDI;
    double *const sZ = lds + 2 * W2 * LDI;
    double *const lbuf0 = lds + 3 * W2 * LDI;                 // 2 x 64 doubles
    unsigned *const s_cnt = (unsigned *)(lbuf0 + 128);        // 3 words per wave
    int *const s_failp = (int *)(s_cnt + 3 * (NT / 64));
#define s_fail (*s_failp)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (ph && tid == 0) ph[0] = wall_clock64();
    // 1. load the Gram blocks (lower triangles) into LDS; with nsplit > 1 the
    // blocks arrive as nsplit row-split partials (stride sstride), added in
    // split order; with nsplit 0 they are the upper triangular factors
    // themselves (QR of the block-column pairs).
    if (nsplit <= 1) {
        // one summed block (or a factor): every load of a thread issued
        // before the first store, so the phase costs one memory latency
        constexpr int NIT = (W2 * W2) / (2 * NT);
        static_assert(NIT * 2 * NT == W2 * W2, "Gram load geometry");
        d2 va[NIT], vb[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = 2 * tid + 2 * NT * it;
            // upper tiles of a Gram are never read (zeros go to LDS); a factor
            // (nsplit 0) is upper
            const bool skip = nsplit > 0 && (e / W2) / 16 > (e % W2) / 16;
            va[it] = skip ? d2{0.0, 0.0} : *(const d2 *)(pa + e);
            vb[it] = skip ? d2{0.0, 0.0} : *(const d2 *)(pb + e);
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = 2 * tid + 2 * NT * it, col = e / W2, row = e % W2;
            *(d2 *)(sF + col * LDI + row) = va[it];
            *(d2 *)(sG + col * LDI + row) = vb[it];
        }
        if (tid == 0) s_fail = 0;
    } else {
        for (int e = 2 * tid; e < W2 * W2; e += 2 * NT) {
            // upper tiles of a Gram are never read
            if ((e / W2) / 16 > (e % W2) / 16) continue;
            d2 a = *(const d2 *)(pa + e), b = *(const d2 *)(pb + e);
            for (int sp = 1; sp < nsplit; ++sp) {
                a += *(const d2 *)(pa + sp * sstride + e);
                b += *(const d2 *)(pb + sp * sstride + e);
            }
            const int col = e / W2, row = e % W2;
            *(d2 *)(sF + col * LDI + row) = a;
            *(d2 *)(sG + col * LDI + row) = b;
        }
        if (tid == 0) s_fail = 0;
    }
    __syncthreads();
    if (ph && tid == 0) ph[1] = wall_clock64();

    // 2. Cholesky factorizations, lane = row, one wave per matrix.  With
    // nsplit 0 the factors came in (QR of the block-column pairs): only their
    // diagonals are checked for zeros and non-finite values.
    if (nsplit == 0) {
        if (tid < W2) {
            const double df = sF[tid * LDI + tid], dg = sG[tid * LDI + tid];
            if (!(fabs(df) > 0.0 && fabs(df) < INFINITY && fabs(dg) > 0.0 && fabs(dg) < INFINITY))
                s_fail = 1;
        }
    } else if constexpr (W2 >= 32 && NT >= 128) {
        // Blocked right-looking Cholesky, one wave per matrix, panels of 16
        // columns (2w = 32 or 64; lanes past the block's rows idle).  A
        // panel (its rows c0.. of columns c0..c0+15, lane = row) is factored
        // in registers, the entries of a column reaching the later panel
        // columns by readlane; the panel goes back to LDS and the trailing
        // lower tiles take the update A22 -= L21 L21^T as FP64 MFMA products
        // (tile (ti, tj): A operand L rows of ti, B operand L rows of tj,
        // four k-steps of 4 panel columns).
        constexpr int NBK = W2 / 16;
        if (wave < 2) {
            double *M = wave ? sG : sF;
            bool ok = true;
            // lane j (< 16) holds the diagonals of columns 16 kb + j before
            // the factorization; it tests the pivot of that column itself
            // once the panel is factored
            double d0[NBK];
#pragma unroll
            for (int kb = 0; kb < NBK; ++kb)
                d0[kb] = (lane < 16) ? M[(16 * kb + lane) * LDI + 16 * kb + lane] : 1.0;
#pragma unroll
            for (int kb = 0; kb < NBK; ++kb) {
                const int c0 = 16 * kb, row = c0 + lane;
                const bool live = row < W2;
                double pv[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) pv[t] = live ? M[(c0 + t) * LDI + row] : 0.0;
                double own = 1.0;           // lane j: the pivot of column c0 + j
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const double piv = readlane_d(pv[j], j);
                    if (lane == j) own = pv[j];
                    const double inv = rsqrt_nr(piv);
                    const double l = (lane >= j) ? pv[j] * inv : 0.0;
                    pv[j] = l;
#pragma unroll
                    for (int t = j + 1; t < 16; ++t) pv[t] = fma(-l, readlane_d(l, t), pv[t]);
                }
                if (lane < 16) ok = ok && (own > PIV_REL<W2>() * d0[kb]) && (own < INFINITY);
                if (live) {
#pragma unroll
                    for (int t = 0; t < 16; ++t) M[(c0 + t) * LDI + row] = pv[t];
                }
                wave_fence();
                const int i16 = lane & 15, k4 = lane >> 4;
#pragma unroll
                for (int ti = kb + 1; ti < NBK; ++ti)
#pragma unroll
                    for (int tj = kb + 1; tj <= ti; ++tj) {
                        // element r of lane l: row 16 ti + 4 r + l/16, column 16 tj + l%16
                        double *const ct = M + (16 * tj + i16) * LDI + 16 * ti + k4;
                        d4 acc = d4{ct[0], ct[4], ct[8], ct[12]};
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const double *const lc = M + (c0 + 4 * s + k4) * LDI;
                            acc = mfma16(-lc[16 * ti + i16], lc[16 * tj + i16], acc);
                        }
                        ct[0] = acc[0];
                        ct[4] = acc[1];
                        ct[8] = acc[2];
                        ct[12] = acc[3];
                    }
                wave_fence();
            }
            // F_hat = L^T: column i of F_hat is row i of L.
            double a[W2];
            if (lane < W2) {
#pragma unroll
                for (int k = 0; k < W2; ++k) a[k] = M[k * LDI + lane];
            }
            wave_fence();
            if (lane < W2) {
#pragma unroll
                for (int k = 0; k < W2; ++k) M[lane * LDI + k] = (k <= lane) ? a[k] : 0.0;
            }
            if (!ok) s_fail = 1;
        }
    } else {
        constexpr bool two = (W2 == 64);
        const int mat = two ? wave : (lane >> 5);
        const int i = two ? lane : (lane & 31);
        if ((two ? (wave < 2) : (wave == 0)) && i < W2) {
            double *M = mat ? sG : sF;
            double *lb = lbuf0 + 64 * mat;
            double a[W2];
#pragma unroll
            for (int k = 0; k < W2; ++k) a[k] = M[k * LDI + i];
            const double d0 = M[i * LDI + i];    // column i's diagonal before the factorization
            double own = 1.0;                      // the pivot of column i, kept by lane i
#pragma unroll
            for (int j = 0; j < W2; ++j) {
                double piv;
                if (two) {
                    piv = readlane_d(a[j], j);
                } else {
                    const double p0 = readlane_d(a[j], j), p1 = readlane_d(a[j], 32 + j);
                    piv = mat ? p1 : p0;
                }
                if (i == j) own = a[j];
                const double inv = rsqrt_nr(piv);
                const double l = (i >= j) ? a[j] * inv : 0.0;
                a[j] = l;
                lb[i] = l;
                wave_fence();
#pragma unroll
                for (int k = j + 1; k < W2; k += 2) {
                    const d2 lk = *(const d2 *)(lb + k - (k & 1));
                    if (k & 1) {
                        a[k] = fma(-l, lk[1], a[k]);
                        if (k + 1 < W2) a[k + 1] = fma(-l, (*(const d2 *)(lb + k + 1))[0], a[k + 1]);
                    } else {
                        a[k] = fma(-l, lk[0], a[k]);
                        if (k + 1 < W2) a[k + 1] = fma(-l, lk[1], a[k + 1]);
                    }
                }
                wave_fence();
            }
            // F_hat = L^T: column i of F_hat is row i of L.
#pragma unroll
            for (int k = 0; k < W2; ++k) M[i * LDI + k] = (k <= i) ? a[k] : 0.0;
            if (!((own > PIV_REL<W2>() * d0) && (own < INFINITY))) s_fail = 1;
        }
    }
    __syncthreads();
    if (ph && tid == 0) ph[2] = wall_clock64();
    if (__builtin_amdgcn_readfirstlane(s_fail)) {      // uniform: every lane read the same word
        for (int e = tid; e < W2 * W2; e += NT) zt[e] = (e % W2 == e / W2) ? 1.0 : 0.0;
        if (tid == 0) {
            myc[0] = 0;
            myc[1] = 0;
            myc[2] = 0;
            myc[3] = 0;
            atomicOr(status + ST_FLAGS, FLAG_CHOL);
            atomicMin(status + ST_FAILPAIR, failcode);
        }
        return;
    }

    pointwise_solve<W2, LP, ORD, GEN>(sF, sG, sZ, s_cnt, inner_max, tol, sort, variant, zt, myc, ph);
#undef s_fail
}

// Device body: one workgroup of NW waves updates the rows [rb, re) (a
// multiple of 16 rows) of a row sequence by zt (column-major W2 x W2),
// staged in LDS (sz, update_lds<W2>() doubles).  locate(v, Y, m, r) maps
// sequence row v (the first of a 16-row tile, which never straddles two
// matrices) to the matrix Y (ld m) and its row r; in Y the block-column
// pair (p, q) is updated.
template <int W2, int NW, class Locate>
__device__ __forceinline__ void update_row_seq(Locate locate, int p, int q, int64_t rb,
                                               int64_t re, const double *__restrict__ zt,
                                               double *__restrict__ sz)
{
    constexpr int W = W2 / 2, NB = W2 / 16, KS = W2 / 4, LDZ = W2 + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NTH = 64 * NW;
    if constexpr ((W2 * W2) % NTH == 0) {
        // every load of a thread issued before the first store: one memory
        // latency before the rows can start instead of one per element
        constexpr int NZ = (W2 * W2) / NTH;
        double zv[NZ];
#pragma unroll
        for (int it = 0; it < NZ; ++it) zv[it] = zt[tid + NTH * it];
#pragma unroll
        for (int it = 0; it < NZ; ++it) {
            const int e = tid + NTH * it;
            sz[(e / W2) * LDZ + (e % W2)] = zv[it];
        }
    } else {
        for (int e = tid; e < W2 * W2; e += NTH) sz[(e / W2) * LDZ + (e % W2)] = zt[e];
    }
    __syncthreads();
    // Lane (i, k) = (lane % 16, lane / 16).  Columns 0..W-1 of the pair are
    // block column p, W..2W-1 block column q; every k-step's column offset
    // is a uniform multiple of m.
    const int k4 = lane >> 4, i16 = lane & 15;
    for (int64_t v0 = rb + 16 * wave; v0 < re; v0 += 16 * NW) {
        // keep the Z_tilde fragment reads inside the loop (in LDS, not in
        // 128 registers hoisted out of it)
        __asm__ volatile("" ::: "memory");
        double *Y;
        int64_t m, r0;
        locate(v0, Y, m, r0);
        const double *bp = Y + ((int64_t)p * W + k4) * m + i16;
        const double *bq = Y + ((int64_t)q * W + k4) * m + i16;
        double xb[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s)
            xb[s] = (4 * s < W) ? bp[(int64_t)(4 * s) * m + r0] : bq[(int64_t)(4 * s - W) * m + r0];
        d4 acc[NB];
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) acc[jb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                // A'[j][k] = Z_tilde[4s+k][16jb+j], lane j + 16k
                const double za = sz[(16 * jb + i16) * LDZ + 4 * s + k4];
                acc[jb] = mfma16(za, xb[s], acc[jb]);
            }
        // element r of acc[jb] in lane l is output column 16jb + 4r + l/16, row l%16
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c0 = 16 * jb + 4 * r;
                double *dst = (c0 < W) ? (double *)bp + (int64_t)c0 * m + r0
                                       : (double *)bq + (int64_t)(c0 - W) * m + r0;
                *dst = acc[jb][r];
            }
    }
}

// The same for the rows [rb, re) of one matrix Y (ld m).
template <int W2, int NW>
__device__ __forceinline__ void update_rows(double *__restrict__ Y, int64_t m, int p, int q,
                                            int64_t rb, int64_t re,
                                            const double *__restrict__ zt,
                                            double *__restrict__ sz)
{
    update_row_seq<W2, NW>(
        [=](int64_t v, double *&y, int64_t &ld, int64_t &r) {
            y = Y;
            ld = m;
            r = v;
        },
        p, q, rb, re, zt, sz);
}

}  // namespace hz
