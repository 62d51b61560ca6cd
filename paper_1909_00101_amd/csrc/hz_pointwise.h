// hz_pointwise.h -- the pointwise sweeps of the inner solvers, real and complex:
// one pivot block pair's triangular factors in LDS, their columns in registers
// (Sections 2.1, 2.4, 2.5 and 3.5.3 of the paper).
#pragma once
#include "hz_device.h"
#include "hz_internal.h"

namespace hz {

// The four pivot entries of a column pair (x, y) held as ND rows per lane,
// summed over the lanes of its group (group_sum4): a_xx = f_x^T f_x, a_yy,
// a_xy, b_xy = g_x^T g_y (b_xx = b_yy = 1 after the prescaling, Section 2.1).
// Odd variants use the enhanced dot products of Appendix A.
template <int GW, int ND, bool GEN>
__device__ __forceinline__ void pair_dots(const double (&fx)[ND], const double (&fy)[ND],
                                          const double (&gx)[ND], const double (&gy)[ND],
                                          int variant, double &axx, double &ayy, double &axy,
                                          double &bxy)
{
    axx = 0.0; ayy = 0.0; axy = 0.0; bxy = 0.0;
    if (GEN && (variant & 1)) {
        // the rounded-down products and their errors are summed apart
        double ex = 0.0, ey = 0.0, exy = 0.0, eb = 0.0;
#pragma unroll
        for (int r = 0; r < ND; ++r) {
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
        for (int r = 0; r < ND; ++r) {
            axx = fma(fx[r], fx[r], axx);
            ayy = fma(fy[r], fy[r], ayy);
            axy = fma(fx[r], fy[r], axy);
            bxy = fma(gx[r], gy[r], bxy);
        }
        group_sum4<GW>(axx, ayy, axy, bxy);
    }
}

// [x_i x_j] <- [x_i x_j] [[z11, z12], [z21, z22]] on ND (even) rows per lane.
// In assembly so that both columns stay in their registers: written as
// expressions, x_i came out in fresh ones and was copied back, 24 moves to
// the 96 products of a step of 2w = 64.  Two rows are interleaved, which covers
// the latency of the products.
template <int ND>
__device__ __forceinline__ void rotate_rows(double (&xi)[ND], double (&xj)[ND], double z11,
                                            double z21, double z12, double z22)
{
#pragma unroll
    for (int r = 0; r < ND; r += 2) {
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

// Complex columns (re, im interleaved), in place as above: x <- ox x + cx y, y <-
// oy y + cy x with real ox, oy (12 products per entry pair) ...
template <int ND>
__device__ __forceinline__ void rotate_own(double (&x)[ND], double (&y)[ND], double ox, double cxr,
                                           double cxi, double oy, double cyr, double cyi)
{
#pragma unroll
    for (int k = 0; k < ND; k += 2) {
        double t, u;
        __asm__("v_mul_f64 %[t], %[a], %[cyr]\n\t"
                "v_mul_f64 %[u], %[b], %[cyr]\n\t"
                "v_fma_f64 %[t], -%[b], %[cyi], %[t]\n\t"
                "v_fma_f64 %[u], %[a], %[cyi], %[u]\n\t"
                "v_mul_f64 %[a], %[a], %[ox]\n\t"
                "v_mul_f64 %[b], %[b], %[ox]\n\t"
                "v_fma_f64 %[a], %[c], %[cxr], %[a]\n\t"
                "v_fma_f64 %[b], %[d], %[cxr], %[b]\n\t"
                "v_fma_f64 %[a], -%[d], %[cxi], %[a]\n\t"
                "v_fma_f64 %[b], %[c], %[cxi], %[b]\n\t"
                "v_fma_f64 %[c], %[c], %[oy], %[t]\n\t"
                "v_fma_f64 %[d], %[d], %[oy], %[u]"
                : [a] "+v"(x[k]), [b] "+v"(x[k + 1]), [c] "+v"(y[k]), [d] "+v"(y[k + 1]),
                  [t] "=&v"(t), [u] "=&v"(u)
                : [ox] "v"(ox), [cxr] "v"(cxr), [cxi] "v"(cxi), [oy] "v"(oy), [cyr] "v"(cyr),
                  [cyi] "v"(cyi));
    }
}

// ... and [x y] <- [x y] [[p11, p12], [p21, p22]] with complex entries (16).
template <int ND>
__device__ __forceinline__ void rotate_any(double (&x)[ND], double (&y)[ND], double p11r,
                                           double p11i, double p21r, double p21i, double p12r,
                                           double p12i, double p22r, double p22i)
{
#pragma unroll
    for (int k = 0; k < ND; k += 2) {
        double t, u, v, w;
        __asm__("v_mul_f64 %[t], %[a], %[p12r]\n\t"
                "v_mul_f64 %[u], %[b], %[p12r]\n\t"
                "v_mul_f64 %[v], %[b], %[p11i]\n\t"
                "v_mul_f64 %[w], %[a], %[p11i]\n\t"
                "v_fma_f64 %[t], -%[b], %[p12i], %[t]\n\t"
                "v_fma_f64 %[u], %[a], %[p12i], %[u]\n\t"
                "v_fma_f64 %[a], %[a], %[p11r], -%[v]\n\t"
                "v_fma_f64 %[b], %[b], %[p11r], %[w]\n\t"
                "v_fma_f64 %[t], -%[d], %[p22i], %[t]\n\t"
                "v_fma_f64 %[u], %[c], %[p22i], %[u]\n\t"
                "v_fma_f64 %[a], %[c], %[p21r], %[a]\n\t"
                "v_fma_f64 %[b], %[d], %[p21r], %[b]\n\t"
                "v_fma_f64 %[a], -%[d], %[p21i], %[a]\n\t"
                "v_fma_f64 %[b], %[c], %[p21i], %[b]\n\t"
                "v_fma_f64 %[c], %[c], %[p22r], %[t]\n\t"
                "v_fma_f64 %[d], %[d], %[p22r], %[u]"
                : [a] "+v"(x[k]), [b] "+v"(x[k + 1]), [c] "+v"(y[k]), [d] "+v"(y[k + 1]),
                  [t] "=&v"(t), [u] "=&v"(u), [v] "=&v"(v), [w] "=&v"(w)
                : [p11r] "v"(p11r), [p11i] "v"(p11i), [p21r] "v"(p21r), [p21i] "v"(p21i),
                  [p12r] "v"(p12r), [p12i] "v"(p12i), [p22r] "v"(p22r), [p22i] "v"(p22i));
    }
}

// A pair of columns (x, y) of a lane group in registers, ND doubles per lane
// of F_hat, G_hat and Z_hat each.
template <int ND> struct ColPair {
    double fx[ND], gx[ND], zx[ND], fy[ND], gy[ND], zy[ND];
};

// What a step needs to know, and the counters it adds to (wave-uniform; per
// lane, so LP times the groups' counts).
struct StepArgs {
    double tol, tol2;
    int sort, variant;
    unsigned n_all, n_big;
};

// The lanes whose pair's columns change places: x, the first or second of the
// pair by index, and the larger column belong together when sorting.
template <bool KEEP, bool GEN>
__device__ __forceinline__ unsigned long long swap_mask(bool lt, bool gt, bool first, int sort)
{
    const unsigned long long m_lt = __builtin_amdgcn_ballot_w64(lt);
    if (GEN && !sort) return 0;
    if (!KEEP) return m_lt;
    const unsigned long long m_gt = __builtin_amdgcn_ballot_w64(gt),
                             m_first = __builtin_amdgcn_ballot_w64(first);
    return (m_first & m_lt) | (~m_first & m_gt);
}

// Counts the transformations of the lanes in m_rot and the big ones among
// them, from the scaled cosines rb, rs (criterion C1) or, for variants 4 and 5,
// from the unscaled ones (C2).
template <bool GEN>
__device__ __forceinline__ void count_big(double rb, double rs, double t, unsigned long long m_rot,
                                          StepArgs &A)
{
    unsigned long long m_big;
    if (GEN && (A.variant & 4))
        m_big = __builtin_amdgcn_ballot_w64(rb * t != 1.0) |
                __builtin_amdgcn_ballot_w64(rs * t != 1.0);
    else
        m_big = __builtin_amdgcn_ballot_w64(rb != 1.0) | __builtin_amdgcn_ballot_w64(rs != 1.0);
    A.n_all += (unsigned)__popcll(m_rot);
    A.n_big += (unsigned)__popcll(m_rot & m_big);
}

// Real columns: a 16-byte slot holds two rows.
struct RealCols {
    template <int W2> static constexpr int slots() { return W2 / 2; }
    // entry e of slot p in the unit column c
    static __device__ __forceinline__ double unit(int p, int e, int c)
    {
        return (2 * p + e == c) ? 1.0 : 0.0;
    }
    // slot p of column c of L^T, L lower in M (ld ldc)
    static __device__ __forceinline__ d2 of_lower(const double *M, int ldc, int p, int c)
    {
        const double a = M[2 * p * ldc + c], b = M[(2 * p + 1) * ldc + c];
        return d2{2 * p <= c ? a : 0.0, 2 * p + 1 <= c ? b : 0.0};
    }

    // One pointwise step on the group's pair (Section 2.1): the relative
    // orthogonality test, the 2x2 transformation, its classification (big
    // unless criterion C1, or C2 for variants 4 and 5, says small, Section
    // 2.5) and the sorting heuristic: the column with the smaller index gets
    // the larger transformed diagonal entry, which is b'' (or the larger
    // column of a pair that is orthogonal already).  first: x has the smaller
    // index (always, unless KEEP).  A pair that is left alone takes the
    // identity -- its x counts as zero, which gives it exactly -- so that
    // the wave has one path; a wave in which every pair is left alone skips
    // it.  The lane masks are taken from plain comparisons, which cost one
    // instruction each.  Returns whether any pair of the wave changes.
    template <int GW, int ND, bool KEEP, bool GEN>
    static __device__ __forceinline__ bool step(ColPair<ND> &c, bool first, StepArgs &A)
    {
        double axx, ayy, axy, bxy;
        pair_dots<GW, ND, GEN>(c.fx, c.fy, c.gx, c.gy, A.variant, axx, ayy, axy, bxy);
        const bool orth_a = axy * axy < axx * ayy * A.tol2, orth_b = fabs(bxy) < A.tol;
        const bool lt = axx < ayy, gt = ayy < axx;
        const unsigned long long m_rot = ~(__builtin_amdgcn_ballot_w64(orth_a) &
                                           __builtin_amdgcn_ballot_w64(orth_b));
        // x is s, the smaller one (of equal ones, the one with the larger index),
        // and x gets b''; they change places where both or neither holds
        const bool xs = KEEP ? (first ? lt : !gt) : lt;
        const bool xb = (GEN && !A.sort) ? !xs : (KEEP ? first : true);
        const unsigned long long m_swap = swap_mask<KEEP, GEN>(lt, gt, first, A.sort);
        if ((m_rot | m_swap) == 0) return false;
        const bool orth = orth_a && orth_b;
        double rb, qb, rs, rr, t;
        hz_real_2x2_fast(axx, ayy, axy, orth ? 0.0 : bxy, orth, rb, qb, rs, rr, t);
        count_big<GEN>(rb, rs, t, m_rot, A);
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
        rotate_rows<ND>(c.fx, c.fy, z11, z21, z12, z22);
        rotate_rows<ND>(c.gx, c.gy, z11, z21, z12, z22);
        rotate_rows<ND>(c.zx, c.zy, z11, z21, z12, z22);
        return true;
    }
};

// Complex columns: a slot holds one entry.
struct CplxCols {
    template <int W2> static constexpr int slots() { return W2; }
    static __device__ __forceinline__ double unit(int p, int e, int c)
    {
        return (p == c && e == 0) ? 1.0 : 0.0;
    }

    // As the real step, with the complex 2x2 transformation (Section 2.1.1).
    // x and y have real coefficients of their own and complex ones of each
    // other, unless they change places.
    template <int GW, int ND, bool KEEP, bool GEN>
    static __device__ __forceinline__ bool step(ColPair<ND> &c, bool first, StepArgs &A)
    {
        double axx = 0.0, ayy = 0.0, ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;
#pragma unroll
        for (int k = 0; k < ND; k += 2) {
            if (GEN && (A.variant & 1)) {
                // variants 1 and 5: squared norms by the enhanced procedure of
                // Appendix A (the off-diagonal entries stay ordinary)
                axx += enh_abs2(c.fx[k], c.fx[k + 1]);
                ayy += enh_abs2(c.fy[k], c.fy[k + 1]);
            } else {
                axx = fma(c.fx[k], c.fx[k], fma(c.fx[k + 1], c.fx[k + 1], axx));
                ayy = fma(c.fy[k], c.fy[k], fma(c.fy[k + 1], c.fy[k + 1], ayy));
            }
            ar = fma(c.fx[k], c.fy[k], fma(c.fx[k + 1], c.fy[k + 1], ar));
            ai = fma(c.fx[k], c.fy[k + 1], fma(-c.fx[k + 1], c.fy[k], ai));
            br = fma(c.gx[k], c.gy[k], fma(c.gx[k + 1], c.gy[k + 1], br));
            bi = fma(c.gx[k], c.gy[k + 1], fma(-c.gx[k + 1], c.gy[k], bi));
        }
        group_sum4<GW>(axx, ayy, ar, ai);
        group_sum2<GW>(br, bi);
        const bool orth_a = fma(ar, ar, ai * ai) < axx * ayy * A.tol2;
        const bool orth_b = fma(br, br, bi * bi) < A.tol2;
        const bool lt = axx < ayy, gt = ayy < axx;
        const unsigned long long m_rot = ~(__builtin_amdgcn_ballot_w64(orth_a) &
                                           __builtin_amdgcn_ballot_w64(orth_b));
        const bool xs = KEEP ? (first ? lt : !gt) : lt;
        const unsigned long long m_swap = swap_mask<KEEP, GEN>(lt, gt, first, A.sort);
        if ((m_rot | m_swap) == 0) return false;
        const bool orth = orth_a && orth_b;
        // oriented from b to s
        const double sg = xs ? -1.0 : 1.0;
        double rb, cbr, cbi, rs, csr, csi, t;
        hz_cplx_2x2_fast(xs ? ayy : axx, xs ? axx : ayy, ar, sg * ai, orth ? 0.0 : br,
                         orth ? 0.0 : sg * bi, orth, rb, cbr, cbi, rs, csr, csi, t);
        count_big<GEN>(rb, rs, t, m_rot, A);
        const double ox = xs ? rs : rb, oy = xs ? rb : rs;
        const double cxr = xs ? csr : cbr, cxi = xs ? csi : cbi;
        const double cyr = xs ? cbr : csr, cyi = xs ? cbi : csi;
        if (m_swap == 0) {
            rotate_own<ND>(c.fx, c.fy, ox, cxr, cxi, oy, cyr, cyi);
            rotate_own<ND>(c.gx, c.gy, ox, cxr, cxi, oy, cyr, cyi);
            rotate_own<ND>(c.zx, c.zy, ox, cxr, cxi, oy, cyr, cyi);
        } else {
            const bool sw = KEEP ? (xs == first) : lt;
            const double p11r = sw ? cyr : ox, p11i = sw ? cyi : 0.0;
            const double p21r = sw ? oy : cxr, p21i = sw ? 0.0 : cxi;
            const double p12r = sw ? ox : cyr, p12i = sw ? 0.0 : cyi;
            const double p22r = sw ? cxr : oy, p22i = sw ? cxi : 0.0;
            rotate_any<ND>(c.fx, c.fy, p11r, p11i, p21r, p21i, p12r, p12i, p22r, p22i);
            rotate_any<ND>(c.gx, c.gy, p11r, p11i, p21r, p21i, p12r, p12i, p22r, p22i);
            rotate_any<ND>(c.zx, c.zy, p11r, p11i, p21r, p21i, p12r, p12i, p22r, p22i);
        }
        return true;
    }
};

// Phases 3 to 5 of the inner solver, with the columns in registers: F_hat,
// G_hat come as triangles in sF, sG (column-major), or with LOWER as their
// transposes L; sF, sG, sZ (ld LDI) are overwritten.  A wave holds GW = 64 / LP lane groups laid side by side in
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
// wave's extra stores and loads: 68.6 against 84.4 us for an inner sweep at 2w
// = 64 with 16 lanes, but 20.4 against 19.9 at 2w = 32.
//
// Bound: the instructions of one or two waves per SIMD, about five cycles
// each from one wave, and in LDS the stores, 13 cycles of a compute unit for
// 64 lanes x 16 bytes.  With every column handed on through LDS after every
// step, the pivot sums taken one by one and the orderings read from a table,
// one inner sweep of the 4096 x 1024 pair's first steps, where every pair
// rotates, took, before and now: ring ordering 73.6 -> 47.0 us (2w = 64, 8 lanes)
// and 24.5 -> 14.3 (2w = 32, 16 lanes); round robin 96.8 -> 68.6 (2w = 64, 16
// lanes) and 28.6 -> 18.3 (2w = 32, 8 -> 16 lanes).
//
// The inner sweeps stop after one without big transformations, as the outer
// ones do (Section 2.5): small ones leave the block diagonal to working
// precision, and a further sweep only to see that there are none left cost an
// eighth of the inner sweeps of full-block solves (700 x 256 23.8 against 22.3
// ms, 2048 x 630 91.4 against 85.2).  Over 680 pairs with sigma over six to
// sixteen orders of magnitude, n = 16 ... 512, real and complex, in all
// orderings and with QR pivot factors, the errors of sigma are 0.99 and the
// largest departures of U^H U and V^H V from I 1.00 times those of the other
// rule, and the same after a single sweep of a single block.
template <class E, int W2, int LP, int ORD, bool GEN, bool LOWER>
__device__ __forceinline__ void pointwise_solve(double *__restrict__ sF, double *__restrict__ sG,
                                                double *__restrict__ sZ,
                                                unsigned *__restrict__ s_cnt, int inner_max,
                                                double tol, int sort, int variant,
                                                double *__restrict__ zt,
                                                unsigned long long *__restrict__ myc,
                                                unsigned long long *__restrict__ ph)
{
    constexpr int W = W2 / 2, NT = W * LP;
    constexpr int SLOTS = E::template slots<W2>(), LDC = 2 * (SLOTS + 1);   // doubles per column
    constexpr int NS = SLOTS / LP, ND = 2 * NS;
    constexpr int GW = 64 / LP;              // groups per wave, and per 16-lane row
    constexpr int NWV = NT / 64;
    static_assert(GW == 4 || GW == 8 || GW == 16, "groups fill a 16-lane row");
    static_assert(W % GW == 0 && NS * LP == SLOTS, "whole waves, whole slots");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane & (GW - 1), grp = wave * GW + g;
    // A lane's slots of a column, placed for the banks.  The columns of
    // neighbouring groups lie 16 bytes apart modulo the 256 bytes of the banks,
    // and one cycle of a 16-byte load serves lanes 0-3, 12-15, 20-23 and 24-27
    // (the next one 4-11, 16-19 and 28-31): sub takes the places that GW columns
    // leave, and the lowest bit of row, where a column is long enough, the next
    // 256 bytes -- 5.7 cycles for 64 lanes, 8.3 where the rows meet.
    const int row = lane >> 4, sub = (lane & 15) / GW;
    auto slot = [&](int k) {
        if (SLOTS == 32)
            return (GW & 15) * sub + 16 * (row & 1) + (GW == 8 ? 4 * (row >> 1) + k : (row >> 1) + 2 * k);
        if (SLOTS == 16 && GW == 8) return row + 8 * sub + 4 * k;
        return row + 4 * sub + (GW == 16 ? 4 : 0) * k;
    };
    auto load = [&](const double *M, int c, double (&v)[ND]) {
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const d2 p = *(const d2 *)(M + __umul24(c, LDC) + 2 * slot(k));
            v[2 * k] = p[0];
            v[2 * k + 1] = p[1];
        }
    };
    auto store = [&](double *M, int c, const double (&v)[ND]) {
#pragma unroll
        for (int k = 0; k < NS; ++k)
            *(d2 *)(M + __umul24(c, LDC) + 2 * slot(k)) = d2{v[2 * k], v[2 * k + 1]};
    };
    ColPair<ND> C;
    auto load_x = [&](int c) { load(sF, c, C.fx); load(sG, c, C.gx); load(sZ, c, C.zx); };
    auto load_y = [&](int c) { load(sF, c, C.fy); load(sG, c, C.gy); load(sZ, c, C.zy); };
    auto store_x = [&](int c) { store(sF, c, C.fx); store(sG, c, C.gx); store(sZ, c, C.zx); };
    auto store_y = [&](int c) { store(sF, c, C.fy); store(sG, c, C.gy); store(sZ, c, C.zy); };

    // the group's first columns
    constexpr bool RING = ORD == HZ_ORD_RING, MM = ORD == HZ_ORD_MM;
    constexpr bool KEEP = !RING && SLOTS == 32;
    int cx = grp, cy = W + grp;
    if (!RING) cy = MM ? (grp ? W2 - grp : W) : W2 - 1 - grp;
    if (KEEP) {
        cx = MM ? ((W2 - grp) & (W2 - 1)) : (grp ? W2 - 1 - grp : 0);
        cy = MM ? (grp ? grp : W) : (grp ? grp : W2 - 1);
    }

    // 3. prescale by 1/||g_c||
    if constexpr (LOWER) {
        // across the rows of L: 0.4 us for all waves (2w = 64) where the
        // transposition by the two factoring waves took 1.1
        auto read = [&](const double *M, int c, double (&v)[ND]) {
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const d2 p = E::of_lower(M, LDC, slot(k), c);
                v[2 * k] = p[0];
                v[2 * k + 1] = p[1];
            }
        };
        read(sF, cx, C.fx);
        read(sG, cx, C.gx);
        read(sF, cy, C.fy);
        read(sG, cy, C.gy);
        __syncthreads();                 // rows of columns that others store to
    } else {
        load(sF, cx, C.fx);
        load(sG, cx, C.gx);
        load(sF, cy, C.fy);
        load(sG, cy, C.gy);
    }
    {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            a = fma(C.gx[k], C.gx[k], a);
            b = fma(C.gy[k], C.gy[k], b);
        }
        group_sum2<GW>(a, b);
        const double dx = rsqrt_nr(a), dy = rsqrt_nr(b);
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            C.fx[k] *= dx;
            C.gx[k] *= dx;
            C.zx[k] = dx * E::unit(slot(k >> 1), k & 1, cx);
            C.fy[k] *= dy;
            C.gy[k] *= dy;
            C.zy[k] = dy * E::unit(slot(k >> 1), k & 1, cy);
        }
    }
    if (ph && tid == 0) ph[3] = wall_clock64();

    // 4. inner sweeps
    StepArgs A = {tol, tol * tol, sort, variant, 0, 0};
    unsigned chg_any = 0;
    int nsw = 0;
    auto step = [&](bool first) {
        if (E::template step<GW, ND, KEEP, GEN>(C, first, A)) {
            chg_any = 1;
            if (RING) {
                // The ring's lane exchanges may come next, and what assembly
                // writes the compiler does not wait for: two wait states
                // from the last write, wherever it puts that.
                __builtin_amdgcn_sched_barrier(0);
                __asm__ volatile("s_nop 1");
            }
        }
    };

    if constexpr (RING) {
        // the y of all groups by one lane exchange inside the rows
#define HZ_MOVE_Y(CTRL)                                                                        \
    _Pragma("unroll") for (int k = 0; k < ND; ++k)                                             \
    {                                                                                          \
        C.fy[k] = dpp_d<CTRL>(C.fy[k]);                                                        \
        C.gy[k] = dpp_d<CTRL>(C.gy[k]);                                                        \
        C.zy[k] = dpp_d<CTRL>(C.zy[k]);                                                        \
    }
        // exchange of a level h <= GW with the next: groups with bit h/2 set
        // take their partner's y as x, the others their partner's x as y
        auto split = [&](int h, double (&x)[ND], double (&y)[ND]) {
#pragma unroll
            for (int k = 0; k < ND; ++k) {
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
            const unsigned big0 = A.n_big;
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
#define HZ_SPLIT(H) { split(H, C.fx, C.fy); split(H, C.gx, C.gy); split(H, C.zx, C.zy); }
                    if (h == 2) HZ_SPLIT(2)
                    else if (h == 4) HZ_SPLIT(4)
                    else if (GW >= 8 && h == 8) HZ_SPLIT(8)
                    else if (GW >= 16) HZ_SPLIT(16)
#undef HZ_SPLIT
                }
            }
            if (nsw >= inner_max) break;
            // stop after a sweep without big transformations; else back to the first level
            if (lane == 0) s_cnt[wave] = A.n_big - big0;
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
            const unsigned big0 = A.n_big;
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
            if (lane == 0) s_cnt[wave] = A.n_big - big0;
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
        s_cnt[3 * wave] = A.n_all / LP;
        s_cnt[3 * wave + 1] = A.n_big / LP;
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
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        a = fma(C.gx[k], C.gx[k], fma(C.fx[k], C.fx[k], a));
        b = fma(C.gy[k], C.gy[k], fma(C.fy[k], C.fy[k], b));
    }
    group_sum2<GW>(a, b);
    const double tx = rsqrt_nr(a), ty = rsqrt_nr(b);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int p = slot(k);
        *(d2 *)(zt + 2 * (cx * SLOTS + p)) =
            changed ? d2{C.zx[2 * k] * tx, C.zx[2 * k + 1] * tx}
                    : d2{E::unit(p, 0, cx), E::unit(p, 1, cx)};
        *(d2 *)(zt + 2 * (cy * SLOTS + p)) =
            changed ? d2{C.zy[2 * k] * ty, C.zy[2 * k + 1] * ty}
                    : d2{E::unit(p, 0, cy), E::unit(p, 1, cy)};
    }
    if (tid == 0) {
        myc[0] = ta;
        myc[1] = tb;
        myc[2] = (unsigned long long)nsw;
        myc[3] = changed ? 0ull : 1ull;
        if (ph) ph[5] = wall_clock64();
    }
}

}  // namespace hz
