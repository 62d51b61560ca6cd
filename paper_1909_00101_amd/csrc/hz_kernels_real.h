// hz_kernels_real.h -- FP64 device bodies shared by the single-pair kernels
// (hz_real.hip) and the batched kernels (hz_batched.hip): the pivot Gram
// block of a block-column pair, the inner solve of one pivot block pair and
// the in-place block update of a row range.
#pragma once
#include "hz_device.h"
#include "hz_internal.h"
#include "hz_pointwise.h"

namespace hz {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

// v_mfma_f32_16x16x4_f32: A[i][k] lane i + 16k, B[k][j] lane j + 16k,
// C[i][j] lane j + 16*(i/4), element i%4 (checked on gfx950).
__device__ __forceinline__ f4 mfma16f(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

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
template <int W2> constexpr int inner_lds() { return 3 * W2 * (W2 + 2) + 128 + 16; }

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
    unsigned long long *__restrict__ myc, int *__restrict__ status, int failcode,
    unsigned long long *__restrict__ ph, double *__restrict__ lds)
{
    constexpr int NT = (W2 / 2) * LP;
    constexpr int LDI = W2 + 2;
    static_assert(NT >= 64, "bad inner geometry");
    // With the ring the factors stay lower, L = F_hat^T.
    constexpr bool LOWER = W2 >= 32 && NT >= 128 && ORD == HZ_ORD_RING;
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
    // themselves (QR of the block-column pairs), taken in as L with LOWER.
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
            if (LOWER && nsplit == 0) {
                sF[row * LDI + col] = va[it][0];
                sF[(row + 1) * LDI + col] = va[it][1];
                sG[row * LDI + col] = vb[it][0];
                sG[(row + 1) * LDI + col] = vb[it][1];
            } else {
                *(d2 *)(sF + col * LDI + row) = va[it];
                *(d2 *)(sG + col * LDI + row) = vb[it];
            }
        }
        if (tid == 0) s_fail = 0;
    } else {
        // SB partials of every element in flight at a time
        constexpr int NIT = (W2 * W2) / (2 * NT), SB = NIT > 16 ? 1 : 16 / NIT;
        d2 va[NIT], vb[NIT];
        for (int s0 = 0; s0 < nsplit; s0 += SB) {
            d2 ta[SB][NIT], tb[SB][NIT];
#pragma unroll
            for (int u = 0; u < SB; ++u)
                if (s0 + u < nsplit) {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        const int e = 2 * tid + 2 * NT * it;
                        // upper tiles of a Gram are never read
                        if ((e / W2) / 16 > (e % W2) / 16) continue;
                        ta[u][it] = *(const d2 *)(pa + (s0 + u) * sstride + e);
                        tb[u][it] = *(const d2 *)(pb + (s0 + u) * sstride + e);
                    }
                }
#pragma unroll
            for (int u = 0; u < SB; ++u)
                if (s0 + u < nsplit) {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        va[it] = (s0 + u) ? va[it] + ta[u][it] : ta[u][it];
                        vb[it] = (s0 + u) ? vb[it] + tb[u][it] : tb[u][it];
                    }
                }
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = 2 * tid + 2 * NT * it, col = e / W2, row = e % W2;
            if (col / 16 > row / 16) continue;
            *(d2 *)(sF + col * LDI + row) = va[it];
            *(d2 *)(sG + col * LDI + row) = vb[it];
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
    } else if constexpr (LOWER) {
        // Blocked right-looking Cholesky in panels of 16 columns, one wave per
        // matrix for a panel (lane = row, in registers).  A column's entries reach
        // the others by products with a row broadcast; as that stays within 16
        // lanes, the diagonal block's rows are kept in every 16-lane row (q)
        // beside the panel's (pv), and pivots and reciprocal roots are formed
        // there: no scalar on the chain.  Entries above the diagonal are left as
        // they come; nothing reads them.  The trailing lower tiles take A22 -= L21
        // L21^T as FP64 MFMA products (tile (ti, tj): A operand L rows of ti, B
        // operand L rows of tj, four k-steps of 4 panel columns), at 2w = 64 by all
        // waves, half of them per matrix.  Bound: the instructions of the one wave,
        // 170 cycles a column, and the latency of LDS around the tiles.  Against
        // the form below (readlane, pivots kept by selects, two waves, and its
        // transposition, which the prescale makes up for by reading across): 2w =
        // 64 10.0 -> 8.3 us, 2w = 32 4.3 -> 3.5, 4096x1024 60.0 -> 58.65 ms.  The
        // other orderings keep that one: behind this one the compiler made their
        // sweeps 1 % slower (2w = 64, many sweeps: 291 -> 295 us).
        constexpr int NBK = W2 / 16;
        constexpr int WPM = W2 == 64 ? NT / 128 : 1;     // waves per matrix for the tiles
        const int uwave = __builtin_amdgcn_readfirstlane(wave);
        double *const M = (uwave & 1) ? sG : sF;
        // lane j: column j's diagonal before the factorization
        const double d0 = (lane < W2) ? M[lane * LDI + lane] : 0.0;
        static_for<NBK>([&](auto kb_c) {
            constexpr int kb = decltype(kb_c)::value, c0 = 16 * kb;
            if (uwave < 2) {
                const int row = c0 + lane;
                const bool live = row < W2;
                double pv[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) pv[t] = live ? M[(c0 + t) * LDI + row] : 0.0;
                // the diagonal block's rows, in every 16-lane row (the last
                // panel has no others)
                constexpr bool REP = kb + 1 < NBK;
                double q[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) q[t] = REP ? M[(c0 + t) * LDI + c0 + (lane & 15)] : pv[t];
                double inv = rsqrt_nr(bcast_row<0>(q[0]));
                static_for<16>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    const double lq = q[j] * inv, mq = q[j] * -inv, lp = pv[j] * inv, mp = pv[j] * -inv;
                    pv[j] = REP ? lp : lq;
                    if constexpr (j < 15) {
                        // the chain: the next pivot and its reciprocal root
                        fmac_row<j + 1, 1>(q + j + 1, lq, mq);
                        const double piv = bcast_row<j + 1>(q[j + 1]);
                        const double y = __builtin_amdgcn_rsq(piv);
                        __builtin_amdgcn_sched_barrier(0);
                        fmac_row<j + 2, 14 - j>(q + j + 2, lq, mq);
                        if (REP) fmac_row<j + 1, 15 - j>(pv + j + 1, lq, mp);
                        __builtin_amdgcn_sched_barrier(0);
                        const double e = fma(-piv * y, y, 1.0);
                        inv = fma(y * e, fma(0.375, e, 0.5), y);
                    }
                });
                if (live) {
#pragma unroll
                    for (int t = 0; t < 16; ++t) M[(c0 + t) * LDI + row] = pv[t];
                }
            }
            if constexpr (kb + 1 < NBK) {
                if (WPM > 1) __syncthreads();
                else wave_fence();
                const int i16 = lane & 15, k4 = lane >> 4;
                if (WPM > 1 || uwave < 2) {
                    // a wave's tiles together: every operand loaded first, the
                    // products of the tiles in turn (element r of lane l: row
                    // 16 ti + 4 r + l/16, column 16 tj + l%16)
                    constexpr int NTR = NBK - 1 - kb, TILES = NTR * (NTR + 1) / 2;
                    constexpr int TW = (TILES + WPM - 1) / WPM;
                    double *ct[TW];
                    d4 acc[TW];
                    double la[TW][4], lb[TW][4];
#pragma unroll
                    for (int u = 0; u < TW; ++u) {
                        // tile n of the lower triangle, row by row (beyond the last: the last)
                        int n = u * WPM + (WPM > 1 ? uwave >> 1 : 0), ti = 0;
                        n = n < TILES ? n : TILES - 1;
#pragma unroll
                        for (int k = 1; k < NTR; ++k) ti += n >= k * (k + 1) / 2;
                        const int tj = n - ti * (ti + 1) / 2;
                        ct[u] = M + (16 * (kb + 1 + tj) + i16) * LDI + 16 * (kb + 1 + ti) + k4;
                        acc[u] = d4{ct[u][0], ct[u][4], ct[u][8], ct[u][12]};
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const double *const lc = M + (c0 + 4 * s + k4) * LDI + 16 * (kb + 1) + i16;
                            la[u][s] = -lc[16 * ti];
                            lb[u][s] = lc[16 * tj];
                        }
                    }
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int u = 0; u < TW; ++u) acc[u] = mfma16(la[u][s], lb[u][s], acc[u]);
#pragma unroll
                    for (int u = 0; u < TW; ++u)
                        if (u * WPM + (WPM > 1 ? uwave >> 1 : 0) < TILES) {
                            ct[u][0] = acc[u][0];
                            ct[u][4] = acc[u][1];
                            ct[u][8] = acc[u][2];
                            ct[u][12] = acc[u][3];
                        }
                }
                if (WPM > 1) __syncthreads();
                else wave_fence();
            }
        });
        if (uwave < 2) {
            // the pivots, from the roots on the diagonal of L (the pivot of a
            // column that is not positive leaves a NaN there)
            wave_fence();
            const double r = (lane < W2) ? M[lane * LDI + lane] : 1.0;
            if (!(r * r > PIV_REL<W2>() * d0 && r < INFINITY)) s_fail = 1;
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

    pointwise_solve<RealCols, W2, LP, ORD, GEN, LOWER>(sF, sG, sZ, s_cnt, inner_max, tol, sort,
                                                       variant, zt, myc, ph);
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

// The same on FP32 rows (tiles of 32 rows), with Z_tilde rounded to FP32 (sz:
// W2 * (W2 + 1) floats).
template <int W2, int NW, class Locate>
__device__ __forceinline__ void update32_row_seq(Locate locate, int p, int q, int64_t rb,
                                                 int64_t re, const double *__restrict__ zt,
                                                 float *__restrict__ sz)
{
    constexpr int W = W2 / 2, NB = W2 / 16, KS = W2 / 4, LDZ = W2 + 1, NTH = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    {
        // every load of a thread issued before the first store
        constexpr int NZ = (W2 * W2) / NTH;
        static_assert(NZ * NTH == W2 * W2, "Z_tilde staging geometry");
        double zv[NZ];
#pragma unroll
        for (int it = 0; it < NZ; ++it) zv[it] = zt[tid + NTH * it];
#pragma unroll
        for (int it = 0; it < NZ; ++it) {
            const int e = tid + NTH * it;
            sz[(e / W2) * LDZ + (e % W2)] = (float)zv[it];
        }
    }
    __syncthreads();
    const int k4 = lane >> 4, i16 = lane & 15;
    for (int64_t v0 = rb + 32 * wave; v0 < re; v0 += 32 * NW) {
        __asm__ volatile("" ::: "memory");
        float *Y;
        int64_t m, r0;
        locate(v0, Y, m, r0);
        float *bp = Y + ((int64_t)p * W + k4) * m + 2 * i16;
        float *bq = Y + ((int64_t)q * W + k4) * m + 2 * i16;
        f2 xb[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s)
            xb[s] = (4 * s < W) ? *(const f2 *)(bp + (int64_t)(4 * s) * m + r0)
                                : *(const f2 *)(bq + (int64_t)(4 * s - W) * m + r0);
        f4 ae[NB], ao[NB];
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) {
            ae[jb] = f4{0.f, 0.f, 0.f, 0.f};
            ao[jb] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                const float za = sz[(16 * jb + i16) * LDZ + 4 * s + k4];
                ae[jb] = mfma16f(za, xb[s][0], ae[jb]);
                ao[jb] = mfma16f(za, xb[s][1], ao[jb]);
            }
        // output column 16jb + 4*k4 + r, rows r0 + 2*i16 (+1): stored through
        // the base pointers (which already carry the k4 column offset)
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c0 = 16 * jb + 3 * k4 + r;   // + k4 via the base pointer
                const int cabs = 16 * jb + 4 * k4 + r;
                float *dst = (cabs < W) ? bp + (int64_t)c0 * m + r0 : bq + (int64_t)(c0 - W) * m + r0;
                *(f2 *)dst = f2{ae[jb][r], ao[jb][r]};
            }
    }
}

// Off-diagonal measure of the FP32 phase (reading R20) of one Gram block A:
// max over its off-diagonal entries of |A_ij| / sqrt(A_ii A_jj), by a
// workgroup of NT threads; lds: W2 + NT doubles.
template <int W2, int NT>
__device__ __forceinline__ void offdiag_block(const double *__restrict__ A,
                                              double *__restrict__ out, double *__restrict__ lds)
{
    double *const dg = lds, *const red = lds + W2;
    const int tid = threadIdx.x;
    for (int i = tid; i < W2; i += NT) dg[i] = A[i * W2 + i];
    __syncthreads();
    double mx = 0.0;
    // every load of a thread issued before the first use (the upper
    // entries are loaded and left unused)
    constexpr int NIT = (W2 * W2) / NT;
    static_assert(NIT * NT == W2 * W2, "off-diagonal geometry");
    double av[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) av[it] = A[tid + NT * it];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = tid + NT * it, col = e / W2, row = e % W2;
        if (row > col) {
            const double v = fabs(av[it]) / sqrt(dg[row] * dg[col]);
            mx = (v > mx) ? v : mx;
        }
    }
    red[tid] = mx;
    __syncthreads();
    for (int h = NT / 2; h > 0; h >>= 1) {
        if (tid < h) red[tid] = (red[tid + h] > red[tid]) ? red[tid + h] : red[tid];
        __syncthreads();
    }
    if (tid == 0) *out = red[0];
}

// Side workgroup b of an inner launch (see InnerSide).
template <int W2, int NT>
__device__ __forceinline__ void inner_side(const InnerSide &S, int npairs, int b,
                                           double *__restrict__ lds)
{
    if (b >= npairs * S.nblk) {
        const int pm = b - npairs * S.nblk;
        offdiag_block<W2, NT>(S.blocks + pm * S.bstride, S.offd + pm, lds);
        return;
    }
    const int pr = b / S.nblk;
    if (S.cnt[(size_t)pr * 4 + 3]) return;   // Z_tilde = I
    const int p = S.pairs[2 * pr], q = S.pairs[2 * pr + 1];
    const int64_t rb = (int64_t)(b - pr * S.nblk) * S.rows;
    const int64_t re = rb + S.rows < S.nzw ? rb + S.rows : S.nzw;
    const double *zt = S.Zt + (size_t)pr * (W2 * W2);
    if (S.f32) {
        float *const Z = (float *)S.Zw;
        const int64_t m = S.nzw;
        update32_row_seq<W2, NT / 64>(
            [=](int64_t v, float *&y, int64_t &ld, int64_t &r) {
                y = Z;
                ld = m;
                r = v;
            },
            p, q, rb, re, zt, (float *)lds);
    } else {
        update_rows<W2, NT / 64>((double *)S.Zw, S.nzw, p, q, rb, re, zt, lds);
    }
}

}  // namespace hz
