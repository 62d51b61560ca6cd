// hz_device.h -- device-side primitives shared by the real and complex
// kernels of the blocked implicit Hari-Zimmermann GSVD (gfx950, wave64).
#pragma once
#include <type_traits>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hz {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

// One v_mfma_f64_16x16x4_f64: C(16x16) += A(16x4) * B(4x16).
// Lane layout (checked on gfx950): A[i][k] in lane i + 16k, B[k][j] in lane
// j + 16k, C[i][j] in lane j + 16*(i%4), element i/4 of the d4.
__device__ __forceinline__ d4 mfma16(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Sum over aligned groups of W lanes by a xor butterfly.  IEEE addition is
// commutative, so every lane of a group ends with the bitwise same value and
// the association order is fixed: the result is reproducible run to run.
template <int W>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int m = 1; m < W; m <<= 1)
        v += __shfl_xor(v, m, 64);
    return v;
}

__device__ __forceinline__ double wave_sum(double v) { return group_sum<64>(v); }

// DPP lane exchange of a double within a row of 16 lanes (two 32-bit moves).
// Every pattern used here reads a lane of the same row, so bound_ctrl (read
// 0 from an invalid source lane) never applies; it lets the move write a
// fresh register instead of one tied to, and first copied from, the source.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Sum over aligned groups of L = 2, 4, 8 or 16 lanes with DPP only (no LDS
// traffic): quad xor-1 and xor-2 permutations, then the 8-lane half mirror
// and the 16-lane mirror.  Each stage adds a lane's value to its partner's
// (commutative), so all lanes of a group hold the bitwise same sum.
template <int L>
__device__ __forceinline__ double dpp_group_sum(double v)
{
    static_assert(L == 2 || L == 4 || L == 8 || L == 16, "group of 2..16 lanes");
    v += dpp_d<0xB1>(v);                      // quad_perm [1,0,3,2]
    if (L >= 4) v += dpp_d<0x4E>(v);          // quad_perm [2,3,0,1]
    if (L >= 8) v += dpp_d<0x141>(v);         // row_half_mirror
    if (L >= 16) v += dpp_d<0x140>(v);        // row_mirror
    return v;
}

// DPP move of a double into lanes of the 4-lane banks in BANKS only (the
// other lanes keep old): lane n of a 16-lane row reads the lane of the same
// row that CTRL names.
template <int CTRL, int BANKS>
__device__ __forceinline__ double dpp_into(double old, double v)
{
    const long long o = __builtin_bit_cast(long long, old), b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)b, CTRL, 0xF, BANKS, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, 0xF, BANKS, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// v_permlane32_swap / v_permlane16_swap on doubles: the upper half of a
// changes places with the lower half of b (the odd 16-lane rows of a with the
// even rows of b).
__device__ __forceinline__ void swap32(double &a, double &b)
{
    const long long x = __builtin_bit_cast(long long, a), y = __builtin_bit_cast(long long, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __builtin_bit_cast(double, ((long long)hi[0] << 32) | lo[0]);
    b = __builtin_bit_cast(double, ((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ void swap16(double &a, double &b)
{
    const long long x = __builtin_bit_cast(long long, a), y = __builtin_bit_cast(long long, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __builtin_bit_cast(double, ((long long)hi[0] << 32) | lo[0]);
    b = __builtin_bit_cast(double, ((long long)hi[1] << 32) | lo[1]);
}

// Sums of four values over the lanes that share lane mod GW (GW = 4, 8 or 16
// groups laid side by side in every 16-lane row): the four are reduced
// together, each swap halving the registers (two rows' partial sums change
// places and one add does two of them), so that the reduction and the
// broadcast back take 24 instructions (27 for GW = 4) where a butterfly for
// each takes 36 (48).  Every lane of a group gets the same bits.
template <int GW>
__device__ __forceinline__ void group_sum4(double &s1, double &s2, double &s3, double &s4)
{
    swap32(s1, s2);
    swap32(s3, s4);
    double u = s1 + s2, v = s3 + s4;         // lower half: s1, s3; upper: s2, s4
    swap16(u, v);
    double w = u + v;                        // rows: s1, s3, s2, s4
    if (GW <= 8) w += dpp_d<0x128>(w);       // row_ror:8
    if (GW <= 4) w += dpp_d<0x124>(w);       // row_ror:4
    double x = w;
    swap16(w, x);                            // w: s1 s1 s2 s2, x: s3 s3 s4 s4
    s1 = s2 = w;
    swap32(s1, s2);
    s3 = s4 = x;
    swap32(s3, s4);
}

// The same for two values (15 instructions).
template <int GW>
__device__ __forceinline__ void group_sum2(double &s1, double &s2)
{
    swap32(s1, s2);
    double u = s1 + s2;                      // lower half: s1; upper: s2
    double v = u;
    swap16(u, v);
    u += v;
    if (GW <= 8) u += dpp_d<0x128>(u);       // row_ror:8
    if (GW <= 4) u += dpp_d<0x124>(u);       // row_ror:4
    s1 = s2 = u;
    swap32(s1, s2);
}

// Broadcast lane l's double to the wave (two v_readlane_b32; l uniform).
__device__ __forceinline__ double readlane_d(double v, int l)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// p[i] += r(lane T + i of the lane's 16-lane row) * m, i < N: the broadcast is
// part of the multiply-add (row_newbcast, the one move that FP64 instructions
// take), one instruction where readlane needs two and a product.  The first
// one waits for r to be written (two cycles).
template <int T, int N>
__device__ __forceinline__ void fmac_row(double *p, double r, double m)
{
#define HZ_FR(K, R, M, I) "\n\tv_fmac_f64_dpp %" #K ", %" #R ", %" #M " row_newbcast:%" #I " row_mask:0xf bank_mask:0xf"
    if constexpr (N >= 8) {
        asm("s_nop 1" HZ_FR(0, 8, 9, 10) HZ_FR(1, 8, 9, 11) HZ_FR(2, 8, 9, 12) HZ_FR(3, 8, 9, 13)
            HZ_FR(4, 8, 9, 14) HZ_FR(5, 8, 9, 15) HZ_FR(6, 8, 9, 16) HZ_FR(7, 8, 9, 17)
            : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(p[4]), "+v"(p[5]), "+v"(p[6]),
              "+v"(p[7])
            : "v"(r), "v"(m), "n"(T), "n"(T + 1), "n"(T + 2), "n"(T + 3), "n"(T + 4), "n"(T + 5),
              "n"(T + 6), "n"(T + 7));
        fmac_row<T + 8, N - 8>(p + 8, r, m);
    } else if constexpr (N >= 4) {
        asm("s_nop 1" HZ_FR(0, 4, 5, 6) HZ_FR(1, 4, 5, 7) HZ_FR(2, 4, 5, 8) HZ_FR(3, 4, 5, 9)
            : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3])
            : "v"(r), "v"(m), "n"(T), "n"(T + 1), "n"(T + 2), "n"(T + 3));
        fmac_row<T + 4, N - 4>(p + 4, r, m);
    } else if constexpr (N >= 2) {
        asm("s_nop 1" HZ_FR(0, 2, 3, 4) HZ_FR(1, 2, 3, 5)
            : "+v"(p[0]), "+v"(p[1])
            : "v"(r), "v"(m), "n"(T), "n"(T + 1));
        fmac_row<T + 2, N - 2>(p + 2, r, m);
    } else if constexpr (N == 1) {
        asm("s_nop 1" HZ_FR(0, 1, 2, 3) : "+v"(p[0]) : "v"(r), "v"(m), "n"(T));
    }
#undef HZ_FR
}

// Lane T's value of each 16-lane row to the row.
template <int T>
__device__ __forceinline__ double bcast_row(double v)
{
    double r;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
        : "=v"(r) : "v"(v), "n"(T));
    return r;
}

// f(integral_constant 0) ... f(integral_constant N - 1)
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<N, I + 1>(f);
    }
}

// Reciprocal square root from the hardware estimate y0 = v_rsq_f64(x)
// (relative error e0 about 2^-22) refined by one third-order step
// y = y0 (1 + e/2 + 3e^2/8), e = 1 - x y0^2, which leaves O(e0^3) -- below
// double rounding -- with a dependency depth of four operations.  About one
// ulp for positive normal finite x; exactly 1 for x = 1.  Deterministic.
__device__ __forceinline__ double rsqrt_nr(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    const double p = fma(0.375, e, 0.5);
    return fma(y * e, p, y);
}

// The same from half an ulp lower before its last rounding (still exactly 1 for
// x = 1): the factors that the 2x2 transformations scale columns with must not
// come out too large on average.  The pivot entries take b_xx = 1, a column's
// norm is not formed again within an inner solve, and a transformation with t^2
// = 1 - x^2 multiplies what has crept into it by 1 / t^2: a norm that grows
// leads to |x| >= 1, where there is no transformation, one that shrinks does
// not.  With rsqrt_nr the mean growth of |g''|^2 by a transformation of x <=
// 1e-5 was 1.3e-16 to 3e-16, and over pencils of values in [1e-12, 1e12] (QR
// pivot factors, n = 100, w = 32) 254 of 480 solves broke down; with this one it
// is -1.9e-16 to 2e-17, and none does.
__device__ __forceinline__ double rsqrt_lo(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 0x1.fffffffffffffp-1);
    const double p = fma(0.375, e, 0.5);
    return fma(y * e, p, y);
}

__device__ __forceinline__ double sqrt_nr(double x) { return x * rsqrt_nr(x); }

// x is positive, finite and no denormal (one instruction).
__device__ __forceinline__ bool positive_normal(double x)
{
    return !__builtin_amdgcn_class(x, 0x3FF ^ (1 << 8));
}

// Scheduling fence between LDS traffic of lanes of one wave (LDS executes a
// wave's operations in order; this only stops the compiler from moving
// accesses across it).
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The real 2x2 implicit Hari-Zimmermann transformation (paper, Section
// 2.1.2) of the pivot pair A' = [[aii, aij], [aij, ajj]], B' = [[1, x],
// [x, 1]] in the form in which the inner solver applies it.  Let b be the
// column with the larger diagonal entry of A' (i when equal) and s the other
// one; then
//     b'' = rb b - qb s,   s'' = rr b + rs s
// diagonalize both forms with B' becoming I, and a''_bb >= a''_ss always: the
// printed angle 2 theta lies in [-pi/2, pi/2], which keeps the order of the
// diagonal, so the sorting heuristic needs no transformed diagonal entries.
// The printed entries are cos phi / t and cos psi / t = rb, rs and the sines
// rr, -qb in the places that b and s take (t = sqrt(1 - x^2)).
// With h = a_jj - a_ii and D = 2 a_ij - (a_ii + a_jj) x, tan 2theta =
// sign(h) D / (t |h|), and the coefficient of b in s'' is the root
//     r = 2 (min(a_ii, a_jj) x - a_ij) / (|h| + sqrt(t^2 h^2 + D^2)),
// |r| <= 1, of the quadratic that makes s'' and b'' A'-orthogonal (in the
// Falk-Langemeyer form of the method; eliminating theta, xi and eta from the
// printed formulas gives the same number).  B'-orthogonality makes the other
// one q = (r + x)/(1 + r x), and with w = r + x, o = 1 + r x the squared
// B'-norms are n_s = w^2 + t^2 and n_b = t^2 n_s / o^2, so that
//     rs = n_s^(-1/2), rr = r rs, rb = o rs / t, qb = w rs / t:
// one division and three reciprocal square roots, two of them off the chain,
// where the printed formulas took two divisions and four.  Every sum of
// squares is of positive terms and the small column's coefficient r has full
// relative accuracy: over random pencils of graded diagonals the largest
// relative A'-offdiagonal left behind is 1.5e-14, against 1.8e-11 for the
// printed form in doubles; rb, rs are exactly 1 when r and x vanish beside 1
// (criterion C1).  A' proportional to B' (h = D = 0) takes r = -sign(x), the
// printed congruence with the sign of x carried onto the off-diagonal
// entries so that it is one for x < 0 too; with keep (the pair is left alone;
// the caller passes x = 0) it takes r = 0, the identity, whatever A' is.  Where a square of h or D overflows, or both underflow,
// the root is a NaN and stays one, which the solve reports: a pivot like that
// must not pass for one proportional to B'.  An inner step is bound by the
// instructions of one wave (about five cycles each), of which this takes some
// 43; the printed form with the sort keys took 110, the largest part of a step,
// and whole solves 6 (4096 x 1024) to 13 % (2048 x 630) more.
__device__ __forceinline__ void hz_real_2x2_fast(double aii, double ajj, double aij, double x,
                                                 bool keep, double &rb, double &qb, double &rs,
                                                 double &rr, double &t)
{
    const double t2 = fma(-x, x, 1.0);
    const double h = ajj - aii;
    const double D = fma(-(aii + ajj), x, aij + aij);
    const double hyp2 = fma(t2 * h, h, D * D);
    const double num = fma((aii < ajj) ? aii : ajj, x, -aij);
    const double den = fabs(h) + sqrt_nr(hyp2);
    // num / den to about one ulp; 2 num and not den / 2, which could underflow
    const double y0 = __builtin_amdgcn_rcp(den);
    const double e = fma(-den, y0, 1.0);
    const double r0 = (num + num) * fma(y0, fma(e, e, e), y0);
    const bool prop = fabs(h) + fabs(D) == 0.0;
    const double r = (keep || prop) ? (keep ? 0.0 : -copysign(1.0, x)) : r0;
    const double w = r + x, o = fma(r, x, 1.0);
    const double rt = rsqrt_nr(t2);
    rs = rsqrt_lo(fma(w, w, t2));
    const double k = rt * rs;
    rr = r * rs;
    rb = o * k;
    qb = w * k;
    t = t2 * rt;
}

// The complex 2x2 transformation of Section 2.1.1 in the form of the real one:
// b the column with the larger diagonal entry, s the other, a = f_b^H f_s,
// beta = g_b^H g_s, x = |beta| < 1, t = sqrt(1 - x^2), h = a_bb - a_ss >= 0;
//     b'' = rb b + cb s,   s'' = rs s + cs b,   rb, rs > 0 real.
// With D = 2a - (a_bb + a_ss) beta and m = Im(a conj(beta)), the coefficient
// of b in s'' before scaling is the root
//     r = 2 (a_ss beta - a) / (h + sqrt(t^2 h^2 + |D|^2 - 4 m^2) + 2 i m),
// |r| <= 1, of the quadratic that makes the columns A'-orthogonal, and
// B'-orthogonality gives the other one: with w = r + beta, o = 1 + conj(r) beta,
// n_s = |w|^2 + t^2,
//     rs = n_s^(-1/2), cs = r rs, rb = |o|^2 k, cb = -conj(w o) k, k = (t^2 n_s |o|^2)^(-1/2).
// Eliminating the printed angles gives the same entries (their cosines divided
// by t are rb, rs); with u + i v = e^(-i zeta) a the printed radicand t^2 (h^2 +
// 4 v^2) + (2u - (a_bb + a_ss) x)^2 is the one above.  A' proportional to B'
// takes r = -e^(i zeta) (-1 for beta = 0), the printed congruence; with keep (beta =
// 0 passed) r = 0, the identity, and NaNs stay, both as in the real form.
// A radicand that rounding takes below zero counts as A' proportional to B'.
__device__ __forceinline__ void hz_cplx_2x2_fast(double abb, double ass, double ar, double ai,
                                                 double br, double bi, bool keep, double &rb,
                                                 double &cbr, double &cbi, double &rs, double &csr,
                                                 double &csi, double &t)
{
    const double x2 = fma(br, br, bi * bi), t2 = 1.0 - x2;
    const double h = abb - ass, S = abb + ass;
    const double Dr = fma(-S, br, ar + ar), Di = fma(-S, bi, ai + ai);
    const double m = fma(ai, br, -ar * bi), m2 = m + m;
    const double hyp2 = fma(-m2, m2, fma(t2 * h, h, fma(Dr, Dr, Di * Di)));
    const double nr = fma(ass, br, -ar), ni = fma(ass, bi, -ai);
    // half the denominator, p + i m: its square overflows no earlier than hyp2
    const double p = 0.5 * (h + sqrt_nr(hyp2));
    const double q = fma(p, p, m * m);
    const double y0 = __builtin_amdgcn_rcp(q);
    const double e = fma(-q, y0, 1.0);
    const double y = fma(y0, fma(e, e, e), y0);
    double rr = y * fma(nr, p, ni * m), ri = y * fma(ni, p, -nr * m);
    if (!positive_normal(hyp2)) {
        const double ix = (x2 > 0.0) ? rsqrt_nr(x2) : 0.0;
        const bool prop = (hyp2 < 0.0) | (fabs(h) + fabs(Dr) + fabs(Di) == 0.0);
        const bool zero = fabs(nr) + fabs(ni) == 0.0;       // also where 1 / q overflows
        rr = prop ? (x2 > 0.0 ? -br * ix : -1.0) : (zero ? 0.0 : rr);
        ri = prop ? -bi * ix : (zero ? 0.0 : ri);
    }
    rr = keep ? 0.0 : rr;
    ri = keep ? 0.0 : ri;
    const double wr = rr + br, wi = ri + bi;
    const double orr = fma(rr, br, fma(ri, bi, 1.0)), oi = fma(rr, bi, -ri * br);
    const double ns = fma(wr, wr, fma(wi, wi, t2));
    rs = rsqrt_lo(ns);
    const double o2 = fma(orr, orr, oi * oi);
    const double k = rsqrt_lo(t2 * ns * o2);
    csr = rr * rs;
    csi = ri * rs;
    rb = o2 * k;
    // -conj(w) conj(o) k
    cbr = -k * fma(wr, orr, -wi * oi);
    cbi = k * fma(wr, oi, wi * orr);
    t = sqrt_nr(t2);
}

// Appendix A (enhanced dot products): a*b rounded toward -infinity, from the
// round-to-nearest product p and its exact error e = a*b - p (one FMA): the
// exact product rounds down to p when e >= 0, else to the double just below
// p.  The rounding mode register is left alone; contraction is off here so
// that the product and the sums stay separately rounded operations.
__device__ __forceinline__ double mul_rd(double a, double b)
{
#pragma clang fp contract(off)
    const double p = a * b;
    const double e = fma(a, b, -p);
    // by selects: as branches, 64 of them to a step, they were most of it.  Away
    // from zero for p <= 0 (below +-0: -denorm_min), towards it for p > 0.
    const long long bits = __double_as_longlong((p == 0.0) ? -0.0 : p);
    const long long below = bits + ((p > 0.0) ? -1 : 1);
    return (e < 0.0) ? __longlong_as_double(below) : p;
}

// |re + i im|^2 by the simpler complex procedure of Appendix A: the
// rounded-down squares c_r, c_i and the sum e of their errors, combined as
// (e + min(c_r, c_i)) + max(c_r, c_i).
__device__ __forceinline__ double enh_abs2(double re, double im)
{
#pragma clang fp contract(off)
    const double cr = mul_rd(re, re), ci = mul_rd(im, im);
    const double e = fma(re, re, -cr) + fma(im, im, -ci);
    return (cr <= ci) ? (e + cr) + ci : (e + ci) + cr;
}

// Accumulate a*b into the pair (sum of rounded-down products, sum of their
// non-negative rounding errors).
__device__ __forceinline__ void edot_acc(double a, double b, double &sc, double &sd)
{
#pragma clang fp contract(off)
    const double c = mul_rd(a, b);
    sc = sc + c;
    sd = sd + fma(a, b, -c);
}

}  // namespace hz
