// bsde_f64_math.h -- FP64 elementary functions of the FP64 path kernels,
// specialised to the arguments the Box-Muller transform hands them.
//
// The angle of a Box-Muller pair is 2 pi u with u = (w + 1/2) 2^-32 for a
// 32-bit Philox word w, so its reduction to a quarter turn is exact integer
// arithmetic on w: with q the nearest quarter turn and the remainder
// rho = w - q 2^30 in [-2^29, 2^29), the reduced angle is
// x = 2 pi (rho + 1/2) 2^-32 in [-pi/4, pi/4] (one rounding), and
// sin(2 pi u), cos(2 pi u) are sin x, cos x permuted and negated by q.  On
// [-pi/4, pi/4] the Maclaurin series of sine to degree 17 and of cosine to
// degree 16 leave remainders below 1e-19 and 3e-18, under a quarter of an
// ulp of the results (|cos x| >= 0.707, |sin x| >= 0.637 |x|), so the
// results are within a few ulps.  The general-argument library sincos
// spends most of its instructions on a double-word reduction by pi/2 that
// this angle does not need.
//
// The radius of the pair needs ln u for the same u: with v = w + 1/2 =
// 2^e m, m in [1/sqrt 2, sqrt 2) split off the bits of v, ln u =
// (e - 32) ln 2 + ln m and ln m = 2 atanh(s), s = (m - 1) / (m + 1),
// |s| <= 0.1716, whose odd series 2 s (1 + s^2/3 + s^4/5 + ...) is taken
// as 2 s + s z q(z), z = s^2, with q a degree-6 polynomial fitted to the
// series' tail (relative error 4.7e-16 of a term below 1% of 2 s).  The
// quotient s takes one hardware reciprocal and two residual corrections.
//
// The local volatility needs e^x for x = -y^2 <= 0: x clamped at -708
// (e^-708 is already below the volatility's rounding), x = n ln 2 + r with
// |r| <= ln 2 / 2 (ln 2 in two parts, so r is exact to the last bits), e^r
// by its Maclaurin series to degree 13 (remainder below 6e-18 of e^r), and
// the power 2^n applied to the exponent.
//
// The radius takes the square root from the hardware reciprocal square
// root and Newton steps (sqrt_nonneg).
//
// The path kernels take the logarithm, sine, cosine and powers of two from
// tables (Tables below), each of these series cut short by the table's share
// of the argument; the series by themselves are the tables' yardstick in the
// tests.
//
// Plain double and 32-bit integer arithmetic (and the hardware reciprocal
// and reciprocal-square-root seeds on the device), so the same code also
// compiles for the host: the test suite checks it there against
// high-precision references.
#pragma once

#include <math.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define BSDE_F64_HD __host__ __device__
#else
#define BSDE_F64_HD
#endif

namespace bsde {
namespace f64 {

// Maclaurin coefficients (-1)^k / (2k+1)! of sine and (-1)^k / (2k)! of
// cosine, k = 1..8
constexpr double kS[8] = {-1.0 / 6.0,
                          1.0 / 120.0,
                          -1.0 / 5040.0,
                          1.0 / 362880.0,
                          -1.0 / 39916800.0,
                          1.0 / 6227020800.0,
                          -1.0 / 1307674368000.0,
                          1.0 / 355687428096000.0};
constexpr double kC[8] = {-1.0 / 2.0,
                          1.0 / 24.0,
                          -1.0 / 720.0,
                          1.0 / 40320.0,
                          -1.0 / 3628800.0,
                          1.0 / 479001600.0,
                          -1.0 / 87178291200.0,
                          1.0 / 20922789888000.0};
// 2 pi 2^-32 (the ulp of u in radians)
constexpr double kTwoPiUlp = 6.283185307179586476925286766559 / 4294967296.0;

// sin x and cos x for |x| <= pi/4 (Maclaurin series to degrees 17 and 16)
BSDE_F64_HD inline void sincos_reduced(double x, double &s, double &c)
{
    const double x2 = x * x;
    double ps = kS[7], pc = kC[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) {
        ps = __builtin_fma(ps, x2, kS[k]);
        pc = __builtin_fma(pc, x2, kC[k]);
    }
    s = __builtin_fma(x * x2, ps, x);
    c = __builtin_fma(x2, pc, 1.0);
}

// sin and cos of q pi/2 + x from sx = sin x, cx = cos x:
// sin(q pi/2 + x) = sin x, cos x, -sin x, -cos x;
// cos(q pi/2 + x) = cos x, -sin x, -cos x, sin x
BSDE_F64_HD inline void rotate_quarters(uint32_t q, double sx, double cx, double &s, double &c)
{
    const bool odd = (q & 1u) != 0;
    const double a = odd ? cx : sx;
    const double b = odd ? sx : cx;
    s = (q & 2u) ? -a : a;
    c = ((q + 1u) & 2u) ? -b : b;
}

// sin and cos of the angle 2 pi (w + 1/2) 2^-32 (w a 32-bit word)
BSDE_F64_HD inline void sincos_turn(uint32_t w, double &s, double &c)
{
    // nearest quarter turn (mod 4) and the signed remainder; the 32-bit
    // wrap-around of the sum gives q = 0 for the last eighth of the turn
    const uint32_t q = (w + 0x20000000u) >> 30;
    const int32_t rho = (int32_t)(w - (q << 30));
    const double x = __builtin_fma((double)rho, kTwoPiUlp, 0.5 * kTwoPiUlp);
    double sx, cx;
    sincos_reduced(x, sx, cx);
    rotate_quarters(q, sx, cx, s, c);
}

// ln 2 in two parts: kLn2Hi has 42 significant bits, so e kLn2Hi is exact
// for |e| < 2^11
constexpr double kLn2Hi = 0.693147180559890330187045037746429443359375;
constexpr double kLn2Lo = 5.4979230187083711552420206887e-14;

BSDE_F64_HD inline uint64_t to_bits(double x) { return __builtin_bit_cast(uint64_t, x); }
BSDE_F64_HD inline double from_bits(uint64_t b) { return __builtin_bit_cast(double, b); }

// Hardware seeds: v_rcp_f64 and v_rsq_f64 on the device.  The host build
// (tests only) takes seeds of single-precision accuracy, no better than the
// hardware's, so that the refinement steps below are tested as the device
// needs them.
BSDE_F64_HD inline double reciprocal_seed(double d)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcp(d);
#else
    return (1.0 / d) * (1.0 - 0x1p-24); // single-precision accuracy
#endif
}
BSDE_F64_HD inline double rsqrt_seed(double a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rsq(a);
#else
    // single-precision accuracy, also below the single-precision range
    const double y = 1.0 / __builtin_sqrt(a);
    return y * (1.0 + 0x1p-24);
#endif
}

// sqrt(a) for a normal number a above 2^-900 from a reciprocal square root
// seed y (relative error 2^-24; the hardware's is 2^-24.2): with h = y/2, each
// residual correction g += (a - g^2) h takes g ~ sqrt(a) from relative error
// e to below 2^-23 e, so the second one, far below the last bit, leaves its
// own rounding.
BSDE_F64_HD inline double sqrt_from_seed(double a, double y)
{
    double g = a * y;
    const double h = 0.5 * y;
    g = __builtin_fma(__builtin_fma(-g, g, a), h, g);
    return __builtin_fma(__builtin_fma(-g, g, a), h, g);
}
// for a above 2^-900 (the Box-Muller radius, whose scale the path kernel
// keeps positive)
BSDE_F64_HD inline double sqrt_pos(double a) { return sqrt_from_seed(a, rsqrt_seed(a)); }
// also for a = 0: the seed of a + 2^-1000 (which is a itself unless a is
// zero) stays finite there, and g comes out 0
BSDE_F64_HD inline double sqrt_nonneg(double a)
{
    return sqrt_from_seed(a, rsqrt_seed(a + 0x1p-1000));
}

// ln((w + 1/2) 2^-32) for a 32-bit word w
BSDE_F64_HD inline double log_word(uint32_t w)
{
    const double v = (double)w + 0.5; // exact, in [1/2, 2^32)
    const uint64_t b = to_bits(v);
    const uint32_t hi = (uint32_t)(b >> 32);
    const uint32_t frac_hi = hi & 0x000FFFFFu;
    // mantissas at or above sqrt 2 (its top fraction bits are 0x6A09E)
    // take the next exponent and m in [1/sqrt 2, 1)
    const uint32_t up = frac_hi >= 0x6A09Fu ? 1u : 0u;
    const int e = (int)(hi >> 20) - 1023 + (int)up - 32;
    const double m = from_bits(((uint64_t)(frac_hi | ((0x3FFu - up) << 20)) << 32) |
                               (b & 0xFFFFFFFFull));
    const double f = m - 1.0; // exact
    const double d = m + 1.0;
    // s = f / d from the reciprocal seed y and two residual corrections
    // s += (f - s d) y (each squares the relative error)
    const double y = reciprocal_seed(d);
    double sq = f * y;
    sq = __builtin_fma(__builtin_fma(-sq, d, f), y, sq);
    sq = __builtin_fma(__builtin_fma(-sq, d, f), y, sq);
    const double z = sq * sq;
    // q(z) = 2/3 + 2z/5 + 2z^2/7 + ... by a degree-6 polynomial fitted to its
    // relative error on [0, s_max^2] (Chebyshev nodes, least squares; at most
    // 4.7e-16 with the coefficients in double), in place of the series to
    // z^8: s z q is below 1% of 2 s, so this adds under 5e-18 to ln m
    double q = 0.14616233499191306;
    q = __builtin_fma(q, z, 0.15331740686457643);
    q = __builtin_fma(q, z, 0.18182888493505678);
    q = __builtin_fma(q, z, 0.22222211144430887);
    q = __builtin_fma(q, z, 0.2857142862590908);
    q = __builtin_fma(q, z, 0.3999999999989967);
    q = __builtin_fma(q, z, 0.666666666666667);
    const double ed = (double)e;
    const double hi_part = __builtin_fma(ed, kLn2Hi, 2.0 * sq);
    const double lo_part = __builtin_fma(ed, kLn2Lo, (sq * z) * q);
    return hi_part + lo_part;
}

// e^x for x <= 0 (the local volatility's e^{-y^2})
BSDE_F64_HD inline double exp_nonpos(double x)
{
    x = __builtin_fmax(x, -708.0);
    const double n = __builtin_rint(x * 1.4426950408889634073599246810019);
    double r = __builtin_fma(-n, kLn2Hi, x);
    r = __builtin_fma(-n, kLn2Lo, r);
    double p = 1.0 / 6227020800.0; // 1/13!
    p = __builtin_fma(p, r, 1.0 / 479001600.0);
    p = __builtin_fma(p, r, 1.0 / 39916800.0);
    p = __builtin_fma(p, r, 1.0 / 3628800.0);
    p = __builtin_fma(p, r, 1.0 / 362880.0);
    p = __builtin_fma(p, r, 1.0 / 40320.0);
    p = __builtin_fma(p, r, 1.0 / 5040.0);
    p = __builtin_fma(p, r, 1.0 / 720.0);
    p = __builtin_fma(p, r, 1.0 / 120.0);
    p = __builtin_fma(p, r, 1.0 / 24.0);
    p = __builtin_fma(p, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    // times 2^n, n in [-1022, 0]: exponent field of a normal number
    return p * from_bits((uint64_t)(1023 + (int)n) << 52);
}

// ---------------------------------------------------------------------------
// Table-driven forms for the FP64 path kernels, with the tables in LDS
// (copied by each workgroup from constant data computed at compile time):
//  - ln u of the radius word: u = (w + 1/2) 2^-32 = 2^e m, m in [1/2, 1),
//    bin j of 512 by the top bits of m, with the reciprocal c_j of the bin's
//    centre and -ln c_j: r = m c_j - 1, |r| <= 2^-10, ln u = e ln 2 - ln c_j +
//    ln(1 + r).  e <= 0 and ln m <= 0, so nothing cancels; the last bin has
//    c_j = 1 exactly, so that ln u keeps its relative accuracy as u -> 1;
//  - sine and cosine of the Box-Muller angle: the turn in 1024 sectors
//    centred at j/1024 turns (the axes are centres, so results near zero
//    keep their relative accuracy); the word's remainder rho = w - j 2^22
//    is exact, r = 2 pi (rho + 1/2) 2^-32 lies in [-pi/1024, pi/1024],
//    where sin r and cos r to degrees 5 and 4 leave remainders below 2e-19
//    of r and 2e-18; then the angle-addition formulas with the table's sine
//    and cosine of 2 pi j / 1024;
//  - e^x for x <= 0: x = (256 n + j) ln 2 / 256 + r, |r| <= ln 2 / 512, e^r
//    to degree 4 (remainder below 4e-17 of e^r), times 2^(j/256) and 2^n.
//    The table holds 2^(j/256) with j taken off the exponent field at bit 8
//    below its unit, so that adding the integer 256 n + j there gives
//    2^(n + j/256) in one addition.
// The tables take 26 KB of LDS a workgroup.
// ---------------------------------------------------------------------------
constexpr int kSinCosBins = 1024;
constexpr int kExpBins = 256;
constexpr int kLogBins = 512;
struct alignas(16) Tables {
    double sc[kSinCosBins][2]; // sin, cos of 2 pi j / 1024
    double lg[kLogBins][2];    // c_j, -ln c_j
    double ex[kExpBins];       // 2^(j/256), high word less j << 12
};

// Double-double arithmetic for the tables' compile-time values (error-free
// sums and products of Knuth and Dekker)
struct DD {
    double hi, lo;
};
constexpr DD dd_sum(double a, double b)
{
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
constexpr DD dd_prod(double a, double b)
{
    const double p = a * b;
    const double ca = 134217729.0 * a, ah = ca - (ca - a), al = a - ah;
    const double cb = 134217729.0 * b, bh = cb - (cb - b), bl = b - bh;
    return {p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr DD dd_add(DD a, DD b)
{
    const DD s = dd_sum(a.hi, b.hi);
    return dd_sum(s.hi, s.lo + a.lo + b.lo);
}
constexpr DD dd_mul(DD a, DD b)
{
    const DD p = dd_prod(a.hi, b.hi);
    return dd_sum(p.hi, p.lo + a.hi * b.lo + a.lo * b.hi);
}
constexpr DD dd_div(DD a, DD b)
{
    const double q = a.hi / b.hi;
    const DD r = dd_add(a, dd_mul({-q, 0.0}, b));
    return dd_sum(q, r.hi / b.hi);
}
constexpr DD kDDLn2{0.69314718055994529, 2.3190468138462996e-17};
constexpr DD kDDTwoPi{6.2831853071795862, 2.4492935982947064e-16};

// e^x, sin x and cos x by their Maclaurin series, 0 <= x < 1
struct DDSeries {
    DD exp, sin, cos;
};
constexpr DDSeries dd_series(DD x)
{
    DD term{1.0, 0.0}, part[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    for (int k = 0; k < 28 && term.hi > 1e-36; ++k) {
        part[k & 3] = dd_add(part[k & 3], term);
        term = dd_div(dd_mul(term, x), {(double)(k + 1), 0.0});
    }
    return {dd_add(dd_add(part[0], part[2]), dd_add(part[1], part[3])),
            dd_add(part[1], {-part[3].hi, -part[3].lo}),
            dd_add(part[0], {-part[2].hi, -part[2].lo})};
}
// 2 atanh(1/n) = ln((n + 1) / (n - 1)), n > 1000
constexpr DD dd_log_step(int n)
{
    const DD z = dd_div({1.0, 0.0}, dd_prod((double)n, (double)n));
    DD term = dd_div({2.0, 0.0}, {(double)n, 0.0}), sum{0.0, 0.0};
    for (int k = 1; k < 11; k += 2) {
        sum = dd_add(sum, dd_div(term, {(double)k, 0.0}));
        term = dd_mul(term, z);
    }
    return sum;
}

constexpr Tables make_tables()
{
    Tables T{};
    // the first eighth of the turn, step by step (the errors of the steps
    // stay below 1e-29), and its reflections
    const DDSeries step = dd_series(dd_mul(kDDTwoPi, {1.0 / kSinCosBins, 0.0}));
    DD sd{0.0, 0.0}, cd{1.0, 0.0};
    for (int f = 0; f <= kSinCosBins / 8; ++f) {
        const double s = sd.hi, c = cd.hi;
        for (int q = 0; q < 4; ++q)
            for (int sign = 1; sign >= -1; sign -= 2) {
                const int t = (q * (kSinCosBins / 4) + sign * f) & (kSinCosBins - 1);
                const double sx = sign * s;
                T.sc[t][0] = q == 0 ? sx : q == 1 ? c : q == 2 ? -sx : -c;
                T.sc[t][1] = q == 0 ? c : q == 1 ? -sx : q == 2 ? -c : sx;
            }
        const DD sc = dd_mul(sd, step.cos), cs = dd_mul(cd, step.sin);
        const DD cc = dd_mul(cd, step.cos), ss = dd_mul(sd, step.sin);
        sd = dd_add(sc, cs);
        cd = dd_add(cc, {-ss.hi, -ss.lo});
    }
    T.sc[0][0] = 0.0; // not -0
    T.sc[kSinCosBins / 4][1] = 0.0;
    T.sc[kSinCosBins / 2][0] = 0.0;
    T.sc[3 * kSinCosBins / 4][1] = 0.0;
    // bin j holds m in [512 + j, 513 + j) / 1024; its centre is n / 2048,
    // n = 1025 + 2 j, and ln(n / 2048) goes from bin to bin by ln((n + 2) / n)
    DD lc = dd_add(dd_log_step(2049), {-kDDLn2.hi, -kDDLn2.lo});
    for (int j = 0; j < kLogBins; ++j) {
        const int n = 1025 + 2 * j;
        const double centre = n / 2048.0;
        const double c = 1.0 / centre;
        // ln c = -ln(centre) + ln(c centre), c centre = 1 + delta
        const DD p = dd_prod(c, centre);
        const double delta = (p.hi - 1.0) + p.lo;
        T.lg[j][0] = c;
        T.lg[j][1] = dd_add(lc, {-delta, 0.0}).hi;
        lc = dd_add(lc, dd_log_step(n + 1));
    }
    T.lg[kLogBins - 1][0] = 1.0;
    T.lg[kLogBins - 1][1] = 0.0;
    const DD root = dd_series(dd_mul(kDDLn2, {1.0 / kExpBins, 0.0})).exp;
    DD e{1.0, 0.0};
    for (int j = 0; j < kExpBins; ++j) {
        T.ex[j] = __builtin_bit_cast(
            double, __builtin_bit_cast(uint64_t, e.hi) - ((uint64_t)j << 44));
        e = dd_mul(e, root);
    }
    return T;
}
#if defined(__HIPCC__)
static __device__ const Tables kTables = make_tables();
#else
static constexpr Tables kTables = make_tables();
#endif

// 16-byte parts first, first + stride, ... of the tables
BSDE_F64_HD inline void fill_tables(Tables &T, int first, int stride)
{
    struct alignas(16) Part {
        double a, b;
    };
    constexpr int parts = (int)(sizeof(Tables) / sizeof(Part));
    const Part *src = (const Part *)&kTables;
    Part *dst = (Part *)&T;
#pragma unroll
    for (int t = first; t < parts; t += stride) dst[t] = src[t];
}

// ln((w + 1/2) 2^-32) for a 32-bit word w: 15 FP64 and integer operations
// and one 16-byte LDS read (log_word, with its division and longer series,
// takes 30)
BSDE_F64_HD inline double log_word_tab(uint32_t w, const Tables &T)
{
    const double v = (double)w + 0.5; // exact
#if defined(__HIP_DEVICE_COMPILE__)
    const double m = __builtin_amdgcn_frexp_mant(v);
    const int e = __builtin_amdgcn_frexp_exp(v) - 32;
#else
    int e;
    const double m = frexp(v, &e);
    e -= 32;
#endif
    const uint32_t hi = (uint32_t)(to_bits(m) >> 32);
    const double *row =
        (const double *)((const char *)&T.lg[0][0] + ((hi >> 7) & ((kLogBins - 1) << 4)));
    const double r = __builtin_fma(m, row[0], -1.0);
    // ln(1 + r) = r + r^2 q(r), q of degree 3 interpolating at the Chebyshev
    // nodes of |r| <= 2^-10 (error below 1.9e-14: 2e-17 of r)
    double q = __builtin_fma(r, 0.20000013623927673, -0.2500001589458192);
    q = __builtin_fma(q, r, 0.3333333333333171);
    q = __builtin_fma(q, r, -0.49999999999998107);
    const double l1p = __builtin_fma(r * r, q, r);
    return __builtin_fma((double)e, 0.69314718055994529, row[1]) + l1p;
}

BSDE_F64_HD inline void sincos_turn_tab(uint32_t w, const Tables &T, double &s, double &c)
{
    // nearest sector centre j 2^22 (mod 2^32): the byte offset 16 j of its
    // row, and the signed remainder, the low 22 bits of w
    const uint32_t off = ((w + 0x00200000u) >> 18) & ((kSinCosBins - 1) << 4);
    const int32_t rho = (int32_t)(w << 10) >> 10;
    const double r = __builtin_fma((double)rho, kTwoPiUlp, 0.5 * kTwoPiUlp);
    const double r2 = r * r;
    // sin r = r + r^3 (-1/6 + r^2/120), cos r = 1 + r^2 (-1/2 + r^2/24)
    const double ps = __builtin_fma(r2, kS[1], kS[0]);
    const double pc = __builtin_fma(r2, kC[1], kC[0]);
    const double sr = __builtin_fma(r * r2, ps, r);
    const double cr = __builtin_fma(r2, pc, 1.0);
    const double *row = (const double *)((const char *)&T.sc[0][0] + off);
    const double sa = row[0], ca = row[1];
    s = __builtin_fma(sa, cr, ca * sr);
    c = __builtin_fma(ca, cr, -(sa * sr));
}

// Rounding to an integer by adding and subtracting 1.5 2^52: the sum's low
// word is the integer in two's complement
constexpr double kIntShift = 0x1.8p52;

// 2^(n/256) from the table, n = (int)low word in [-261632, 0] (the result
// is a normal number)
BSDE_F64_HD inline double table_power(uint32_t n, const Tables &T)
{
    const uint64_t b = to_bits(T.ex[n & (kExpBins - 1)]);
    uint32_t hi = (uint32_t)(b >> 32);
#if defined(__HIP_DEVICE_COMPILE__)
    // (written in C this becomes a 64-bit addition with its own shift)
    asm("v_lshl_add_u32 %0, %1, 12, %2" : "=v"(hi) : "v"(n), "v"(hi));
#else
    hi += n << 12;
#endif
    return from_bits(((uint64_t)hi << 32) | (uint32_t)b);
}

// ln 2 / 256 in two parts: the first has 35 significant bits, so
// n kLn2_256Hi is exact for |n| < 2^18 (x >= -708 gives |n| < 261,500)
constexpr double kLn2_256Hi = 0.0027076061741126978;
constexpr double kLn2_256Lo = -5.0411407304988844e-14;

BSDE_F64_HD inline double exp_nonpos_tab(double x, const Tables &T)
{
    x = __builtin_fmax(x, -708.0);
    const double shifted = __builtin_fma(x, 369.32993046757465, kIntShift); // 256 / ln 2
    const double N = shifted - kIntShift;
    double r = __builtin_fma(-N, kLn2_256Hi, x);
    r = __builtin_fma(-N, kLn2_256Lo, r);
    // e^r - 1 = r + r^2 (1/2 + r (1/6 + r / 24))
    double q = __builtin_fma(r, 1.0 / 24.0, 1.0 / 6.0);
    q = __builtin_fma(q, r, 0.5);
    const double em1 = __builtin_fma(q * r, r, r);
    const double t = table_power((uint32_t)to_bits(shifted), T);
    return __builtin_fma(t, em1, t);
}

// 2^((n - f)/256), n = -N: the factor 2^(-f/256) = e^{-f ln 2 / 256},
// |f| <= 1/2, by its Maclaurin series in f to degree 4 (remainder below 4e-17)
// Coefficients (-ln 2 / 256)^k / k!, k = 1..4
constexpr double kE2m[4] = {-0.0027076061740622863, 3.6655655969101062e-06,
                            -3.3083026805413713e-09, 2.239395190875157e-12};
BSDE_F64_HD inline double exp2_parts(uint32_t n, double f, const Tables &T)
{
    double q = __builtin_fma(f, kE2m[3], kE2m[2]);
    q = __builtin_fma(q, f, kE2m[1]);
    q = __builtin_fma(q, f, kE2m[0]);
    const double e = table_power(n, T);
    return __builtin_fma(e, q * f, e);
}

// 2^(-t/256) for t >= 0: t clamped at 261,485 (2^-1021.4, far below the
// volatility's rounding), N = rint(t) and f = t - N (exact, in [-1/2, 1/2])
BSDE_F64_HD inline double exp2_neg_tab(double t, const Tables &T)
{
    t = __builtin_fmin(t, 261485.0);
    const double shifted = kIntShift - t;
    return exp2_parts((uint32_t)to_bits(shifted), t + (shifted - kIntShift), T);
}

// 2^(-y^2/256): the bump volatility's e^{-(x - log c)^2} when the FP64 paths
// carry y = kappa (x - log c) with kappa^2 = 256 log2 e, so that the
// exponent needs no reduction constant.  The square is never rounded by
// itself: N = rint(y^2) and f = y^2 - N come from one fused multiply-add each.
// |y| clamped at 511 (2^-1020; |x - log c| = 26.6).
BSDE_F64_HD inline double exp2_neg_sq_tab(double y, const Tables &T)
{
    double a;
#if defined(__HIP_DEVICE_COMPILE__)
    // (fmin of a value carried through a loop costs a second instruction that
    // quiets signalling NaNs)
    asm("v_min_f64 %0, |%1|, %2" : "=v"(a) : "v"(y), "s"(511.0));
#else
    a = __builtin_fmin(__builtin_fabs(y), 511.0);
#endif
    const double shifted = __builtin_fma(-a, a, kIntShift);
    const double f = __builtin_fma(a, a, shifted - kIntShift);
    return exp2_parts((uint32_t)to_bits(shifted), f, T);
}

} // namespace f64
} // namespace bsde
