// gp_crmath.h -- correctly rounded float32 sin, cos and log for the
// evaluation kernels.
//
// The function set of Sec. III-D1 names sin, cos and log but no library; a
// float32 evaluation that rounds each function's exact value once, to
// nearest (ties to even), as IEEE arithmetic does for +, -, *, / and sqrt,
// makes a program's float32 value independent of which library computed it.
// With these three, every function of the benchmark set {add, sub, mul,
// protected div, neg, protected log, protected sqrt, sin, cos} is correctly
// rounded, so a program's output is one fixed float32 number per row.
//
// Method (each function): the float argument is widened to double (exact),
// the function is evaluated in double with a relative error below 2^-50,
// and the result is rounded to float.  That rounding is the correctly
// rounded one unless the double result lies within the error bound of a
// float rounding boundary (the midpoint of two neighbouring floats); there,
// and only there, an exception table holds the inputs whose double result
// falls on the wrong side (found by running every float through these
// functions against an independent reference, crmath_check.cpp).
//
//   sin, cos: x = k (pi/128) + r, |r| <= pi/256: for |x| < 2^24 by a two-part
//     Cody-Waite reduction whose first product is exact in the FMA; beyond, by
//     Payne-Hanek on |x|: the 24-bit mantissa times a 160-bit window of the
//     binary digits of 2/pi, in 32-bit integer limbs.  Then
//     sin x = S cos r + C sin r with S, C the sine and cosine of
//     (k mod 256) pi/128 from a table (cos x takes k + 64), sin r and cos r by
//     minimax polynomials of two coefficients each.
//   log: a = 2^e m, m in [1, 2); c = 1/(bucket centre of m) from a 256-entry
//     table (c has 24 bits, so m c - 1 is exact); log a = E ln 2 - log c' +
//     log1p(m c - 1) with log1p by a minimax polynomial through r^5
//     (|m c - 1| <= 2^-8), the table's -log c' and ln 2 each rounded to double
//     (four entries then moved, see below).
// Table sizes: 256 entries of 16 bytes each (8 KB of LDS for the two) let the
// polynomials stop two or three operations short of what 128 entries need; a
// table index of eight bits is also a byte of the rounded quotient.  Where a
// last-bit choice in the table decides the rounding of a hard input, the entry
// holds the neighbouring double (gen_crmath_tables.py), so that the common
// paths of sin, cos and log need no exception lookups.  VALU instructions per
// row: sin and cos 17 (23 and 21 with 128 entries, three-part reduction and a
// fix-up of -0), log 20 (27 with exception lookups); measured in a loop of
// each function at three wavefronts per SIMD, 20.0 and 22.6 issue slots.
// The code is host- and device-compilable so that the exhaustive checker can
// run the very same functions on the CPU.  The tables are taken by pointer
// (the evaluation kernels stage them in LDS) and the double constants as a
// struct (sincos_k, log_k: built once per instruction, shared by the rows a
// lane evaluates).
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define GP_CRF __host__ __device__ __forceinline__
#define GP_CRTAB __device__ static constexpr
#else
#include <cmath>
#define GP_CRF inline
#define GP_CRTAB static constexpr
#endif

#include "gp_crmath_tables.h"

namespace gp {
namespace crm {

// A constant handed to a double FMA through a scalar register pair: it is
// then an operand of v_fma_f64 itself, instead of a vector register pair
// the compiler would fill with two moves per use or keep occupied for the
// whole kernel.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ double kreg(double c) {
    asm volatile("" : "+s"(c));
    return c;
}
// The same constant in a vector register pair: the operand of an FMA whose
// other two operands already include a scalar one (one scalar operand per
// vector instruction), set once and shared by the rows of a lane.
__device__ __forceinline__ double kvreg(double c) {
    double v;
    asm volatile("v_mov_b64 %0, %1" : "=v"(v) : "s"(c));
    return v;
}
#else
inline double kreg(double c) { return c; }
inline double kvreg(double c) { return c; }
#endif

GP_CRF uint64_t dbits(double v) {
    uint64_t u;
    __builtin_memcpy(&u, &v, sizeof u);
    return u;
}
GP_CRF uint32_t fbits(float v) {
    uint32_t u;
    __builtin_memcpy(&u, &v, sizeof u);
    return u;
}
GP_CRF float bitsf(uint32_t u) {
    float v;
    __builtin_memcpy(&v, &u, sizeof v);
    return v;
}

// Rounding the double y to float can differ from rounding the exact value
// only if y lies within its error bound of a float rounding boundary: the
// 29 bits below float precision within kHardUlps double ulps of one half.
// (The error bound 2^-50 |y| is at most 2^3 double ulps of y; 16 doubles it.)
constexpr uint32_t kHardUlps = 16;
GP_CRF bool near_boundary(double y) {
    const uint32_t lo = static_cast<uint32_t>(dbits(y)) & 0x1FFFFFFFu;
    return lo - (0x10000000u - kHardUlps) <= 2u * kHardUlps;
}

// The correctly rounded result of an input the exception table lists, else
// the rounding f of the double result.
template <int N>
GP_CRF float exception(const uint32_t (&tab)[N][2], int n, uint32_t key, float f) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("");   // keeps the search behind its (rarely taken) branch
#endif
    for (int i = 0; i < n; ++i)
        if (tab[i][0] == key) return bitsf(tab[i][1]);
    return f;
}

// ---- sin, cos ----
// x = k (pi/128) + r, |r| <= pi/256; with j = k mod 256 (plus 64 for cos,
// cos x = sin(x + pi/2)), sin x = S_j cos r + C_j sin r for S_j, C_j the
// sine and cosine of j pi/128 from a table, and the minimax polynomials
// sin r = r (1 + r^2 (kS3 + kS5 r^2)), error below 2^-55 relative, and
// cos r = 1 + r^2 (kC2 + kC4 r^2), error below 2^-52.
constexpr double kInvPi128 = 0x1.45f306dc9c883p+5;   // 128/pi
// pi/128 = kPi128a + kPi128b + O(2^-113)
constexpr double kPi128a = 0x1.921fb54442d18p-6;
constexpr double kPi128b = 0x1.1a62633145c07p-60;
constexpr double kS3 = -0x1.5555555544483p-3, kS5 = 0x1.1110b7b9a17b3p-7;
constexpr double kC2 = -0x1.ffffffffc4522p-2, kC4 = 0x1.5554b8fc59271p-5;

// 1.5 * 2^52: x + kRound is x rounded to an integer, held in the low bits of
// the double's significand (|x| < 2^51); cos adds its quarter turn, 64
// table steps, in the same operation
constexpr double kRound = 0x1.8p+52;
constexpr double kRoundCos = 0x1.8p+52 + 64.0;

// inputs from here on (in magnitude) take the Payne-Hanek reduction
constexpr float kSinCosLarge = 0x1p+24f;

// The double constants of sin (is_cos false) or cos as operands.  The
// kernels build this once per instruction and share it among the rows a lane
// holds.
struct SinCosK {
    double inv, rnd, pa, pb, s3, s5, c2, c4;
};
GP_CRF SinCosK sincos_k(bool is_cos) {
    return SinCosK{kreg(kInvPi128), kvreg(is_cos ? kRoundCos : kRound), kreg(kPi128a), kreg(kPi128b),
                   kvreg(kS3),      kreg(kS5),                          kvreg(kC2),    kreg(kC4)};
}

// sin r and cos r for |r| <= pi/256 (slightly more after rounding of k).
// The sign of a zero r is kept: sin r = r (1 + ...).
GP_CRF void sincos_poly(double r, const SinCosK& K, double* sr, double* cr) {
    const double r2 = r * r;
    *sr = r * fma(r2, fma(K.s5, r2, K.s3), 1.0);
    *cr = fma(r2, fma(K.c4, r2, K.c2), 1.0);
}
// sin(j pi/128 + r) and its derivative cos(j pi/128 + r)
GP_CRF double sin_from_table(const SinCosEntry& e, double r, const SinCosK& K) {
    double sr, cr;
    sincos_poly(r, K, &sr, &cr);
    return fma(e.c, sr, e.s * cr);
}

// |x| < 2^24: k and r by a two-part Cody-Waite reduction.  k is the integer
// nearest x * 128/pi (from the exact product: a tie or a neighbouring integer
// only moves r within the polynomials' range), and the low word of
// x * 128/pi + K.rnd is k (k + 64 for cos) modulo 2^32, so that a negative k
// indexes the table as k mod 256 does.  x - k kPi128a is a multiple of 2^-58
// below 2^-5 (x is a multiple of 2^-30 where k is not 0), so the first FMA is
// exact; the second rounds once, and the part of pi/128 left out is below
// k 2^-113 < 2^-83.  Every step is odd in x (k, r and the table's sines change
// sign, its cosines do not), zeros included (the table's sine of 0 is -0), so
// sin(-x) = -sin x and cos(-x) = cos x hold bit for bit.
struct SinCosArg {
    double r;
    uint32_t off;   // byte offset of entry (k or k + 64) mod 256
};
GP_CRF SinCosArg sincos_reduce(double x, const SinCosK& K) {
    const double kr = fma(x, K.inv, K.rnd);
    const double k = kr - K.rnd;
    const double r = fma(-k, K.pb, fma(-k, K.pa, x));
    return SinCosArg{r, (static_cast<uint32_t>(dbits(kr)) & 0xFFu) << 4};
}
GP_CRF const SinCosEntry& sincos_entry(const SinCosEntry* tab, uint32_t off) {
    return *reinterpret_cast<const SinCosEntry*>(reinterpret_cast<const char*>(tab) + off);
}
GP_CRF double sincos_small(double x, const SinCosEntry* tab, const SinCosK& K) {
    const SinCosArg a = sincos_reduce(x, K);
    return sin_from_table(sincos_entry(tab, a.off), a.r, K);
}

// The binary digits of 2/pi in 32-bit words, after one word of zeros (the
// word index of digit p >= 1, weight 2^-p, is (p + 31) / 32).
GP_CRTAB uint32_t kTwoOverPi[13] = {0u,          0xa2f9836eu, 0x4e441529u, 0xfc2757d1u, 0xf534ddc0u,
                                   0xdb629599u, 0x3c439041u, 0xfe5163abu, 0xdebbc561u, 0xb7246e3au,
                                   0x424dd2e0u, 0x06492eeau, 0x09d1921cu};

// Payne-Hanek for finite |x| = M 2^E >= 2^24 (ub: the float bits of |x|).
// Digits of 2/pi of weight 2^(E-p) >= 4 multiply the integer M into
// multiples of 4 and are dropped: the window is digits p = E-1 .. E+158 (160
// bits), so Z = M * window * 2^-158 = |x| 2/pi mod 4 carries 158 fraction
// bits and an error below 2^-134.  64 Z = |x| 128/pi mod 256: k is its
// nearest integer (bits 152 up, after adding 2^151) and r = (64 Z - k) pi/128.
GP_CRF double sincos_large(uint32_t ub, bool is_cos, const SinCosEntry* tab, const SinCosK& K) {
    const uint32_t M = (ub & 0x7FFFFFu) | 0x800000u;
    const int E = static_cast<int>(ub >> 23) - 150;
    const int p0 = E - 1;
    const int k0 = (p0 + 31) >> 5;
    const int s = (p0 + 31) & 31;
    uint32_t z[5];
    uint64_t c = 0;
    for (int j = 4; j >= 0; --j) {
        const uint32_t w = s ? (kTwoOverPi[k0 + j] << s) | (kTwoOverPi[k0 + j + 1] >> (32 - s))
                             : kTwoOverPi[k0 + j];
        const uint64_t t = static_cast<uint64_t>(M) * w + c;
        z[j] = static_cast<uint32_t>(t);
        c = t >> 32;
    }
    // bit 151 of Z is bit 23 of z[0]; k = bits 152..159
    z[0] += 0x800000u;
    const int k = static_cast<int>(z[0] >> 24);
    const int j = (k + (is_cos ? 64 : 0)) & 255;
    // D = (bits 0..151) - 2^151: signed, 152 fraction bits of 64 Z
    const int64_t top = static_cast<int64_t>(z[0] & 0xFFFFFFu) - 0x800000ll;
    const bool dneg = top < 0;
    uint32_t d[5] = {static_cast<uint32_t>(top), z[1], z[2], z[3], z[4]};
    if (dneg) {   // |D|: two's complement negation across the limbs
        uint64_t b = 1;
        for (int i = 4; i >= 0; --i) {
            const uint64_t t = static_cast<uint64_t>(~d[i]) + b;
            d[i] = static_cast<uint32_t>(t);
            b = t >> 32;
        }
    }
    // normalise |D| to 64 significant bits
    int j0 = 0;
    while (j0 < 2 && d[j0] == 0u) ++j0;
    const int l = __builtin_clz(d[j0] | 1u);   // (d[j0] != 0 for every float input)
    uint64_t hi = (static_cast<uint64_t>(d[j0]) << 32) | d[j0 + 1];
    if (l) hi = (hi << l) | (d[j0 + 2] >> (32 - l));
    double D = ldexp(static_cast<double>(hi), 160 - 64 - 152 - 32 * j0 - l);
    if (dneg) D = -D;
    return sin_from_table(tab[j], D * kPi128a, K);
}

// Correctly rounded sin (is_cos false) or cos of a float, in two parts so
// that a lane holding several rows can test them all before one branch:
// sincos_common is the result for |x| < 2^24, without a branch or an exception
// (the exhaustive checker finds none there); an input for which
// sincos_rare_input holds (|x| >= 2^24, inf, NaN) takes sincos_rare's
// result instead: Payne-Hanek reduction, or NaN.  Tiny arguments need no
// case of their own: for |x| < 2^-12 the double result lies within
// x^2 / 6 < 2^-26.6 (relative) of x, or x^2 / 2 < 2^-25 of 1, so it rounds
// to x (sin) or 1 (cos), as the exact value does.
GP_CRF float sincos_common(float x, const SinCosEntry* tab, const SinCosK& K) {
    // (an input sincos_rare_input flags gets a meaningless value here, read
    // from within the table since its offset is masked, and replaced by
    // sincos_rare's)
    return static_cast<float>(sincos_small(static_cast<double>(x), tab, K));
}

GP_CRF bool sincos_rare_input(float x) { return !(fabsf(x) < kSinCosLarge); }   // (NaN included)

GP_CRF float sincos_rare(float x, bool is_cos, const SinCosEntry* tab, const SinCosK& K) {
    const uint32_t ub = fbits(x) & 0x7FFFFFFFu;
    float f;
    if (ub < 0x7F800000u) {
        const double yl = sincos_large(ub, is_cos, tab, K);
        f = static_cast<float>(yl);
        if (near_boundary(yl))
            f = is_cos ? exception(kCosExc, kCosExcN, ub, f) : exception(kSinExc, kSinExcN, ub, f);
    } else {
        f = x - x;   // NaN
    }
    return (!is_cos && (fbits(x) >> 31)) ? -f : f;
}

GP_CRF float sincos_cr(float x, bool is_cos, const SinCosEntry* tab, const SinCosK& K) {
    float f = sincos_common(x, tab, K);
    if (sincos_rare_input(x)) f = sincos_rare(x, is_cos, tab, K);
    return f;
}

GP_CRF float sin_cr(float x, const SinCosEntry* tab, const SinCosK& K) { return sincos_cr(x, false, tab, K); }
GP_CRF float cos_cr(float x, const SinCosEntry* tab, const SinCosK& K) { return sincos_cr(x, true, tab, K); }

// ---- log ----
// ln 2 rounded to double: E ln 2 is then off by |E| 2^-55.3 at most, which
// is below 2^-53.8 of the result for every E != 0 (|log a| >= |E| ln 2 -
// ln(2)/2 there)
constexpr double kLn2 = 0x1.62e42fefa39efp-1;
// log1p r = r + r^2 (kL2 + kL3 r + kL4 r^2 + kL5 r^3) for -0.55 2^-8 <= r <=
// 2^-8, minimax relative to r: error below 2^-48 of r, attained only at the
// ends, so that with a table entry L != 0 it is below 2^-50 of the result,
// and in the two buckets with L = 0 the exhaustive checker decides
constexpr double kL2 = -0x1.fffffffffdc11p-2, kL3 = 0x1.55555589a58bdp-2, kL4 = -0x1.00002862ec298p-2,
                 kL5 = 0x1.9830ade37075bp-3;

struct LogK {
    double l2, l3, l4, l5, ln2;
};
GP_CRF LogK log_k() { return LogK{kreg(kL2), kreg(kL3), kvreg(kL4), kreg(kL5), kreg(kLn2)}; }

// the mantissas from 1 + 106/256 (about sqrt 2) on are halved and their
// exponent raised by one: adding 150 steps of 2^-8 carries them into it
constexpr uint32_t kLogCarry = 150u << 15;

// log a for a normal positive finite float given by its bits u (the sign is
// ignored), in double: E ln 2 + L + log1p(r) with r = m c - 1 exact (24-bit m
// times the 24-bit c).  The table's L carries its double rounding, below
// 2^-53 |L|.  Where E = 0 and L != 0, |r| <= 0.34 |L|, so the result is at
// least 0.66 |L| and that rounding is below 2^-52.4 of it; with the rounding
// of log1p and of the final addition the relative error stays below 2^-50
// (E ln 2 + L is exact when E = 0).  That bound does not hold in the four
// buckets whose L is not -log(c) rounded but moved by 8 to 192 units
// (gen_crmath_tables.py, NUDGE): with E near 0 they are within 2^-45 only, and
// what carries the claim there, as for every float, is the exhaustive check.
GP_CRF double log_double(uint32_t u, const LogEntry* tab, const LogK& K) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int E = __builtin_amdgcn_frexp_expf(bitsf(u + kLogCarry - 0x800000u));
#else
    const int E = static_cast<int>(((u + kLogCarry) >> 23) & 0xFFu) - 127;
#endif
    const double m = static_cast<double>(bitsf((u & 0x7FFFFFu) | 0x3F800000u));
    // byte offset of the entry of the top eight mantissa bits
    const uint32_t off = (u >> 11) & 0xFF0u;
    const LogEntry& t = *reinterpret_cast<const LogEntry*>(reinterpret_cast<const char*>(tab) + off);
    const double r = fma(m, t.c, -1.0);   // exact
    const double p = fma(fma(fma(K.l5, r, K.l4), r, K.l3), r, K.l2);
    const double l1p = fma(r * r, p, r);
    return fma(static_cast<double>(E), K.ln2, t.hi) + l1p;
}

// Correctly rounded log of a float a > 0 that is normal, +inf or NaN (the
// protected log only takes |a| > 0.001).  No input needs an exception.
static_assert(kLogExcN == 0, "log takes no exception lookups");
GP_CRF float log_cr(float a, const LogEntry* tab, const LogK& K) {
    const float f = static_cast<float>(log_double(fbits(a), tab, K));   // (finite for +inf and NaN; replaced below)
    return a <= 0x1.fffffep+127f ? f : a;                               // +inf (and NaN) unchanged
}

// ---- log(1 + e^-a), the log-loss's ----
// In double, rounded once: e = e^-a as 2^k p(s) with s = -a - k ln 2, |s| <=
// ln 2 / 2 and p its series through s^8 (relative error below 2^-31.7), then the
// log of x = 1 + e in [1, 2) from log's table.  d is what 1 + e rounds off, so
// that the result keeps its relative precision down to the smallest e (the
// table's first entry has c = 1 and L = 0).  From a = 200 on the result is 0 in
// float.  Within 0.503 units in the last place of every float tried (one in 97
// up to 208; the device library's log1pf(expf(-a)) 1.5), in some 45 VALU
// instructions a row fewer: 500 programs of up to 200 nodes on 1.1M rows of 28
// features, 9.80 ms with the library's, 9.16 with this.
constexpr double kLog2e = 0x1.71547652b82fep+0;
constexpr double kRound52 = 0x1.8p+52;
constexpr double kInvFact[9] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320};

GP_CRF float log1p_exp_neg(float a, const LogEntry* tab, const LogK& K) {
    const double A = static_cast<double>(a < 200.0f ? a : 200.0f);     // (200 for NaN; the caller's own terms keep that)
    const double kr = fma(A, -kLog2e, kRound52);
    const double s = fma(kr - kRound52, -kLn2, -A);
    double p = kInvFact[8];
    for (int q = 7; q >= 0; --q) p = fma(p, s, kInvFact[q]);
    const uint64_t pb = dbits(p) + (static_cast<uint64_t>(static_cast<uint32_t>(dbits(kr))) << 52);
    double e;
    __builtin_memcpy(&e, &pb, sizeof e);
    e = e < 0x1.ffffffffffffep-1 ? e : 0x1.ffffffffffffep-1;           // x stays below 2
    const double x = 1.0 + e;
    const double d = e - (x - 1.0);
    const uint32_t hi = static_cast<uint32_t>(dbits(x) >> 32);
    const LogEntry& t = *reinterpret_cast<const LogEntry*>(reinterpret_cast<const char*>(tab) + ((hi >> 8) & 0xFF0u));
    // (as in log_double, mantissas from 1 + 106/256 on count as halved)
    const double base = t.hi + (hi >= 0x3FF6A000u ? kLn2 : 0.0);
    const double r = fma(d, t.c, fma(x, t.c, -1.0));
    const double q = fma(fma(fma(K.l5, r, K.l4), r, K.l3), r, K.l2);
    return static_cast<float>(base + fma(r * r, q, r));
}

}  // namespace crm
}  // namespace gp
