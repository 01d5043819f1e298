// Natural logarithm of a positive normal double by table, for the per-bin
// Poisson terms of the basis form: the table-driven method of P. T. P. Tang (ACM
// Trans. Math. Softw. 16, 1990, 378), with the interval from the leading bits of a
// shifted argument and a reciprocal in place of its breakpoint.
//
// x = 2^k z with z in [0.6875, 1.375); the top eight bits of z's offset pick
// one of 256 intervals with a reciprocal c of its centre, r = z c - 1 is formed
// with one rounding (|r| <= 2^-8), and
//   ln x = k ln 2 - ln c + (r - r^2/2 + r^3/3 - ... - r^6/6).
// The two intervals beside z = 1 have c = 1 exactly, so that near x = 1 the
// result is accurate relative to its own small size (near a fit's minimum the
// terms n ln(n / mu) are such numbers); elsewhere its absolute error stays
// within a few 1e-16 times max(1, |ln x|), where the library function's is relative.
//
// 15 instructions and one 16-byte LDS read, against 28 of the series in
// lnpos.h with its reciprocal of (m + 1).  The table is formed by the compiler
// from the series of the inverse hyperbolic tangent.
#pragma once

#include <cmath>
#include <cstring>

namespace nr {

constexpr int kLnTab = 256;
constexpr unsigned kLnOff = 0x3fe60000u;  // high word of 0.6875
constexpr double kLn2 = 0.69314718055994530942;

struct LnEntry {
    double c, l;  // 1 / centre and -ln c
};

struct alignas(16) LnTable {
    LnEntry e[kLnTab];
};

constexpr double ln_centre(int i) {  // centre of interval i
    // intervals below z = 1 are 2^-9 wide, those above 2^-8
    return i < 160 ? 0.6875 + (i + 0.5) / 512.0 : 1.0 + (i - 160 + 0.5) / 256.0;
}

constexpr LnTable make_ln_table() {
    LnTable t{};
    for (int i = 0; i < kLnTab; ++i) {
        const double c = (i == 159 || i == 160) ? 1.0 : 1.0 / ln_centre(i);
        // -ln c = 2 atanh(s), s = (1 - c) / (1 + c), |s| < 0.19
        const double s = (1.0 - c) / (1.0 + c), z = s * s;
        double p = 0.0;
        for (int k = 29; k >= 3; k -= 2) p = (p + 1.0 / k) * z;
        t.e[i].c = c;
        t.e[i].l = 2.0 * s + 2.0 * s * p;
    }
    return t;
}

// x positive and normal; tab: the table, wherever it was placed
#if defined(__HIPCC__)
__host__ __device__
#endif
inline double ln_tab(double x, const LnEntry* tab) {
    unsigned w[2];  // low, high
    memcpy(w, &x, 8);
    const int off = (int)(w[1] - kLnOff);
    const int k = off >> 20;
    const LnEntry t = tab[(off >> 12) & (kLnTab - 1)];
    w[1] -= (unsigned)off & 0xfff00000u;
    double z;
    memcpy(&z, w, 8);
    const double r = fma(z, t.c, -1.0);
    double p = fma(r, -1.0 / 6.0, 1.0 / 5.0);
    p = fma(r, p, -1.0 / 4.0);
    p = fma(r, p, 1.0 / 3.0);
    p = fma(r, p, -0.5);
    return fma((double)k, kLn2, t.l) + fma(r * r, p, r);
}

}  // namespace nr
