// Critical values of the chi-square distribution (host code, no HIP): the
// statistics that enclose the decisions of one alpha, so that the depths that
// run from bit planes evaluate no tail outside them.  Computed for each call,
// for the degrees of freedom that the call can reach: about 0.06 us a value, so
// an alpha that was not seen before costs what a repeated one does.
#pragma once

#include <array>
#include <cmath>
#include <limits>

namespace bns {

constexpr int kCritDf = 128;  // df below this; bit planes reach (kBitCards - 1)^2 kBitCards = 80

// 1 / (k + h) for the terms of the closed forms.
struct CritInv {
    double v[2][kCritDf];
    constexpr CritInv() : v() {
        for (int k = 0; k < kCritDf; ++k) {
            v[0][k] = 1.0 / (double)(k + 1);
            v[1][k] = 1.0 / ((double)(k + 1) + 0.5);
        }
    }
};
inline constexpr CritInv kCritInv{};

// Upper tail of the chi-square distribution with df degrees of freedom at 2 x
// and the Gamma(df / 2, 1) density there (closed forms for integer df).
inline double chi2_upper(int df, double x, double *dens) {
    const double pi = 3.141592653589793;
    const int odd = df & 1, n = df >> 1;
    double term = odd ? 2.0 * std::sqrt(x / pi) : 1.0, sum = 0.0, last = 0.0;
    for (int k = 0; k < n; ++k) {
        sum += term;
        last = term;
        term *= x * kCritInv.v[odd][k];
    }
    const double ex = std::exp(-x);
    *dens = n > 0 ? ex * last : ex / std::sqrt(pi * x);
    return (odd ? std::erfc(std::sqrt(x)) : 0.0) + ex * sum;
}

// z with upper normal tail q in (0, 1) (Abramowitz and Stegun 26.2.23: to 5e-4).
inline double normal_upper(double q) {
    const double u = std::sqrt(-2.0 * std::log(q < 0.5 ? q : 1.0 - q));
    const double z = u - (2.515517 + 0.802853 * u + 0.010328 * u * u) /
                             (1.0 + 1.432788 * u + 0.189269 * u * u + 0.001308 * u * u * u);
    return q < 0.5 ? z : -z;
}

// x with chi2_upper(df, x) = q, q in [1e-90, 1 - 1e-9], to a part in 10^6; zn =
// normal_upper(q).  Halley's method from the Wilson-Hilferty approximation, kept inside a shrinking
// bracket: with the density g and its slope g r, r = (df / 2 - 1) / x - 1, a
// step of h leaves about h (h r)^2 / 12, so usually one evaluation does.
inline double chi2_half_quantile(int df, double q, double zn) {
    if (df == 2) return -std::log(q);
    const double wh = 2.0 / (9.0 * df), c = 1.0 - wh + zn * std::sqrt(wh), a1 = 0.5 * df - 1.0;
    double x = std::fmax(0.5 * df * c * c * c, 1e-3 * df), lo = 0.0, hi = 700.0;
    if (!(x < hi)) x = 0.5 * hi;
    for (int it = 0; it < 200; ++it) {
        double g;
        const double f = chi2_upper(df, x, &g) - q;
        if (f > 0) lo = x;
        else hi = x;
        const double h0 = f / g, r = a1 / x - 1.0, h = h0 / (1.0 + 0.5 * h0 * r);
        double nx = x + h;
        const bool in = nx > lo && nx < hi;
        if (!in) nx = 0.5 * (lo + hi);
        const bool done = (in && std::fabs(h) <= 5e-3 * x && std::fabs(h0 * r) <= 0.02) || hi - lo <= 1e-12 * hi;
        x = nx;
        if (done) break;
    }
    return x;
}

struct CritVal {
    double x, y;
};
using CritMask = std::array<bool, kCritDf>;  // degrees of freedom in use

// out[df] for the degrees of freedom of need: a statistic below x has p >
// alpha + reach, one above y has p < alpha - reach (others: nothing certain).
// reach covers the re-check band and, with 1e-3, four times the propagated
// FP32 error bound (at most 1e-4 for df < kCritDf).
inline void crit_values(double alpha, double band, const CritMask &need, CritVal *out) {
    const double reach = std::fmax(band, 1e-3), inf = std::numeric_limits<double>::infinity();
    const double up = alpha + reach, dn = alpha - reach;
    const double zu = up < 1.0 - 1e-9 ? normal_upper(up) : 0.0, zd = dn > 1e-12 ? normal_upper(dn) : 0.0;
    for (int df = 0; df < kCritDf; ++df) {
        out[df] = CritVal{0.0, inf};
        if (df == 0 || !need[(size_t)df]) continue;
        // (a part in 10^5 to spare)
        if (up < 1.0 - 1e-9) out[df].x = 2.0 * chi2_half_quantile(df, up, zu) * (1.0 - 1e-5);
        if (dn > 1e-12) out[df].y = 2.0 * chi2_half_quantile(df, dn, zd) * (1.0 + 1e-5);
    }
}

// The degrees of freedom of the tests of depths 0 and 1 of variables whose
// cardinalities (at most max_card) are marked in card: (a - 1)(b - 1) and
// (a - 1)(b - 1) c, or with adjusted df everything up to the largest.
inline CritMask crit_need(const bool *card, int max_card, bool adjusted) {
    CritMask need{};
    int top = 0;
    for (int a = 2; a <= max_card; ++a)
        for (int b = a; b <= max_card; ++b) {
            if (!card[a] || !card[b]) continue;
            const int d = (a - 1) * (b - 1);
            need[(size_t)d] = true;
            for (int c = 2; c <= max_card; ++c)
                if (card[c]) {
                    need[(size_t)(d * c)] = true;
                    if (d * c > top) top = d * c;
                }
        }
    for (int d = 1; adjusted && d <= top; ++d) need[(size_t)d] = true;
    return need;
}

}  // namespace bns
