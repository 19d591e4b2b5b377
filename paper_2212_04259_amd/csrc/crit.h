// Critical values of the chi-square distribution (host code, no HIP): the
// statistics that enclose the decisions of one alpha, so that the depths that
// run from bit planes evaluate no tail outside them.  Computed for the degrees
// of freedom that a call can reach, about 0.1 us each (1.4 us an alpha for two
// to four categories, 7.5 for the adjusted df of up to five), and kept for the
// next call with the same alphas.
#pragma once

#include <array>
#include <cmath>
#include <limits>

namespace bns {

constexpr int kCritDf = 96;  // df below this; bit planes reach (kBitCards - 1)^2 kBitCards = 80

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

// A quantile x (half a statistic) and the density there, to a part in 10^5 and
// in 10 for tails in [1e-90, 1 - 1e-9].
struct HalfQuantile {
    double x, g;
};

// x with chi2_upper(df, x) = q by Halley's method from (x, its tail - q, its
// density), kept inside a shrinking bracket.  With the density's slope g r, r =
// (df / 2 - 1) / x - 1, a step of h leaves at most about h (h r)^2 / 6.
inline HalfQuantile chi2_solve(int df, double q, double x, double f, double g) {
    const double a1 = 0.5 * df - 1.0;
    double lo = 0.0, hi = 700.0;
    for (int it = 0; it < 200; ++it) {
        if (f > 0) lo = x;
        else hi = x;
        const double h0 = f / g, r = a1 / x - 1.0, h = h0 / (1.0 + 0.5 * h0 * r);
        const bool in = x + h > lo && x + h < hi;
        if ((in && std::fabs(h) <= 0.02 * x && std::fabs(h0 * r) <= 0.05) || hi - lo <= 1e-12 * hi)
            return HalfQuantile{in ? x + h : x, g * (1.0 + h * r)};
        x = in ? x + h : 0.5 * (lo + hi);
        f = chi2_upper(df, x, &g) - q;
    }
    return HalfQuantile{x, g};
}

// The same from the Wilson-Hilferty approximation; zn = normal_upper(q).
// Usually one evaluation.
inline HalfQuantile chi2_half_quantile(int df, double q, double zn) {
    if (df == 2) return HalfQuantile{-std::log(q), q};
    const double wh = 2.0 / (9.0 * df), c = 1.0 - wh + zn * std::sqrt(wh);
    const double x = std::fmin(std::fmax(0.5 * df * c * c * c, 1e-3 * df), 350.0);
    double g;
    const double f = chi2_upper(df, x, &g) - q;
    return chi2_solve(df, q, x, f, g);
}

// Statistics that enclose the decisions of one alpha and df.  An FP32
// statistic below x has p > alpha + band, one above y has p < alpha - band, by
// more than four times its error bound (a relative error below 4e-6 for the
// tables of the bit-plane paths); an FP64 statistic below x64 has p > alpha,
// one above y64 has p < alpha.
struct CritVal {
    double x, y, x64, y64;
};
constexpr double kCritSpare32 = 1e-4, kCritSpare64 = 4e-5;
using CritMask = std::array<bool, kCritDf>;  // degrees of freedom in use

// out[df] for the degrees of freedom of need (others: nothing certain).  fp64:
// no FP32 statistic is compared (x and y are x64 and y64).
inline void crit_values(double alpha, double band, bool fp64, const CritMask &need, CritVal *out) {
    const double inf = std::numeric_limits<double>::infinity();
    const bool able = alpha >= 1e-90 && alpha <= 1.0 - 1e-9;
    const double zn = able ? normal_upper(alpha) : 0.0;
    const double up = alpha + band;
    // (alpha = band: a p below half an ulp of alpha is not within the band)
    const double dn = alpha == band ? alpha * 1e-16 : alpha - band;
    for (int df = 0; df < kCritDf; ++df) {
        CritVal v{0.0, inf, 0.0, inf};
        if (able && need[(size_t)df]) {
            const HalfQuantile h = chi2_half_quantile(df, alpha, zn);
            v.x64 = 2.0 * h.x * (1.0 - kCritSpare64);
            v.y64 = 2.0 * h.x * (1.0 + kCritSpare64);
            if (fp64) {
                v.x = v.x64;
                v.y = v.y64;
            } else {
                if (up <= 1.0 - 1e-9) v.x = 2.0 * chi2_solve(df, up, h.x, -band, h.g).x * (1.0 - kCritSpare32);
                if (dn >= 1e-90) v.y = 2.0 * chi2_solve(df, dn, h.x, alpha - dn, h.g).x * (1.0 + kCritSpare32);
            }
        }
        out[df] = v;
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
