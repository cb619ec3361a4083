// A track's column from a power series about one time of a chunk of segments, with
// a bound on its error that says when the column is certain.
//
// With tc a time of the chunk, U = 1 + (tc - T0)/tau and d = (t - tc)/(tau + tc - T0),
// the spin-down factor of Eq. 1 is U^e (1 + d)^e, so
//     x = f0 g D T_sft ~ A (1 + c1 d + ... + c6 d^6) D,
//     A = f0 T_sft U^e, c_k = C(e, k).
// Against the contract's chain of correctly rounded operations x is off by less than
//     m = 2 A (1.25 |C(e, 7)| dmax^7 + (1 + |y| + |e|) 2^-44),  y = e log U,
// for |d| <= dmax <= 1/8, -4 <= e < 0 and any 0 < D < 2 (|v| < c):
//   the truncation, whose terms shrink by at most (7 + |e|)/8 dmax <= 11/64 each: below
//   1.25 |C(e, 7)| dmax^7 A D, the first term of m;
//   relative to x, which (1 + d)^e <= (7/8)^-4 < 1.71 keeps below 1.71 A D < 3.42 A: the
//   enclosure value's 2^-50 (1 + |y| + |e|) in A and 3 |e| 2^-53 for its U; the chain's
//   own (3 |e| + 6) 2^-53; and at most 60 2^-53 for d, the coefficients, the polynomial
//   (sum |c_k d^k| < 1.71 as well) and the products, together below
//   2^-46.6 (1 + |y| + |e|) and so below 2^-44.8 A (1 + |y| + |e|), of a second term
//   twice as large and more;
//   2^-51 in D itself where it is formed by FMAs, below 2^-50.2 A.
// The column trunc(x + 1.5 - k_lo) is then certain unless x + 1.5 - k_lo lies within
// m of an integer.  It is taken on top of 2^20, where the sum's low word is its
// fraction in units of 2^-32 and the low 20 bits of its high word its integer part:
// for x < 2^19, k_lo < 2^18 and rows of fewer than 2^18 columns (a negative
// column wraps to at least 2^19, past any row).
#pragma once
#include "pow_enclose.h"

#pragma clang fp contract(off)

namespace ltgw {

// Where the series is used: dmax, |e| and m in bins.
constexpr double kExpandMaxStep = 0.125, kExpandMaxE = 4.0, kExpandMaxMargin = 0x1p-14;

// C(e, 1) .. C(e, 7)
LTGW_HD void expand_series(double e, double (&c)[7]) {
    double v = e;
    c[0] = v;
#pragma unroll
    for (int k = 1; k < 7; ++k) {
        v = v * ((e - (double)k) * (1.0 / (double)(k + 1)));
        c[k] = v;
    }
}

// m; c7 = C(e, 7)
LTGW_HD double expand_margin(double A, double dmax, double c7, double y, double e) {
    const double d2 = dmax * dmax;
    return (A + A) * (1.25 * std::fabs(c7) * ((d2 * d2) * (d2 * dmax)) +
                      ((1.0 + std::fabs(y)) + std::fabs(e)) * 0x1p-44);
}

LTGW_HD bool expand_holds(double dmax, double m, double e) {
    return dmax <= kExpandMaxStep && m <= kExpandMaxMargin && e >= -kExpandMaxE;
}

// The margin in units of 2^-32, with the rounding of the sum on 2^20.
LTGW_HD unsigned expand_margin_units(double m) { return (unsigned)(m * 0x1p32) + 4u; }

// k[0..6] = A, A c1 .. A c6
LTGW_HD double expand_x(const double (&k)[7], double d, double D) {
    double p = k[6];
#pragma unroll
    for (int i = 5; i >= 0; --i) p = std::fma(p, d, k[i]);
    return p * D;
}

// shift20 = 2^20 + 1.5 - k_lo.  The column; *z below 2 mi: not certain.
LTGW_HD unsigned expand_column(double x, double shift20, unsigned mi, unsigned *z) {
    const uint64_t w = bits_of(x + shift20);
    *z = (unsigned)w + mi;
    return (unsigned)(w >> 32) & 0xfffffu;
}

}  // namespace ltgw
