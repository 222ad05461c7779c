// pt_rows.hpp -- exchange thresholds of a pair of neighbouring temperatures
// (Sec. "Parallel Tempering", Eq. pt): ceil(exp(x) 2^32), x = (beta_i -
// beta_{i+1}) 4m, for the energy differences 4m, m = 1 .. mmax, as a row that
// ends where the threshold is constant.  Plain C++ but for pt_threshold, which
// the exchange kernel calls.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace mcs {

// Entry 0 of a row (no exchange asks for it): the call's first round above these
// bits, in them the first m whose threshold is 0.
constexpr int kPtZeroBits = 24;

// The threshold is 1 from x = -22.5 (exp(x) 2^32 < 0.73) until exp(x) is 0: the
// entries up to `cut`, and the first m whose threshold is 0.
struct PtPair {
    int64_t cut, zero;
};

inline PtPair pt_pair(double b0, double b1, int64_t mmax)
{
    const double d = b0 - b1;
    auto first_below = [&](double x) {  // first m with d 4m < x, at most mmax + 1
        const double m = std::floor(x / (4.0 * d));
        int64_t k = m < 0.0 ? 0 : m > (double)mmax ? mmax + 1 : (int64_t)m;
        while (k <= mmax && !(d * (double)(4 * k) < x)) ++k;
        return k;
    };
    PtPair p;
    p.cut = std::min(first_below(-22.5), mmax);
    p.zero = first_below(-744.0);
    while (p.zero <= mmax && std::exp(d * (double)(4 * p.zero)) != 0.0) ++p.zero;
    return p;
}

// The row of a pair, `row` > cut entries.
inline void pt_row(double b0, double b1, const PtPair &p, int64_t row, uint64_t round0, uint64_t *x)
{
    x[0] = round0 << kPtZeroBits | (uint64_t)p.zero;
    for (int64_t m = 1; m <= p.cut; ++m) x[m] = (uint64_t)std::ceil(std::ldexp(std::exp((b0 - b1) * (double)(4 * m)), 32));
    for (int64_t m = p.cut + 1; m < row; ++m) x[m] = m < p.zero ? 1u : 0u;
}

// The threshold of m >= 1: beyond the row 1, then 0.
constexpr uint64_t pt_threshold(const uint64_t *x, int row, int m)
{
    return m < row ? x[m] : m < (int)(x[0] & ((1u << kPtZeroBits) - 1u)) ? 1u : 0u;
}

}  // namespace mcs
