// The dyadic pair that a residual layer's kernels use for the residual term (host arithmetic only).
#pragma once
#include <stdint.h>

#include <initializer_list>

namespace ivit {

// A residual value is one of 256, and the kernels' 24-bit form of its term takes b < 2^23 and c <= 30.  For a pair beyond that: one
// within it that gives the same term for all 256 values, the pair rounded to 23 bits or its neighbour (for almost every pair one
// of them does), or the pair itself where neither does, which then takes 64-bit arithmetic.  1576 x 2304 x 768 with a pair of 30 bits,
// whose term was a 64-bit multiply-add of its own until the 24-bit form: 8.3 us then, 8.6 in 64-bit arithmetic, 8.0 with this.
struct ResidualPair { int32_t b, c; };
inline ResidualPair residual_pair(int32_t b, int32_t c, int rnd) {
    int k = c > 30 ? c - 30 : 0;
    while (k < 31 && b >> k >= 1 << 23) ++k;
    if (k == 0 || k > 30 || b < 1 || c - k < 1) return ResidualPair{b, c};
    const int32_t near = (int32_t)(((int64_t)b + ((int64_t)1 << (k - 1))) >> k), other = (b >> k) + (near == b >> k);
    for (const int32_t t : {near, other}) {
        if (t < 1 || t >= 1 << 23) continue;
        const int cc = c - k;
        bool same = true;
        for (int v = -128; v < 128 && same; ++v)
            same = ((int64_t)v * b + ((int64_t)rnd << (c - 1))) >> c == ((int64_t)v * t + ((int64_t)rnd << (cc - 1))) >> cc;
        if (same) return ResidualPair{t, cc};
    }
    return ResidualPair{b, c};
}

}  // namespace ivit
