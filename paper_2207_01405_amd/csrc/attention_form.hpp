// Which Shiftmax parameters take the 24-bit IntDiv of attention.hip (host arithmetic only).
#pragma once
#include <stdint.h>

namespace ivit {

// That form divides by one 24 x 24-bit product of which the upper word is the quotient: with M - (k_out - 1) = 24 it is
// (inv 2^(8-up)) (e 2^up) / 2^32, inv = floor(2^M / sum) the row's reciprocal and e an entry of the ShiftExp table, which is kept in
// 16 bits and scaled by 2^up.  The number of bits `up`, or -1 where it does not apply.  With e0 = I_0 << N, the largest entry
// and the smallest sum, in [2^j, 2^(j+1)): e0 2^up <= 2^(M-15) - 2^up takes 16 bits, and inv 2^(8-up) <= 2^24, with equality only
// for sum = e0 = 2^j, where the reciprocal is lowered by one (see div_factor).  Below e0 = 2^(k_out-1) + 1 the reciprocal alone can
// have more than 24 bits.  Against the 32-bit form at e0 = 2^14 and 2^8: 3072 pairs of 197 tokens and 64 features 66.1 -> 53.9 us,
// 8192 windows x 3 heads 65.9 -> 44.5.
constexpr int intdiv24_up(int64_t i0, int n_shift, int m_bits, int k_out) {
    const int64_t e0 = i0 << n_shift;
    if (m_bits - (k_out - 1) != 24 || e0 <= (int64_t)1 << (k_out - 1) || e0 > 65535) return -1;
    int j = 0;
    while (e0 >> (j + 1)) ++j;
    return m_bits - 16 - j > 0 ? m_bits - 16 - j : 0;
}

}  // namespace ivit
