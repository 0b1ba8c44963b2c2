// Host side of ArithP and ArithQ (arith.hpp): which moduli fit them, and the bound G of their products.
#pragma once
#include <cmath>
#include <stdint.h>

namespace d2 {

// G of ArithP (`wide` false) or ArithQ (`wide`) for the modulus q = 2^b - c: the smallest number such that a product
// of any value the policy lets into a butterfly is below G q (arith.hpp), or 0 if the modulus does not fit.
inline uint32_t pm_growth(uint64_t q, bool wide)
{
    const int b = 64 - __builtin_clzll(q);
    if (b < 34 || b > 61) return 0;
    const uint64_t c = ((uint64_t)1 << b) - q;
    if (c >> 31) return 0;                                   // 2c is a 32-bit factor
    const long double one = std::ldexp(1.0L, b), gamma = std::ldexp((long double)c, 32) / one;
    if (std::ldexp((long double)c, 64 - b) >= one) return 0; // one correction step has to be enough (pm_canon)
    for (uint32_t G = wide ? 6 : 8; G <= 4096; ++G) {
        // the largest value between two butterflies; a folded value is at most (1 + slack) q
        const long double slack = (long double)c * (3 + 2 * G) / one;
        const long double top = (wide ? 1 + slack + 2 * G : 64 + 16.0L * G) * q;
        if ((wide && slack > 0.25L) || top >= std::ldexp(1.0L, wide ? 64 : 63)) return 0;
        const long double product = ((2 + gamma) * (1 + top / std::ldexp(1.0L, 64)) + 2) * one + std::ldexp(1.0L, 33);
        if (product <= (long double)G * q) return G;
    }
    return 0;
}

}  // namespace d2
