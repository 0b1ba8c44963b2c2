// Every limb of a polynomial belongs to exactly one part of a split launch, whatever the sizes, and no split that was passed over
// is better than the one chosen.
#include <chrono>
#include <cstdio>
#include <initializer_list>

#include "../paper_2207_04604_amd/csrc/limb_split.hpp"

// Where what is read lies under what is written: only limb on limb may the parts of a polynomial go to several workgroups.
static bool crossing_known()
{
    static uint64_t w[64];
    const size_t N = 4, LN = 12;
    const uint64_t *at = w + 16;
    return !d2::crosses(w, 16, at, 4, 0) && d2::crosses(w, 17, at, 4, 0) && d2::crosses(w + 19, 24, at, 4, 0) && !d2::crosses(w + 20, 24, at, 4, 0) &&
           d2::crosses(w + 16, 24, at, 4, 0) && !d2::crosses(w + 16, LN, at, 2 * LN, LN) && !d2::crosses(w + 16 + LN, LN, at, 2 * LN, LN) &&
           d2::crosses(w + 16 + LN - N, LN, at, 2 * LN, LN) && d2::crosses(w + 14, 2 * LN, at, 2 * LN, LN) &&
           !d2::crosses(w + 4, LN, at, 2 * LN, LN) && d2::crosses(w + 6, LN, at, 2 * LN, LN);
}

int main()
{
    if (!crossing_known()) return std::printf("crosses\n"), 1;
    long splits = 0, uneven = 0, whole = 0;
    for (uint32_t L = 1; L <= 16; ++L)
        for (uint64_t n : {1ull, 2ull, 31ull, 33ull, 64ull, 85ull, 127ull, 128ull, 153ull, 200ull, 255ull, 256ull, 257ull, 300ull, 700ull, 1025ull, 2048ull,
                           2049ull, 70000ull, 0x7fffffffull * 880})
            for (uint32_t resident : {1u, 2u, 4u, 8u})
                for (float fixed : {0.5f, 1.2f, 2.4f}) {
                    const d2::LimbSplit s = d2::split_limbs(L, n, resident, fixed);
                    const uint32_t head = s.word & 0xffffu, rest = s.word >> 16;
                    int seen[16] = {};
                    for (uint32_t z = 0; z < s.parts; ++z) {        // limb_range in kernels.hpp
                        const uint32_t first = z ? head + (z - 1) * rest : 0;
                        uint32_t end = first + (z ? rest : head);
                        end = end < L ? end : L;
                        if (first >= end) return std::printf("empty part: L %u n %llu\n", L, (unsigned long long)n), 1;
                        for (uint32_t i = first; i < end; ++i) ++seen[i];
                    }
                    for (uint32_t i = 0; i < L; ++i)
                        if (seen[i] != 1) return std::printf("limb %u: L %u n %llu\n", i, L, (unsigned long long)n), 1;
                    if (L > 1 && n <= 4 * 256 * (uint64_t)(resident < 2 ? resident : 2)) {
                        const float alone = resident >= 8 ? 3.0f : resident >= 4 ? 2.2f : resident >= 2 ? 1.4f : 1.0f;
                        float least = d2::split_time(L, (uint32_t)n, L, L, resident, alone, fixed) / 1.05f;
                        for (uint32_t r = 1; r < L; ++r)
                            for (uint32_t h : {r, L - r}) {
                                const float t = h < r ? least : d2::split_time(L, (uint32_t)n, h, r, resident, alone, fixed);
                                least = t < least ? t : least;
                            }
                        if (s.parts > 1 && d2::split_time(L, (uint32_t)n, head, rest, resident, alone, fixed) != least)
                            return std::printf("not the best: L %u n %llu\n", L, (unsigned long long)n), 1;
                        if (s.parts == 1 && d2::split_time(L, (uint32_t)n, L, L, resident, alone, fixed) / 1.05f != least)
                            return std::printf("better in parts: L %u n %llu\n", L, (unsigned long long)n), 1;
                    }
                    if (s.parts == 1) ++whole;
                    else ++splits;
                    if (s.parts > 1 && head != rest) ++uneven;
                }
    // host time in front of a launch, the worst of its sizes (least of several runs: the machine may be busy)
    double worst = 0;
    for (uint32_t L : {4u, 8u, 16u})
        for (uint32_t n : {40u, 153u, 500u, 1024u, 1600u, 2048u})
            for (uint32_t resident : {1u, 2u, 8u}) {
                double best = 1e9;
                for (int run = 0; run < 20; ++run) {
                    const auto t0 = std::chrono::steady_clock::now();
                    for (int i = 0; i < 10; ++i) {
                        volatile uint32_t word = d2::split_limbs(L, n, resident, 0.5f).word;
                        (void)word;
                    }
                    const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 10;
                    best = us < best ? us : best;
                }
                worst = best > worst ? best : worst;
            }
    std::printf("%ld %ld %ld %.2f\n", whole, splits, uneven, worst);
    return 0;
}
