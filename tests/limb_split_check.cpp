// Every limb of a polynomial belongs to exactly one part of a split launch, whatever the sizes.
#include <cstdio>
#include <initializer_list>

#include "../paper_2207_04604_amd/csrc/limb_split.hpp"

int main()
{
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
                    if (s.parts == 1) ++whole;
                    else ++splits;
                    if (s.parts > 1 && head != rest) ++uneven;
                }
    std::printf("%ld %ld %ld\n", whole, splits, uneven);
    return 0;
}
