// How many workgroups share the limbs of one polynomial, for launches that leave compute units idle (host code).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace d2 {

// A polynomial that is read, `in`, lies in whole or in part where `out` is written, other than limb on limb (`LN` words to a polynomial of
// all limbs; 0: `in` has none): its workgroup may read before it writes, but not while another writes.  Of several ciphertexts this
// never was defined, as each has its workgroup.
inline bool crosses(const void *out, size_t out_words, const void *in, size_t in_words, size_t LN)
{
    const uintptr_t o = (uintptr_t)out, i = (uintptr_t)in;
    if (o >= i + 8 * in_words || i >= o + 8 * out_words) return false;
    return !LN || (o > i ? o - i : i - o) % (8 * LN) != 0;
}

constexpr uint32_t SE_UNITS = 8, SHADER_ENGINES = 32;     // 256 compute units

struct LimbSplit {
    uint32_t parts;         // gridDim.z
    uint32_t word;          // limbs of part 0 | limbs of each further part << 16 (limb_range)
};

// Time of a launch of `n` polynomials in parts, in units of one limb's work on a compute unit that has one workgroup.
// Workgroups go to the 32 shader engines in turn, whatever these have left to do, and there to 8 compute units.  Where
// a unit holds one workgroup the next goes to the unit that is free first; where it holds several (`resident`) they are dealt
// out in turn, and `alone` says how much longer one takes by itself than its share of a full unit.
// `fixed`: what every part repeats (the samples, an encoding), in the same unit.
inline float split_time(uint32_t L, uint32_t n, uint32_t head, uint32_t rest, uint32_t resident, float alone, float fixed)
{
    float load[SE_UNITS] = {}, most[SE_UNITS] = {};
    uint32_t unit = 0, start = 0, done = 0, limbs = head;         // the first shader engine: workgroups 0, 32, 64, ...
    for (uint32_t i = 0; done < L; i += SHADER_ENGINES) {
        while (i >= start + n) {
            start += n;
            done += limbs;
            limbs = L - done < rest ? L - done : rest;
            if (done >= L) break;
        }
        if (done >= L) break;
        const float cost = (float)limbs + fixed;
        if (resident == 1) {
            unit = 0;
            for (uint32_t u = 1; u < SE_UNITS; ++u)
                if (load[u] < load[unit]) unit = u;
        }
        load[unit] += cost;
        if (cost > most[unit]) most[unit] = cost;
        if (resident > 1) unit = (unit + 1) % SE_UNITS;
    }
    float time = 0;
    for (uint32_t u = 0; u < SE_UNITS; ++u) {
        const float t = load[u] + (alone - 1) * most[u];
        if (t > time) time = t;
    }
    return time;
}

// The least that this can be: the work spread evenly over the units of the first shader engine, or the largest part by itself.  Most splits
// need not be played through (host time in front of a launch, 16 limbs 2 to 5 us, 31 without this).
inline float split_time_least(uint32_t L, uint32_t n, uint32_t head, uint32_t rest, float alone, float fixed)
{
    float work = 0;
    for (uint32_t done = 0, limbs = head, start = 0; done < L; done += limbs, start += n, limbs = L - done < rest ? L - done : rest)
        work += (float)((start + n + SHADER_ENGINES - 1) / SHADER_ENGINES - (start + SHADER_ENGINES - 1) / SHADER_ENGINES) * ((float)limbs + fixed);
    const float even = work / SE_UNITS, part = alone * ((float)head + fixed);
    return (even > part ? even : part) * 0.9999f;            // (sums in another order)
}

// The split of L limbs that takes least time by that rule, if it takes 5 % less than whole polynomials do; `n`: workgroups
// of whole polynomials.  Measured over 752 shapes (encryption, decryption, conversion and refresh shares, N = 2^10 to
// 2^14, 30 to 60 bits, 2 to 8 limbs, 4 to 1,700 indices): 1.263 times as fast as whole polynomials in the geometric mean, where
// the best split of each is 1.279; slowest 0.977 (refresh shares, N = 1024, six limbs, 700 indices, 43.1 / 44.1 us).
// Some of them, whole / split, us:
//   encryption, 54 bits, N = 8192, 4 limbs   n = 8 69.6 / 24.1 (1 + 1 + 1 + 1), 153 70.2 / 56.0 (3 + 1), 300 139 / 110 (3 + 1)
//   share       36 bits, N = 4096, 3 limbs   n = 40 11.5 / 6.3 (1 + 1 + 1), 153 11.5 / 8.8 (1 + 1 + 1)
//   refresh     54 bits, N = 2^14, 8 limbs   n = 16 168 / 49 (by ones), 50 168 / 99 (4 + 4), 153 338 / 274 (6 + 2)
// (Refresh shares as they were with masks of 1.2 limbs.)  Beyond four turns of the chip the last one matters little.
inline LimbSplit split_limbs(uint32_t L, uint64_t n, uint32_t resident, float fixed)
{
    LimbSplit best = {1, L};
    if (L < 2 || n > 4 * 256 * (uint64_t)(resident < 2 ? resident : 2)) return best;
    const float alone = resident >= 8 ? 3.0f : resident >= 4 ? 2.2f : resident >= 2 ? 1.4f : 1.0f;
    const float whole = split_time(L, (uint32_t)n, L, L, resident, alone, fixed);
    float least = whole / 1.05f;
    for (uint32_t rest = 1; rest < L; ++rest)
        for (int k = 0; k < 2; ++k) {                       // equal parts; all limbs but `rest` in the first
            const uint32_t head = k ? L - rest : rest;
            if (head < rest || (k && head == rest) || split_time_least(L, (uint32_t)n, head, rest, alone, fixed) >= least) continue;
            const float t = split_time(L, (uint32_t)n, head, rest, resident, alone, fixed);
            if (t < least) {
                least = t;
                best.parts = 1 + (L - head + rest - 1) / rest;
                best.word = head | rest << 16;
            }
        }
    return best;
}

}  // namespace d2
