// Host build of the sums that stand in for the first one or two stages of a transform on small inputs (sum_small of
// the policies in paper_2207_04604_amd/csrc/arith.hpp) against 128-bit integers: the residue, and the bound the
// stages that follow start from; the same for an encoded message (sum_encoded); and a lazy value as the multiplicand of keys (factor_key_add).  Compiled and run by tests/test_sum_small.py; exits non-zero on a violation.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define D2_DEV inline
static inline double __longlong_as_double(long long v) { double d; std::memcpy(&d, &v, 8); return d; }
static inline long long __double_as_longlong(double d) { long long v; std::memcpy(&v, &d, 8); return v; }
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
static inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return (uint64_t)(((unsigned __int128)a * b) >> 64); }

#include "../paper_2207_04604_amd/csrc/arith.hpp"
#include "../paper_2207_04604_amd/csrc/pm_growth.hpp"

typedef unsigned __int128 u128;
typedef __int128 i128;
using namespace d2;

static uint64_t state = 0x9E3779B97F4A7C15ull;
static uint64_t rnd()
{   // splitmix64
    uint64_t z = (state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static Tw split(uint64_t w, uint64_t q)
{
    const int s = 64 - __builtin_clzll(q) - 31;
    const uint64_t low = ((uint64_t)1 << s) - 1, v = (uint64_t)(((u128)w << 32) % q);
    return Tw{(w & low) | (w >> s) << 32, (v & low) | (v >> s) << 32};
}
template <class A> struct Of;
template <> struct Of<ArithP> {
    static ArithP::Mod mod(uint64_t q) { return ArithP::mod(q, pm_growth(q, false) * q); }
    static TwPm tw(uint64_t w, uint64_t q) { return pm_tw(split(w, q)); }
    static bool ok(uint64_t x, uint64_t q, int) { return (u128)x < 4 * (u128)q; }
    static i128 value(uint64_t x) { return (i128)x; }
};
template <> struct Of<ArithQ> : Of<ArithP> {
    static ArithQ::Mod mod(uint64_t q) { return ArithQ::mod(q, pm_growth(q, true) * q); }
};
template <> struct Of<ArithF> {
    static ArithF::Mod mod(uint64_t q) { return ArithF::mod(q); }
    static ArithF::Twid tw(uint64_t w, uint64_t q) { return ArithF::tw(w, q); }
    static bool ok(double x, uint64_t q, int ss) { return __builtin_fabs(x) <= 16.0 * (ss - 1) * (double)q + 32; }
    static i128 value(double x) { return (i128)x; }
};
template <> struct Of<Arith32> {
    static Arith32::Mod mod(uint64_t q) { return Arith32::mod(q); }
    static Arith32::Twid tw(uint64_t w, uint64_t q) { return Arith32::Twid{(uint32_t)w, (uint32_t)((w << 32) / q)}; }
    static bool ok(uint32_t x, uint64_t q, int) { return x < 4 * q; }
    static i128 value(uint32_t x) { return (i128)x; }
};

template <class A, int SS>
static void check(uint64_t q)
{
    const typename A::Mod md = Of<A>::mod(q);
    const uint64_t ends[] = {0, 1, q - 1, q / 2, q / 2 + 1, q - 2};
    for (int rep = 0; rep < 40000; ++rep) {
        int32_t s[SS];
        typename A::Small c[SS];
        i128 want = s[0] = rep % 3 == 0 ? (rep & 4 ? 32 : -32) : (int)(rnd() % 65) - 32;
        for (int j = 1; j < SS; ++j) {
            const uint64_t w = rep % 5 < 3 ? ends[rnd() % 6] : rnd() % q;
            const bool neg = rnd() & 1;
            s[j] = rep % 3 < 2 ? (rnd() & 1 ? 32 : -32) : (int)(rnd() % 65) - 32;
            c[j] = A::small(Of<A>::tw(w, q), neg, md);
            want += (neg ? -(i128)w : (i128)w) * s[j];
        }
        const typename A::elem x = A::sum_small(s, c, md);
        if ((Of<A>::value(x) - want) % (i128)q != 0 || !Of<A>::ok(x, q, SS)) {
            std::printf("FAILED: kind %d, SS = %d, q = %llu\n", A::KIND, SS, (unsigned long long)q);
            std::exit(1);
        }
    }
}

// +-lam m0 + e0 +- I (+-lam m1 + e1) with any I
template <class A>
static void check_encoded(uint64_t q, uint64_t most_times_q)
{
    const typename A::Mod md = Of<A>::mod(q);
    const uint64_t ends[] = {0, 1, q - 1, q / 2, q / 2 + 1, q - 2};
    const uint32_t ms[] = {0, 1, (1u << 30) - 1, (1u << 30) - 2, 65536, 12288};
    for (int rep = 0; rep < 40000; ++rep) {
        const uint64_t w = rep % 5 < 3 ? ends[rnd() % 6] : rnd() % q, lam = rep % 4 < 2 ? ends[rnd() % 6] : rnd() % q;
        const uint64_t lam_i = (uint64_t)((u128)w * lam % q);
        const bool neg = rnd() & 1, minus = rnd() & 1;          // -I, -lam
        const uint32_t cap = (uint32_t)(q < 1u << 30 ? q - 1 : (1u << 30) - 1);
        uint32_t m[2];
        int32_t e[2];
        for (int j = 0; j < 2; ++j) {
            m[j] = rep % 3 ? ms[rnd() % 6] : (uint32_t)(rnd() >> 34);
            if (m[j] > cap) m[j] = cap;
            e[j] = rep % 2 ? (rnd() & 1 ? 32 : -32) : (int)(rnd() % 65) - 32;
        }
        typename A::Small c[2];
        c[1] = A::small(Of<A>::tw(w, q), neg, md);
        const typename A::elem x = A::sum_encoded(m, e, Of<A>::tw(lam, q), Of<A>::tw(lam_i, q), minus, minus != neg, c, md);
        const i128 sign = minus ? -1 : 1, second = sign * (i128)((u128)lam_i * m[1] % q) + (i128)w * e[1];
        const i128 v = Of<A>::value(x), want = sign * (i128)((u128)lam * m[0] % q) + e[0] + (neg ? -second : second);
        if ((v - want) % (i128)q != 0 || (v < 0 ? -v : v) >= (i128)most_times_q * q) {
            std::printf("FAILED: encoded, kind %d, q = %llu\n", A::KIND, (unsigned long long)q);
            std::exit(1);
        }
    }
}

template <class A>
static void check_factor(uint64_t q, bool wide)
{
    const uint64_t G = pm_growth(q, wide), top = wide ? q + 2 * G * q + q / 4 : 64 * q + 16 * G * q;
    const ModPm md = Of<A>::mod(q);
    const uint64_t us[] = {top, top - 1, q, q - 1, 0, top & ~0xffffffffull, ((top >> 32) << 32) - 1};
    const uint64_t ks[] = {q - 1, q - 2, 0, 1, 0xffffffffull, q & ~0xffffffffull, q / 2};
    for (int rep = 0; rep < 40000; ++rep) {
        const uint64_t u = rep % 3 ? us[rnd() % 7] : (uint64_t)(((u128)rnd() * top) >> 64);
        const uint64_t k = rep % 4 ? ks[rnd() % 7] : rnd() % q, x = rep % 2 ? (wide ? top : 64 * q + 8 * G * q) : rnd() % q;
        const uint64_t r = A::factor_key_add(A::factor(u, md), A::key_of(k, 0), x, md);
        const uint64_t want = (uint64_t)(((u128)(u % q) * k + x) % q);
        if (r % q != want || A::canon_acc(r, md) != want || (u128)r > (u128)x + 2 * G * (u128)q) {
            std::printf("FAILED: factor, kind %d, q = %llu\n", A::KIND, (unsigned long long)q);
            std::exit(1);
        }
    }
}

int main(int argc, char **argv)
{
    for (int i = 1; i < argc; ++i) {
        const uint64_t q = std::strtoull(argv[i], nullptr, 10);
        int n = 0;
        if (pm_growth(q, false)) { check<ArithP, 2>(q); check<ArithP, 4>(q); check_factor<ArithP>(q, false); check_encoded<ArithP>(q, 2 * pm_growth(q, false)); ++n; }
        if (pm_growth(q, true)) { check<ArithQ, 2>(q); check<ArithQ, 4>(q); check_factor<ArithQ>(q, true); check_encoded<ArithQ>(q, 2 * pm_growth(q, true)); ++n; }
        if (q < 1ull << 44) { check<ArithF, 2>(q); check<ArithF, 4>(q); check_encoded<ArithF>(q, 18); ++n; }
        if (q < 1ull << 30) { check<Arith32, 2>(q); check<Arith32, 4>(q); check_encoded<Arith32>(q, 5); ++n; }
        std::printf("%d ", n);
    }
    return 0;
}
