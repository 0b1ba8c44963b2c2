// Host build of ArithP and ArithQ (paper_2207_04604_amd/csrc/arith.hpp, the plain-C side) against 128-bit integers:
// every operation gives its residue and stays inside its bound for inputs at the ends of their ranges, and whole
// chains of butterflies that always take the largest value there is stay inside the policy's bounds from stage to
// stage.  Moduli: 2^b - k 2N + 1 for every b a policy takes, the smallest and the largest c that fit.  Compiled and
// run by tests/test_pm_policies.py; exits non-zero on a violation.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#define D2_DEV inline
static inline double __longlong_as_double(long long v) { double d; std::memcpy(&d, &v, 8); return d; }
static inline long long __double_as_longlong(double d) { long long v; std::memcpy(&v, &d, 8); return v; }
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
static inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return (uint64_t)(((unsigned __int128)a * b) >> 64); }
// the rest of what the kernels' header names; nothing here is run by more than one thread
#define __global__
#define __shared__ static
#define __launch_bounds__(...)
static struct { uint32_t x, y; } threadIdx, blockIdx, gridDim;
static inline void __syncthreads() {}
static inline int __shfl_xor(int v, int) { return v; }
static inline int __popc(uint32_t v) { return __builtin_popcount(v); }
static inline uint32_t __brev(uint32_t v)
{
    uint32_t r = 0;
    for (int i = 0; i < 32; ++i) r |= ((v >> i) & 1u) << (31 - i);
    return r;
}

#include "../paper_2207_04604_amd/csrc/kernels.hpp"
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
#define CHECK(cond, what, q)                                                                                 \
    do {                                                                                                     \
        if (!(cond)) {                                                                                       \
            std::printf("FAILED line %d: %s, q = %llu\n", __LINE__, what, (unsigned long long)(q));          \
            std::exit(1);                                                                                    \
        }                                                                                                    \
    } while (0)

static uint64_t mod_of(i128 v, uint64_t q)
{
    const i128 r = v % (i128)q;
    return (uint64_t)(r < 0 ? r + q : r);
}
static Tw entry(uint64_t w, uint64_t q)
{
    const int s = 64 - __builtin_clzll(q) - 31;
    const uint64_t low = ((uint64_t)1 << s) - 1, v = (uint64_t)(((u128)w << 32) % q);
    return Tw{(w & low) | (w >> s) << 32, (v & low) | (v >> s) << 32};
}
static std::vector<uint64_t> values(uint64_t top, uint64_t q, int n)      // of [0, top]
{
    std::vector<uint64_t> v = {0, 1, top, top - 1, top & ~0xffffffffull, (top & ~0xffffffffull) - 1, top | 0xffffffffull};
    if (v.back() > top) v.pop_back();
    for (uint64_t f : {q - 1, q, q + 1, 2 * q - 1, 2 * q, (uint64_t)0xffffffff, (uint64_t)1 << 32})
        if (f <= top) v.push_back(f);
    for (int i = 0; i < n; ++i) v.push_back((uint64_t)(((u128)rnd() * ((u128)top + 1)) >> 64));
    return v;
}
static std::vector<uint64_t> multiplicands(uint64_t q, int n)
{
    const int s = 64 - __builtin_clzll(q) - 31;
    std::vector<uint64_t> v = {0, 1, q - 1, q - 2, q / 2, (q >> s << s) - 1, ((uint64_t)1 << s) - 1};
    for (int i = 0; i < n; ++i) v.push_back(rnd() % q);
    return v;
}

template <class A>
static void check(uint64_t q, bool wide)
{
    const uint32_t G = pm_growth(q, wide);
    if (!G) return;
    const typename A::Mod md = A::mod(q, G * q);
    const u128 limit = wide ? (u128)1 << 64 : (u128)1 << 63;
    const uint64_t top = wide ? q + 2 * (uint64_t)G * q + q / 4 : 64 * q + 16 * (uint64_t)G * q;
    CHECK((u128)top < limit || wide, "range", q);
    for (uint64_t w : multiplicands(q, 30)) {
        const TwPm tw = A::tw(entry(w, q)), ks = pm_split(w, md);
        CHECK(ks.w00 == tw.w00 && ks.w01 == tw.w01, "split of a key", q);
        for (uint64_t y : values(wide ? q + 2 * (uint64_t)G * q : top, q, 200)) {
            const uint64_t r = A::mul(y, tw, md);
            CHECK(r < (uint64_t)G * q && r % q == (uint64_t)((u128)w * y % q), "mul", q);
            const uint64_t x = (uint64_t)(((u128)rnd() * q) >> 64), ka = A::mul_key_add(y, A::key_of(w, 0), x, md);
            CHECK(ka % q == (uint64_t)(((u128)w * y + x) % q) && ka <= q + q / 4 + (uint64_t)G * q, "mul_key_add", q);
            const uint64_t r32 = A::mul_u32((uint32_t)y, tw, md);
            CHECK(r32 < (uint64_t)G * q && r32 % q == (uint64_t)((u128)w * (uint32_t)y % q), "mul_u32", q);
        }
        for (int xv = -32; xv <= 32; xv += 8)
            for (int yv = -32; yv <= 32; ++yv) {
                uint64_t x, y;
                A::ct_small(xv, yv, x, y, tw, md);
                const u128 most = wide ? (u128)(1 + G) * q : 64 * (u128)q + 33;
                CHECK(x % q == mod_of((i128)xv + (i128)w * yv, q) && y % q == mod_of((i128)xv - (i128)w * yv, q) &&
                          x < most && y < most, "ct_small", q);
            }
    }
    for (uint64_t x : values(wide ? q + 2 * (uint64_t)G * q : top, q, 20000)) CHECK(A::canon_wide(x, md) == x % q, "canon", q);
    for (int v = -32; v <= 32; ++v) CHECK(A::add_small(G * q - 1, v, md) % q == mod_of((i128)(G * q - 1) + v, q), "add_small", q);

    // Chains of forward stages: both inputs of a stage at the largest value the previous one can leave, and random
    // residues of that size; the true bound is followed with exact integers.
    for (int start = 0; start < 3; ++start)
        for (uint64_t w : multiplicands(q, 20)) {
            const TwPm tw = A::tw(entry(w, q));
            uint64_t x = start == 0 ? q - 1 : wide ? (1 + (uint64_t)G) * q : 64 * q + 32, y = start == 2 ? x - q / 3 : x;
            for (int s = start == 0 ? 0 : (wide ? 0 : 1); s < 16; ++s) {
                uint64_t a = x, b = y;
                const uint64_t rx = x % q, t = (uint64_t)((u128)w * (y % q) % q);
                A::ct(a, b, tw, md, s);
                CHECK(a % q == (rx + t) % q && b % q == (rx + q - t) % q, "ct", q);
                const u128 bound = wide ? (u128)((s & 1) ? 1 + G : 1 + 2 * G) * q + q / 4 : (u128)x + (u128)G * q;
                CHECK((start && wide && s == 0) || ((u128)a <= bound && (u128)b <= bound), "forward bound", q);
                x = a > b ? a : b;
                y = start == 1 ? x : (a > b ? b : a);
            }
        }
    // An inverse pass, slot by slot, with the folds the engine uses
    for (int stages : {1, 3, 4})
        for (int first = 0; first < 2; ++first)
            for (int rep = 0; rep < 200; ++rep) {
                const uint64_t folds = inv_folds<A>(first, stages, 16);
                const uint64_t in = first ? q - 1 : (uint64_t)A::INV_LIM / A::INV_PROD * G * q;
                uint64_t x[16], r[16];
                for (int k = 0; k < 16; ++k) {
                    x[k] = rep == 0 ? in : rep == 1 ? (k & 1 ? in : 0) : (uint64_t)(((u128)rnd() * in) >> 64);
                    r[k] = x[k] % q;
                }
                for (int i = 0; i < stages; ++i)
                    for (int k = 0; k < 16; ++k) {
                        if (k & (1 << i)) continue;
                        const uint64_t w = rep < 40 ? q - 1 : rnd() % q;
                        const TwPm tw = A::tw(entry(w, q));
                        const int j = k | (1 << i);
                        const uint64_t sum = (r[k] + r[j]) % q, d = (r[k] + q - r[j]) % q;
                        uint64_t lx = x[k], ly = x[j];
                        A::gs_last(lx, ly, tw, tw, md);
                        CHECK(lx % q == (uint64_t)((u128)w * sum % q) && ly % q == (uint64_t)((u128)w * d % q) &&
                                  lx < (uint64_t)G * q && ly < (uint64_t)G * q, "gs_last", q);
                        A::gs(x[k], x[j], tw, md, (folds >> (16 * i + k)) & 1);
                        r[k] = sum;
                        r[j] = (uint64_t)((u128)w * d % q);
                        CHECK(x[k] % q == r[k] && x[j] % q == r[j] && x[j] < (uint64_t)G * q, "gs", q);
                        CHECK((u128)x[k] <= (u128)(A::INV_LIM / A::INV_PROD) * G * q, "inverse bound", q);
                    }
            }
}

// x +- u key as the kernels store it (a share, a refresh share), x at the largest value a forward transform can leave,
// u and the key at the ends of [0, q).
template <class A, bool NEG>
static void check_store(uint64_t q, bool wide)
{
    const uint32_t G = pm_growth(q, wide);
    if (!G) return;
    typedef Engine<A, 10, 3> ENG;
    constexpr int E = ENG::E, T = ENG::T;
    const typename A::Mod md = A::mod(q, G * q);
    const uint64_t c = ((uint64_t)1 << (64 - __builtin_clzll(q))) - q;
    // wide: 1 + 2G and the excess of a folded value; narrow: a small first stage and 15 further ones
    const uint64_t most = wide ? (1 + 2 * (uint64_t)G) * q + (3 + 2 * (uint64_t)G) * c : (64 + 15 * (uint64_t)G) * q;
    std::vector<uint64_t> dst(E * T), key(E * T), src(E * T);
    const typename A::Factor none[E] = {};
    for (uint64_t x : {most, most - 1, most - (3 + 2 * (uint64_t)G) * c + 1, most - q, (uint64_t)0})
        for (uint64_t k : {(uint64_t)0, (uint64_t)1, q - 1, q / 2, rnd() % q}) {
            const uint64_t us[] = {0, 1, q - 1, q - 2, q / 2, rnd() % q, rnd() % q, rnd() % q};
            uint64_t xs[E];
            for (int i = 0; i < E; ++i) {
                xs[i] = x;
                key[i * T] = k;
                src[i * T] = us[i];
            }
            mul_add_store<ENG, SRC_CANON, NEG>(dst.data(), key.data(), key.data(), src.data(), none, xs, 0, md, q);
            for (int i = 0; i < E; ++i) {
                const uint64_t p = (uint64_t)((u128)us[i] * k % q);
                CHECK(dst[i * T] == (x % q + (NEG ? q - p : p)) % q, NEG ? "x - u key" : "x + u key", q);
            }
        }
}

int main(int argc, char **argv)
{
    int narrow = 0, wide = 0;
    for (int i = 1; i < argc; ++i) {
        const uint64_t q = std::strtoull(argv[i], nullptr, 10);
        narrow += pm_growth(q, false) != 0;
        wide += pm_growth(q, true) != 0;
        check<ArithP>(q, false);
        check<ArithQ>(q, true);
        check_store<ArithP, false>(q, false);
        check_store<ArithP, true>(q, false);
        check_store<ArithQ, false>(q, true);
        check_store<ArithQ, true>(q, true);
    }
    std::printf("%d moduli, %d fit ArithP, %d fit ArithQ\n", argc - 1, narrow, wide);
    return 0;
}
