// Modular arithmetic back-ends ("policies") for the transform engine on gfx950.
//
// On CDNA4 v_mad_u64_u32, v_mul_lo/hi_u32, v_lshl_add_u64 and v_fma_f64 all issue at full
// rate, so the cost of a butterfly is its instruction count.  Six formulations, chosen
// per context from the size and the form of the moduli:
//
//   ArithF  (moduli < 2^44)  residues as signed doubles.  w*y mod q from an error-free
//           product (mul + fma), one rounded quotient and one fma: 6 instructions, result
//           in about (-q/2, q/2); butterflies add and subtract without any correction.
//   ArithS  (other moduli < 2^55)  64-bit integers, Shoup quotient ws = floor(w 2^63 / q).  The
//           quotient estimate drops the low x low partial product (error <= 2), so the
//           product lands in [0, 4q); values grow by at most 4q per forward stage and are
//           never corrected inside a forward transform (65 q < 2^62).
//   ArithB  (other moduli < 2^61)  64-bit integers, exact 63-bit Shoup quotient, Harvey's lazy
//           butterflies: forward values in [0, 4q), inverse values in [0, 2q).
//   ArithP  (moduli in [2^44, 2^55) just below a power of two) and
//   ArithQ  (the same up to 2^60): q = 2^b - c with a small c.  Multiplicands are kept as w and
//           w 2^32 mod q, both split at bit b - 31, so that a product needs no quotient: six
//           multiply-adds give w*y + u directly (see pm_mul_add).  9 instructions per butterfly
//           instead of 15 (ArithS) and 10.5 instead of 21 (ArithB).
//   Arith32 (moduli < 2^30)  32-bit residues (one register and one 4-byte LDS word per
//           coefficient), 32-bit Shoup quotient ws = floor(w 2^32 / q), Harvey's lazy butterflies
//           in 8 instructions.  Used for whole contexts whose primes are below 2^30 and, in every
//           context, for the transforms modulo the plaintext modulus t.
//
// Table entries (twiddles, per-modulus constants) are {w, floor(w 2^63 / q)} for ArithS and ArithB,
// {bits of the double w, unused} for ArithF, the two split multiplicands for ArithP and ArithQ.
// Prepared keys cross the library boundary as values plus 64-bit quotients floor(v 2^64 / q); ArithS and
// ArithB shift those right by one, ArithF, ArithP and ArithQ read the value only.
#pragma once
#include <stdint.h>

#ifndef D2_DEV
#define D2_DEV __device__ __forceinline__
#endif

#pragma clang fp contract(off)

namespace d2 {

struct Tw {          // 16-byte table entry: a fixed multiplicand and its companion word
    uint64_t w;
    uint64_t ws;
};

D2_DEV uint32_t lo32(uint64_t v) { return (uint32_t)v; }
D2_DEV uint32_t hi32(uint64_t v) { return (uint32_t)(v >> 32); }
D2_DEV uint64_t mul32(uint32_t a, uint32_t b) { return (uint64_t)a * b; }

// The hot sequences are pinned with inline assembly on the device: the compiler's own
// selection for the same C spends about 40 % more VALU slots (zero-extension moves, a compare
// in front of every conditional subtraction, 32-bit multiplies split off the 64-bit
// multiply-adds).  The plain C next to each block states what it computes and is what a
// host build of this header runs.
#if defined(__HIP_DEVICE_COMPILE__)
#define D2_GCN_ASM 1
#else
#define D2_GCN_ASM 0
#endif

// x >= m ? x - m : x   (unsigned): subtract, then select on the borrow
D2_DEV uint64_t csub(uint64_t x, uint64_t m)
{
#if D2_GCN_ASM
    uint32_t dlo, dhi;
    const uint32_t xlo = lo32(x), xhi = hi32(x), mlo = lo32(m), mhi = hi32(m);
    asm("v_sub_co_u32 %0, vcc, %2, %4\n\t"
        "v_subb_co_u32 %1, vcc, %3, %5, vcc\n\t"
        "v_cndmask_b32 %0, %0, %2, vcc\n\t"
        "v_cndmask_b32 %1, %1, %3, vcc"
        : "=&v"(dlo), "=&v"(dhi)
        : "v"(xlo), "v"(xhi), "v"(mlo), "v"(mhi)
        : "vcc");
    return ((uint64_t)dhi << 32) | dlo;
#else
    uint64_t d = x - m;
    return x < m ? x : d;
#endif
}

// ---------------------------------------------------------------------------------------
// Global memory access.
//   Per-lane: raw buffer instructions -- a wave-uniform base (descriptor in SGPRs) plus one 32-bit
//   per-lane byte offset and a uniform offset.  Plain 64-bit addressing would hold a VGPR pair per
//   array and slot, and generic pointers become flat instructions, whose completion is counted
//   together with LDS traffic.  The ranges are < 4 GB from the base.
//   Wave-uniform table reads: through the constant address space, which the compiler turns into
//   scalar loads (results in SGPRs) when it can see that the offset is uniform.
// ---------------------------------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct U128 {
    uint64_t lo, hi;
};
D2_DEV uint64_t ld64(const void *base, uint32_t lane_off, uint32_t slot_off)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0xffffffff, 0x00020000);
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, slot_off, 0);
    return ((uint64_t)v.y << 32) | v.x;
#else
    return *(const uint64_t *)((const char *)base + lane_off + slot_off);
#endif
}
D2_DEV U128 ld128(const void *base, uint32_t lane_off, uint32_t slot_off)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0xffffffff, 0x00020000);
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, slot_off, 0);
    return U128{((uint64_t)v.y << 32) | v.x, ((uint64_t)v.w << 32) | v.z};
#else
    const uint64_t *p = (const uint64_t *)((const char *)base + lane_off + slot_off);
    return U128{p[0], p[1]};
#endif
}
D2_DEV void st64(void *base, uint32_t lane_off, uint32_t slot_off, uint64_t val)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xffffffff, 0x00020000);
    u32x2 v;
    v.x = (uint32_t)val;
    v.y = (uint32_t)(val >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(v, r, lane_off, slot_off, 0);
#else
    *(uint64_t *)((char *)base + lane_off + slot_off) = val;
#endif
}
// The same load marked non-temporal (streaming): for data read exactly once.
D2_DEV uint64_t ld64_stream(const void *base, uint32_t lane_off, uint32_t slot_off)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0xffffffff, 0x00020000);
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, slot_off, 2 /* nt */);
    return ((uint64_t)v.y << 32) | v.x;
#else
    return *(const uint64_t *)((const char *)base + lane_off + slot_off);
#endif
}
// The same for pairs of words.
D2_DEV U128 ld128_stream(const void *base, uint32_t lane_off, uint32_t slot_off)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0xffffffff, 0x00020000);
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, slot_off, 2 /* nt */);
    return U128{((uint64_t)v.y << 32) | v.x, ((uint64_t)v.w << 32) | v.z};
#else
    return ld128(base, lane_off, slot_off);
#endif
}
// A store of more than 8 bytes reads its registers after it has issued, and the compiler keeps the next two instructions from overwriting
// them; not where the store has a scalar offset, which is taken to be exempt, but is not on gfx950 (a store followed at once by such an
// instruction wrote the new values for lanes 12 to 15 of every 16).  So the slot's offset goes into the lane's.
D2_DEV void st128_stream(void *base, uint32_t lane_off, uint32_t slot_off, U128 val)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xffffffff, 0x00020000);
    u32x4 v;
    v.x = (uint32_t)val.lo;
    v.y = (uint32_t)(val.lo >> 32);
    v.z = (uint32_t)val.hi;
    v.w = (uint32_t)(val.hi >> 32);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off + slot_off, 0, 2 /* nt */);
#else
    uint64_t *p = (uint64_t *)((char *)base + lane_off + slot_off);
    p[0] = val.lo;
    p[1] = val.hi;
#endif
}
// The same store marked non-temporal (streaming): for data the kernel never reads again, so that it
// does not displace what the kernel does re-read (parked words, keys, twiddles) from the caches.
D2_DEV void st64_stream(void *base, uint32_t lane_off, uint32_t slot_off, uint64_t val)
{
#if D2_GCN_ASM
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xffffffff, 0x00020000);
    u32x2 v;
    v.x = (uint32_t)val;
    v.y = (uint32_t)(val >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(v, r, lane_off, slot_off, 2 /* nt */);
#else
    *(uint64_t *)((char *)base + lane_off + slot_off) = val;
#endif
}
D2_DEV uint64_t const_ld64(const void *base, uint32_t byte_off)
{
#if D2_GCN_ASM
    typedef const __attribute__((address_space(4))) uint64_t *cptr;
    return *(cptr)((uintptr_t)base + byte_off);
#else
    return *(const uint64_t *)((const char *)base + byte_off);
#endif
}
// a value that is the same in every lane of the wavefront, moved to a scalar register
D2_DEV uint32_t wave_uniform(uint32_t v)
{
#if D2_GCN_ASM
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#else
    return v;
#endif
}

// floor(w * 2^64 / q) for w < q < 2^61 by binary long division (set-up paths only).
D2_DEV uint64_t shoup_quotient(uint64_t w, uint64_t q)
{
    uint64_t rem = w, quo = 0;
    for (int i = 0; i < 64; ++i) {
        rem <<= 1;
        quo <<= 1;
        if (rem >= q) { rem -= q; quo |= 1; }
    }
    return quo;
}

// ---------------------------------------------------------------------------------------
// Shared pieces of the two integer policies.
// ---------------------------------------------------------------------------------------
struct ModU {
    uint64_t q;     // modulus
    uint64_t nq;    // 2^64 - q
    uint64_t one_s; // floor(2^63 / q): Shoup quotient of the multiplicand 1
};

struct TwU {        // multiplicand and its 63-bit Shoup quotient
    uint64_t w, ws;
};

// w*y - qh*q mod 2^64, written as w*y + qh*(2^64 - q) so that every term is added:
// a chain of four 64-bit multiply-adds for the cross terms (only its low word matters; it is
// shifted up by 32), then two more for the low x low terms on top of it.
// SC: w sits in scalar registers (a multiplicand shared by the whole wavefront).  2^64 - q is the same
// for the whole workgroup and always comes from scalar registers (no instruction here reads both it
// and w, so the one-scalar-operand limit holds).
#define D2_SHOUP_TAIL_ASM(WC)                                                                      \
    asm("v_mad_u64_u32 %1, vcc, %4, %3, 0\n\t"                                                     \
        "v_mad_u64_u32 %1, vcc, %5, %2, %1\n\t"                                                    \
        "v_mad_u64_u32 %1, vcc, %6, %9, %1\n\t"                                                    \
        "v_mad_u64_u32 %1, vcc, %7, %8, %1\n\t"                                                    \
        "v_lshlrev_b64 %1, 32, %1\n\t"                                                             \
        "v_mad_u64_u32 %0, vcc, %4, %2, %1\n\t"                                                    \
        "v_mad_u64_u32 %0, vcc, %6, %8, %0"                                                        \
        : "=&v"(acc), "=&v"(cross)                                                                 \
        : "v"(y0), "v"(y1), WC(w0), WC(w1), "v"(h0), "v"(h1), "s"(n0), "s"(n1)                     \
        : "vcc")
template <bool SC = false>
D2_DEV uint64_t shoup_tail(uint64_t y, uint64_t w, uint64_t qh, uint64_t nq)
{
    const uint32_t y0 = lo32(y), y1 = hi32(y), w0 = lo32(w), w1 = hi32(w);
    const uint32_t h0 = lo32(qh), h1 = hi32(qh), n0 = lo32(nq), n1 = hi32(nq);
#if D2_GCN_ASM
    uint64_t acc, cross;
    if constexpr (SC) D2_SHOUP_TAIL_ASM("s");
    else D2_SHOUP_TAIL_ASM("v");
    return acc;
#else
    uint64_t acc = mul32(w0, y0);
    acc = mul32(h0, n0) + acc;
    const uint32_t cross = w0 * y1 + w1 * y0 + h0 * n1 + h1 * n0;
    return acc + ((uint64_t)cross << 32);
#endif
}

// u + (w*y - qh*q) mod 2^64: the addend rides on the multiply-add chain of the low x low terms, and the
// cross terms, of which only the low word matters, are added to the high word at the end: one
// instruction less than shoup_tail followed by a 64-bit addition, and two independent chains.
#define D2_SHOUP_TAIL_ADD_ASM(WC)                                                                  \
    asm("v_mad_u64_u32 %1, vcc, %4, %3, 0\n\t"                                                     \
        "v_mad_u64_u32 %0, vcc, %4, %2, %10\n\t"                                                   \
        "v_mad_u64_u32 %1, vcc, %5, %2, %1\n\t"                                                    \
        "v_mad_u64_u32 %0, vcc, %6, %8, %0\n\t"                                                    \
        "v_mad_u64_u32 %1, vcc, %6, %9, %1\n\t"                                                    \
        "v_mad_u64_u32 %1, vcc, %7, %8, %1"                                                        \
        : "=&v"(acc), "=&v"(cross)                                                                 \
        : "v"(y0), "v"(y1), WC(w0), WC(w1), "v"(h0), "v"(h1), "s"(n0), "s"(n1), "v"(u)             \
        : "vcc")
template <bool SC = false>
D2_DEV uint64_t shoup_tail_add(uint64_t y, uint64_t w, uint64_t qh, uint64_t nq, uint64_t u)
{
    const uint32_t y0 = lo32(y), y1 = hi32(y), w0 = lo32(w), w1 = hi32(w);
    const uint32_t h0 = lo32(qh), h1 = hi32(qh), n0 = lo32(nq), n1 = hi32(nq);
#if D2_GCN_ASM
    uint64_t acc, cross;
    if constexpr (SC) D2_SHOUP_TAIL_ADD_ASM("s");
    else D2_SHOUP_TAIL_ADD_ASM("v");
    // one 32-bit addition on the high word (written out: as C it comes back as a move plus a 64-bit add)
    uint32_t top = hi32(acc);
    const uint32_t cl = lo32(cross);
    asm("v_add_u32 %0, %0, %1" : "+v"(top) : "v"(cl));
    return ((uint64_t)top << 32) | lo32(acc);
#else
    uint64_t acc = mul32(w0, y0) + u;
    acc = mul32(h0, n0) + acc;
    const uint32_t cross = w0 * y1 + w1 * y0 + h0 * n1 + h1 * n0;
    return acc + ((uint64_t)cross << 32);
#endif
}

// y*1 - qh*q mod 2^64 (reduction of y itself)
D2_DEV uint64_t shoup_tail_one(uint64_t y, uint64_t qh, uint64_t nq)
{
    const uint32_t h0 = lo32(qh), h1 = hi32(qh), n0 = lo32(nq), n1 = hi32(nq);
    uint64_t acc = mul32(h0, n0) + y;
    const uint32_t cross = h0 * n1 + h1 * n0;
    return acc + ((uint64_t)cross << 32);
}

// floor(ws*y / 2^63) up to an error of 2 (too small): drops the low x low partial product.
// Needs ws < 2^63 and y < 2^63 (then the middle sum cannot overflow).
#define D2_QHAT_APPROX_ASM(WC)                                                                     \
    asm("v_mad_u64_u32 %0, vcc, %5, %2, 0\n\t"                                                     \
        "v_mad_u64_u32 %1, vcc, %5, %3, 0\n\t"                                                     \
        "v_mad_u64_u32 %0, vcc, %4, %3, %0\n\t"                                                    \
        "v_lshrrev_b64 %0, 31, %0\n\t"                                                             \
        "v_lshl_add_u64 %0, %1, 1, %0"                                                             \
        : "=&v"(mid), "=&v"(top)                                                                   \
        : "v"(y0), "v"(y1), WC(s0), WC(s1)                                                         \
        : "vcc")
template <bool SC = false>
D2_DEV uint64_t qhat_approx(uint64_t y, uint64_t ws)
{
    const uint32_t y0 = lo32(y), y1 = hi32(y), s0 = lo32(ws), s1 = hi32(ws);
#if D2_GCN_ASM
    uint64_t mid, top;
    if constexpr (SC) D2_QHAT_APPROX_ASM("s");
    else D2_QHAT_APPROX_ASM("v");
    return mid;
#else
    uint64_t mid = mul32(s1, y0);
    mid = mul32(s0, y1) + mid;
    const uint64_t top = mul32(s1, y1);
    return (top << 1) + (mid >> 31);
#endif
}

// floor(ws*y / 2^63) exactly, for ws < 2^63 and y < 2^63.
#define D2_QHAT_EXACT_ASM(WC)                                                                      \
    asm("v_mad_u64_u32 %0, vcc, %4, %2, 0\n\t"                                                     \
        "v_mad_u64_u32 %1, vcc, %5, %3, 0\n\t"                                                     \
        "v_lshrrev_b64 %0, 32, %0\n\t"                                                             \
        "v_mad_u64_u32 %0, vcc, %5, %2, %0\n\t"                                                    \
        "v_mad_u64_u32 %0, vcc, %4, %3, %0\n\t"                                                    \
        "v_lshrrev_b64 %0, 31, %0\n\t"                                                             \
        "v_lshl_add_u64 %0, %1, 1, %0"                                                             \
        : "=&v"(mid), "=&v"(top)                                                                   \
        : "v"(y0), "v"(y1), WC(s0), WC(s1)                                                         \
        : "vcc")
template <bool SC = false>
D2_DEV uint64_t qhat_exact(uint64_t y, uint64_t ws)
{
    const uint32_t y0 = lo32(y), y1 = hi32(y), s0 = lo32(ws), s1 = hi32(ws);
#if D2_GCN_ASM
    uint64_t mid, top;
    if constexpr (SC) D2_QHAT_EXACT_ASM("s");
    else D2_QHAT_EXACT_ASM("v");
    return mid;
#else
    uint64_t mid = mul32(s1, y0) + (uint64_t)__umulhi(s0, y0);
    mid = mul32(s0, y1) + mid;
    const uint64_t top = mul32(s1, y1);
    return (top << 1) + (mid >> 31);
#endif
}

// ---------------------------------------------------------------------------------------
// ArithS: moduli < 2^55, lazy products in [0, 4q).
// ---------------------------------------------------------------------------------------
struct ArithS {
    typedef uint64_t elem;
    typedef uint64_t word;          // LDS word of an exchange
    typedef ModU Mod;
    typedef TwU Twid;
    static constexpr int KIND = 1, INV_LIM = 0, INV_PROD = 0;

    D2_DEV static Mod mod(uint64_t q) { return Mod{q, 0 - q, 0}; }
    D2_DEV static Mod mod(uint64_t q, uint64_t one_s63) { return Mod{q, 0 - q, one_s63}; }
    D2_DEV static Twid tw(const Tw &t) { return Twid{t.w, t.ws}; }
    D2_DEV static Twid tw(uint64_t w, uint64_t ws64) { return Twid{w, ws64 >> 1}; }
    // element of a prepared key: values at v, 64-bit quotients at vs
    typedef Twid Key;
    D2_DEV static Key key_of(uint64_t v, uint64_t vs) { return tw(v, vs); }
    D2_DEV static Key key(const uint64_t *v, const uint64_t *vs, uint32_t lane_off, uint32_t slot_off)
    {
        return tw(ld64(v, lane_off, slot_off), ld64(vs, lane_off, slot_off));
    }
    // a value that several keys multiply
    typedef elem Factor;
    D2_DEV static Factor factor(elem u, const Mod &) { return u; }
    D2_DEV static elem factor_key_add(const Factor &u, const Key &k, elem x, const Mod &m) { return mul_key_add(u, k, x, m); }
    static constexpr bool SUM_SMALL = false;
    // table entry i: per-lane index / wave-uniform index (scalar registers, see mul<true>)
    static constexpr bool SCALAR_TW = true;
    D2_DEV static Twid load_v(const Tw *table, uint32_t i)
    {
        const U128 e = ld128(table, 16u * i, 0);
        return Twid{e.lo, e.hi};
    }
    D2_DEV static Twid load_u(const Tw *table, uint32_t i)
    {
        return Twid{const_ld64(table, 16u * i), const_ld64(table, 16u * i + 8u)};
    }

    // w*y mod q in [0, 4q), for y < 2^62.
    template <bool SC = false>
    D2_DEV static elem mul(elem y, const Twid &w, const Mod &m)
    {
        return shoup_tail<SC>(y, w.w, qhat_approx<SC>(y, w.ws), m.nq);
    }
    // w*y mod q in [0, 4q) for a 32-bit y (a plaintext coefficient): with y's high word zero the
    // quotient estimate is one partial product (s1 y >> 31 < 2^32, at most 2 too small as in mul) and the
    // tail loses its y1 and h1 terms: 7 instructions instead of 12.
    D2_DEV static elem mul_u32(uint32_t y, const Twid &w, const Mod &m)
    {
        const uint32_t h = (uint32_t)(mul32(hi32(w.ws), y) >> 31);
        const uint64_t acc = mul32(lo32(w.w), y) + mul32(h, lo32(m.nq));
        const uint32_t cross = hi32(w.w) * y + h * hi32(m.nq);
        return acc + ((uint64_t)cross << 32);
    }
    // sums of canonical words (at most 65 of them), left unreduced until sum_end
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t) { return a + b; }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &m) { return canon_wide(s, m); }
    D2_DEV static elem from_small(int32_t v, const Mod &m)
    {
        return v >= 0 ? (uint64_t)v : m.q - (uint64_t)(uint32_t)(-v);
    }
    D2_DEV static elem from_canon(uint64_t v, const Mod &) { return v; }
    D2_DEV static elem add(elem a, elem b) { return a + b; }
    // u * key + x, lazy (x: a forward output); a sum of that kind as the x of another one
    D2_DEV static elem mul_key_add(elem u, const Key &k, elem x, const Mod &m) { return add(mul(u, k, m), x); }
    D2_DEV static elem renorm(elem x, const Mod &m) { return from_canon(canon_acc(x, m), m); }
    // minus a product
    D2_DEV static elem neg(elem x, const Mod &m) { return 4 * m.q - x; }
    // x + v for a small signed v (|v| <= 32), as a forward input: q is added instead of mapping v into
    // [0, q) first (the forward range has room for it)
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &m) { return x + (m.q + (uint64_t)(int64_t)v); }

    // forward: no correction; each stage adds at most 4q to the bound.
    // x' = u + t comes out of the multiply-add chain itself, y' = u + 4q - t = (2u + 4q) - x'.
    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int = 0)
    {
        const elem u = x;
        x = shoup_tail_add<SC>(y, w.w, qhat_approx<SC>(y, w.ws), m.nq, u);
        y = (2 * u + 4 * m.q) - x;
    }
    // First stage on small signed inputs (|xv|, |yv| <= 32): w*yv is an exact 64-bit product (|w yv| < 32q
    // < 2^60), so nothing is reduced: x' = (xv + 32q) + w yv, y' = (xv + 32q) - w yv, both in (0, 64q + 32).
    // The forward bound becomes 64q + 4q per later stage: 64q + 52q + one lazy product < 128q <= 2^62 for
    // the longest ring (2^14) and q < 2^55.
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &m)
    {
        const int64_t t = (int64_t)w.w * (int64_t)yv;
        const uint64_t base = 32 * m.q + (uint64_t)(int64_t)xv;
        x = base + (uint64_t)t;
        y = base - (uint64_t)t;
    }
    D2_DEV static void fwd_pass_begin(elem &, const Mod &) {}
    D2_DEV static void fwd_end(elem &, const Mod &) {}
    // inverse: values in [0, 4q)
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool = false)
    {
        const elem four_q = 4 * m.q;
        const elem s = x + y, d = x + four_q - y;
        x = csub(s, four_q);
        y = mul<SC>(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x + 4 * m.q - y;
        x = mul<SC>(s, ninv, m);
        y = mul<SC>(d, wn, m);
    }
    D2_DEV static void inv_pass_begin(elem &, const Mod &) {}
    D2_DEV static elem inv_input(uint64_t canon, const Mod &) { return canon; }

    // any value < 2^62 -> [0, q)
    D2_DEV static uint64_t canon_wide(elem x, const Mod &m)
    {
        const elem r = shoup_tail_one(x, qhat_exact(x, m.one_s), m.nq);   // [0, 2q)
        return csub(r, m.q);
    }
    // [0, 4q) -> [0, q)
    D2_DEV static uint64_t canon_lazy(elem x, const Mod &m) { return csub(csub(x, 2 * m.q), m.q); }
    D2_DEV static uint64_t canon_fwd(elem x, const Mod &m) { return canon_wide(x, m); }
    D2_DEV static uint64_t canon_inv(elem x, const Mod &m) { return canon_lazy(x, m); }
    // forward output + one lazy product
    D2_DEV static uint64_t canon_acc(elem x, const Mod &m) { return canon_wide(x, m); }
};

// ---------------------------------------------------------------------------------------
// ArithB: moduli < 2^61, Harvey butterflies with an exact quotient.
// ---------------------------------------------------------------------------------------
struct ArithB {
    typedef uint64_t elem;
    typedef uint64_t word;          // LDS word of an exchange
    typedef ModU Mod;
    typedef TwU Twid;
    static constexpr int KIND = 2, INV_LIM = 0, INV_PROD = 0;

    D2_DEV static Mod mod(uint64_t q) { return Mod{q, 0 - q, 0}; }
    D2_DEV static Mod mod(uint64_t q, uint64_t one_s63) { return Mod{q, 0 - q, one_s63}; }
    D2_DEV static Twid tw(const Tw &t) { return Twid{t.w, t.ws}; }
    D2_DEV static Twid tw(uint64_t w, uint64_t ws64) { return Twid{w, ws64 >> 1}; }
    // element of a prepared key: values at v, 64-bit quotients at vs
    typedef Twid Key;
    D2_DEV static Key key_of(uint64_t v, uint64_t vs) { return tw(v, vs); }
    D2_DEV static Key key(const uint64_t *v, const uint64_t *vs, uint32_t lane_off, uint32_t slot_off)
    {
        return tw(ld64(v, lane_off, slot_off), ld64(vs, lane_off, slot_off));
    }
    // a value that several keys multiply
    typedef elem Factor;
    D2_DEV static Factor factor(elem u, const Mod &) { return u; }
    D2_DEV static elem factor_key_add(const Factor &u, const Key &k, elem x, const Mod &m) { return mul_key_add(u, k, x, m); }
    static constexpr bool SUM_SMALL = false;
    // table entry i: per-lane index / wave-uniform index (scalar registers, see mul<true>)
    static constexpr bool SCALAR_TW = true;
    D2_DEV static Twid load_v(const Tw *table, uint32_t i)
    {
        const U128 e = ld128(table, 16u * i, 0);
        return Twid{e.lo, e.hi};
    }
    D2_DEV static Twid load_u(const Tw *table, uint32_t i)
    {
        return Twid{const_ld64(table, 16u * i), const_ld64(table, 16u * i + 8u)};
    }

    // w*y mod q in [0, 2q), for y < 2^63.
    template <bool SC = false>
    D2_DEV static elem mul(elem y, const Twid &w, const Mod &m)
    {
        return shoup_tail<SC>(y, w.w, qhat_exact<SC>(y, w.ws), m.nq);
    }
    // sums of canonical words, canonical at every step
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t q) { return csub(a + b, q); }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &) { return s; }
    D2_DEV static elem from_small(int32_t v, const Mod &m)
    {
        return v >= 0 ? (uint64_t)v : m.q - (uint64_t)(uint32_t)(-v);
    }
    D2_DEV static elem from_canon(uint64_t v, const Mod &) { return v; }
    D2_DEV static elem add(elem a, elem b) { return a + b; }
    // u * key + x, lazy (x: a forward output); a sum of that kind as the x of another one
    D2_DEV static elem mul_key_add(elem u, const Key &k, elem x, const Mod &m) { return add(mul(u, k, m), x); }
    D2_DEV static elem renorm(elem x, const Mod &m) { return from_canon(canon_acc(x, m), m); }
    D2_DEV static elem mul_u32(uint32_t y, const Twid &w, const Mod &m) { return mul(y, w, m); }
    D2_DEV static elem neg(elem x, const Mod &m) { return 2 * m.q - x; }           // minus a product
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &m) { return x + from_small(v, m); }

    // x, y in [0, 4q) -> [0, 4q)
    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int = 0)
    {
        const elem two_q = 2 * m.q;
        const elem u = csub(x, two_q);
        x = shoup_tail_add<SC>(y, w.w, qhat_exact<SC>(y, w.ws), m.nq, u);       // u + t
        y = (2 * u + two_q) - x;                                                // u + 2q - t
    }
    // first stage on small signed inputs: no short cut here (the butterflies need their inputs below 4q)
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &m)
    {
        x = from_small(xv, m);
        y = from_small(yv, m);
        ct<SC>(x, y, w, m);
    }
    D2_DEV static void fwd_pass_begin(elem &, const Mod &) {}
    D2_DEV static void fwd_end(elem &, const Mod &) {}
    // x, y in [0, 2q) -> [0, 2q)
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool = false)
    {
        const elem two_q = 2 * m.q;
        const elem s = x + y, d = x + two_q - y;
        x = csub(s, two_q);
        y = mul<SC>(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x + 2 * m.q - y;
        x = mul<SC>(s, ninv, m);
        y = mul<SC>(d, wn, m);
    }
    D2_DEV static void inv_pass_begin(elem &, const Mod &) {}
    D2_DEV static elem inv_input(uint64_t canon, const Mod &) { return canon; }

    D2_DEV static uint64_t canon_lazy(elem x, const Mod &m) { return csub(csub(x, 2 * m.q), m.q); }
    // any value < 2^63 -> [0, q)
    D2_DEV static uint64_t canon_wide(elem x, const Mod &m)
    {
        const elem r = shoup_tail_one(x, qhat_exact(x, m.one_s), m.nq);
        return csub(r, m.q);
    }
    D2_DEV static uint64_t canon_fwd(elem x, const Mod &m) { return canon_lazy(x, m); }
    D2_DEV static uint64_t canon_inv(elem x, const Mod &m) { return csub(x, m.q); }
    // forward output + one lazy product: [0, 6q)
    D2_DEV static uint64_t canon_acc(elem x, const Mod &m) { return canon_lazy(csub(x, 4 * m.q), m); }
};

// ---------------------------------------------------------------------------------------
// ArithF: moduli < 2^44, residues as doubles holding integers (signed representatives).
// ---------------------------------------------------------------------------------------
struct ArithF {
    typedef double elem;
    typedef uint64_t word;          // LDS word of an exchange
    struct Mod {
        double q, qinv;
        uint64_t qi;
    };
    struct Twid {
        double w;
    };
    static constexpr int KIND = 0, INV_LIM = 0, INV_PROD = 0;

    D2_DEV static double u2d(uint64_t v)    // exact for v < 2^52
    {
        return __longlong_as_double((long long)(v | 0x4330000000000000ull)) - 4503599627370496.0;
    }
    D2_DEV static uint64_t d2u(double r)    // exact for integers 0 <= r < 2^52
    {
        return (uint64_t)__double_as_longlong(r + 4503599627370496.0) & 0x000fffffffffffffull;
    }
    D2_DEV static Mod mod(uint64_t q)
    {
        const double qd = u2d(q);
        return Mod{qd, 1.0 / qd, q};
    }
    // aux: bits of the double 1/q (what the per-modulus table holds for this policy)
    D2_DEV static Mod mod(uint64_t q, uint64_t aux) { return Mod{u2d(q), __longlong_as_double((long long)aux), q}; }
    D2_DEV static Twid tw(const Tw &t) { return Twid{__longlong_as_double((long long)t.w)}; }
    D2_DEV static Twid tw(uint64_t w, uint64_t) { return Twid{u2d(w)}; }
    // element of a prepared key: only the values are read
    typedef Twid Key;
    D2_DEV static Key key_of(uint64_t v, uint64_t vs) { return tw(v, vs); }
    D2_DEV static Key key(const uint64_t *v, const uint64_t *, uint32_t lane_off, uint32_t slot_off)
    {
        return Twid{u2d(ld64(v, lane_off, slot_off))};
    }
    // table entry i: per-lane index / wave-uniform index (scalar registers feed the f64 ALU directly)
    static constexpr bool SCALAR_TW = true;
    D2_DEV static Twid load_v(const Tw *table, uint32_t i)
    {
        return Twid{__longlong_as_double((long long)ld64(table, 16u * i, 0))};
    }
    D2_DEV static Twid load_u(const Tw *table, uint32_t i)
    {
        return Twid{__longlong_as_double((long long)const_ld64(table, 16u * i))};
    }

    // x - round(x/q) q: about (-q/2, q/2)
    D2_DEV static elem reduce(elem x, const Mod &m)
    {
        const double b = __builtin_rint(x * m.qinv);
        return __builtin_fma(-b, m.q, x);
    }
    // w*y mod q as a signed representative, for |w y| < 2^96.  Its magnitude is at most
    // q/2 + 1.5 |w y| 2^-52: the quotient is rounded from h/q computed with a relative error of 2^-52, and
    // the low part l of the product (|l| <= |w y| 2^-53) is added after the reduction.  That is q/2 + 1 for
    // canonical operands and up to 0.75 q for |y| = 42 q at the largest modulus.
    template <bool SC = false>
    D2_DEV static elem mul(elem y, const Twid &w, const Mod &m)
    {
        const double h = w.w * y;
        const double l = __builtin_fma(w.w, y, -h);
        const double b = __builtin_rint(h * m.qinv);
        const double r = __builtin_fma(-b, m.q, h);
        return r + l;
    }
    // sums of canonical words (at most 64 of them: canon_wide), left unreduced until sum_end
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t) { return a + b; }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &m) { return canon_wide(u2d(s), m); }
    D2_DEV static elem from_small(int32_t v, const Mod &) { return (double)v; }
    D2_DEV static elem from_canon(uint64_t v, const Mod &) { return u2d(v); }
    D2_DEV static elem mul_u32(uint32_t y, const Twid &w, const Mod &m) { return mul((double)y, w, m); }
    D2_DEV static elem neg(elem x, const Mod &) { return -x; }
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &) { return x + (double)v; }
    D2_DEV static elem add(elem a, elem b) { return a + b; }
    // u * key + x, lazy (x: a forward output); a sum of that kind as the x of another one
    D2_DEV static elem mul_key_add(elem u, const Key &k, elem x, const Mod &m) { return add(mul(u, k, m), x); }
    D2_DEV static elem renorm(elem x, const Mod &m) { return from_canon(canon_acc(x, m), m); }

    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int = 0)
    {
        const elem t = mul<SC>(y, w, m);
        const elem u = x;
        x = u + t;
        y = u - t;
    }
    // a value that several keys multiply
    typedef elem Factor;
    D2_DEV static Factor factor(elem u, const Mod &) { return u; }
    D2_DEV static elem factor_key_add(const Factor &u, const Key &k, elem x, const Mod &m) { return mul_key_add(u, k, x, m); }
    // s[0] + sum of c[j] s[j], |s| <= 32: the first stages of a transform on small inputs, taken together.  The multiplicands
    // are signed representatives: one product is at most 16 q, three 48 q; twelve further stages and a product with a
    // key take that to 59 q at q = 2^44 (see ct_small), inside the 64 q of canon_wide.
    static constexpr bool SUM_SMALL = true;
    struct Small {
        double w;
    };
    D2_DEV static Small small(const Twid &t, bool neg, const Mod &m)
    {
        const double w = t.w + t.w > m.q ? t.w - m.q : t.w;
        return Small{neg ? -w : w};
    }
    template <int SS>
    D2_DEV static elem sum_small(const int32_t (&s)[SS], const Small (&c)[SS], const Mod &)
    {
        double x = (double)s[0];
#pragma unroll
        for (int j = 1; j < SS; ++j) x = __builtin_fma(c[j].w, (double)s[j], x);
        return x;
    }
    // +-lam m[0] + e[0] +- I (+-lam m[1] + e[1]), m below 2^30: the first stage on an encoded message and its error; c as in
    // sum_small, lam_i = I lam (n0, n1: the product with m[0], m[1] is subtracted).  Two products and 16 q.
    D2_DEV static elem sum_encoded(const uint32_t (&mm)[2], const int32_t (&e)[2], const Twid &lam, const Twid &lam_i, bool n0,
                                   bool n1, const Small (&c)[2], const Mod &m)
    {
        const elem t0 = mul_u32(mm[0], lam, m), t1 = mul_u32(mm[1], lam_i, m), s = sum_small(e, c, m);
        return (n0 ? s - t0 : s + t0) + (n1 ? -t1 : t1);
    }
    // First stage on small signed inputs (|xv|, |yv| <= 32): w*yv is exact in a double (< 2^49), so the
    // stage is one multiplication and two additions.  The values then reach 32q; every later stage adds one
    // product (see mul), i.e. takes a bound of c q to (1 + 1.5 q 2^-52) c q + q/2: 41.3 q after the 13 further
    // stages of the longest ring that starts this way (2^14) at q = 2^44, 42.1 q with one more lazy product
    // on top -- inside what canon_wide accepts (64 q) and far inside the 2^53 of exact integers.
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &)
    {
        const double t = w.w * (double)yv, u = (double)xv;
        x = u + t;
        y = u - t;
    }
    D2_DEV static void fwd_pass_begin(elem &, const Mod &) {}
    D2_DEV static void fwd_end(elem &, const Mod &) {}
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool = false)
    {
        const elem s = x + y, d = x - y;
        x = s;
        y = mul<SC>(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x - y;
        x = mul<SC>(s, ninv, m);
        y = mul<SC>(d, wn, m);
    }
    // the sum path of the inverse doubles every stage: bring it back once per pass
    D2_DEV static void inv_pass_begin(elem &x, const Mod &m) { x = reduce(x, m); }
    D2_DEV static elem inv_input(uint64_t canon, const Mod &) { return u2d(canon); }

    // |x| <= 64 q -> [0, q).  x/q is either an integer or at least 1/q > 2^-44 away from one; the
    // computed quotient is off by at most 2 * 64 * 2^-53 = 2^-46 (the rounding of 1/q and of the
    // fused multiply-add), so with a bias of 2^-46 floor() is exact and the remainder needs no correction.
    D2_DEV static uint64_t canon_wide(elem x, const Mod &m)
    {
        const double b = __builtin_floor(__builtin_fma(x, m.qinv, 0x1p-46));
        return d2u(__builtin_fma(-b, m.q, x));
    }
    D2_DEV static uint64_t canon_lazy(elem x, const Mod &m) { return canon_wide(x, m); }
    D2_DEV static uint64_t canon_fwd(elem x, const Mod &m) { return canon_wide(x, m); }
    D2_DEV static uint64_t canon_inv(elem x, const Mod &m) { return canon_wide(x, m); }
    D2_DEV static uint64_t canon_acc(elem x, const Mod &m) { return canon_wide(x, m); }
};

// ---------------------------------------------------------------------------------------
// Arith32: moduli < 2^30, 32-bit residues, Harvey butterflies with a 32-bit Shoup quotient.
// Forward values in [0, 4q) (< 2^32), a finished forward transform in [0, 2q) so that one more lazy
// product can be added without overflow; inverse values in [0, 2q).
// Table entries hold {w | floor(w 2^32 / q) << 32, -} (8 bytes are read per twiddle).
// ---------------------------------------------------------------------------------------
struct Arith32 {
    typedef uint32_t elem;
    typedef uint32_t word;          // LDS word of an exchange
    struct Mod {
        uint32_t q, two_q, nq;      // nq = 2^32 - q
        uint32_t one_s;             // floor(2^32 / q)
    };
    struct Twid {
        uint32_t w, ws;
    };
    static constexpr int KIND = 3, INV_LIM = 0, INV_PROD = 0;

    D2_DEV static Mod mod(uint64_t q, uint64_t one_s32) { return Mod{(uint32_t)q, 2u * (uint32_t)q, 0u - (uint32_t)q, (uint32_t)one_s32}; }
    D2_DEV static Mod mod(uint64_t q) { return mod(q, (1ull << 32) / q); }
    D2_DEV static Twid tw(const Tw &t) { return Twid{lo32(t.w), hi32(t.w)}; }
    D2_DEV static Twid tw(uint64_t w, uint64_t ws64) { return Twid{(uint32_t)w, hi32(ws64)}; }
    // element of a prepared key: values at v, 64-bit quotients at vs (their high words are the 32-bit quotients)
    typedef Twid Key;
    D2_DEV static Key key_of(uint64_t v, uint64_t vs) { return tw(v, vs); }
    D2_DEV static Key key(const uint64_t *v, const uint64_t *vs, uint32_t lane_off, uint32_t slot_off)
    {
        return tw(ld64(v, lane_off, slot_off), ld64(vs, lane_off, slot_off));
    }
    static constexpr bool SCALAR_TW = true;
    D2_DEV static Twid load_v(const Tw *table, uint32_t i)
    {
        const uint64_t e = ld64(table, 16u * i, 0);
        return Twid{lo32(e), hi32(e)};
    }
    D2_DEV static Twid load_u(const Tw *table, uint32_t i)
    {
        const uint64_t e = const_ld64(table, 16u * i);
        return Twid{lo32(e), hi32(e)};
    }

    // x >= m ? x - m : x for x < 2m: the smaller of x and x - m as unsigned numbers
    D2_DEV static uint32_t csub32(uint32_t x, uint32_t m)
    {
        const uint32_t d = x - m;
        return d < x ? d : x;
    }
    // w*y mod q in [0, 2q), for any 32-bit y: the low word of w y + floor(ws y / 2^32) (2^32 - q)
    template <bool SC = false>
    D2_DEV static elem mul(elem y, const Twid &w, const Mod &m)
    {
        const uint32_t qh = __umulhi(y, w.ws);
        return (uint32_t)(mul32(w.w, y) + mul32(qh, m.nq));
    }
    // sums of canonical words, canonical at every step
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t q) { return csub(a + b, q); }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &) { return s; }
    D2_DEV static elem from_small(int32_t v, const Mod &m) { return v >= 0 ? (uint32_t)v : m.q - (uint32_t)(-v); }
    D2_DEV static elem from_canon(uint64_t v, const Mod &) { return (uint32_t)v; }
    D2_DEV static elem add(elem a, elem b) { return a + b; }
    // u * key + x, lazy (x: a forward output); a sum of that kind as the x of another one
    D2_DEV static elem mul_key_add(elem u, const Key &k, elem x, const Mod &m) { return add(mul(u, k, m), x); }
    D2_DEV static elem renorm(elem x, const Mod &m) { return from_canon(canon_acc(x, m), m); }
    D2_DEV static elem mul_u32(uint32_t y, const Twid &w, const Mod &m) { return mul(y, w, m); }
    D2_DEV static elem neg(elem x, const Mod &m) { return m.two_q - x; }           // minus a product
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &m) { return x + from_small(v, m); }

    // x, y in [0, 4q) -> [0, 4q)
    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int = 0)
    {
        const elem u = csub32(x, m.two_q);
        const elem t = mul<SC>(y, w, m);
        x = u + t;
        y = u + m.two_q - t;
    }
    // first stage on small signed inputs: no short cut (8 instructions per butterfly as it is)
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &m)
    {
        x = from_small(xv, m);
        y = from_small(yv, m);
        ct<SC>(x, y, w, m);
    }
    // a value that several keys multiply
    typedef elem Factor;
    D2_DEV static Factor factor(elem u, const Mod &) { return u; }
    D2_DEV static elem factor_key_add(const Factor &u, const Key &k, elem x, const Mod &m) { return mul_key_add(u, k, x, m); }
    // s[0] + sum of c[j] s[j], |s| <= 32, in [0, 4q)
    static constexpr bool SUM_SMALL = true;
    struct Small {
        Twid w;
        bool neg;
    };
    D2_DEV static Small small(const Twid &t, bool neg, const Mod &) { return Small{t, neg}; }
    template <int SS>
    D2_DEV static elem sum_small(const int32_t (&s)[SS], const Small (&c)[SS], const Mod &m)
    {
        uint32_t x = from_small(s[0], m);
#pragma unroll
        for (int j = 1; j < SS; ++j) {
            const uint32_t t = mul(from_small(c[j].neg ? -s[j] : s[j], m), c[j].w, m);
            x = (j > 1 ? csub32(x, m.two_q) : x) + t;
        }
        return x;
    }
    // +-lam m[0] + e[0] +- I (+-lam m[1] + e[1]), in [0, 4q]
    D2_DEV static elem sum_encoded(const uint32_t (&mm)[2], const int32_t (&e)[2], const Twid &lam, const Twid &lam_i, bool n0,
                                   bool n1, const Small (&c)[2], const Mod &m)
    {
        const uint32_t t0 = mul(mm[0], lam, m), t1 = mul(mm[1], lam_i, m);
        const uint32_t s = csub32(sum_small(e, c, m), m.two_q) + (n0 ? m.two_q - t0 : t0);
        return csub32(s, m.two_q) + (n1 ? m.two_q - t1 : t1);
    }
    D2_DEV static void fwd_pass_begin(elem &, const Mod &) {}
    // the last step of a forward transform: [0, 4q) -> [0, 2q)
    D2_DEV static void fwd_end(elem &x, const Mod &m) { x = csub32(x, m.two_q); }
    // x, y in [0, 2q) -> [0, 2q)
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool = false)
    {
        const elem s = x + y, d = x + m.two_q - y;
        x = csub32(s, m.two_q);
        y = mul<SC>(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x + m.two_q - y;
        x = mul<SC>(s, ninv, m);
        y = mul<SC>(d, wn, m);
    }
    D2_DEV static void inv_pass_begin(elem &, const Mod &) {}
    D2_DEV static elem inv_input(uint64_t canon, const Mod &) { return (uint32_t)canon; }

    // [0, 4q) -> [0, q)
    D2_DEV static uint64_t canon_lazy(elem x, const Mod &m) { return csub32(csub32(x, m.two_q), m.q); }
    // any 32-bit value -> [0, q)
    D2_DEV static uint64_t canon_wide(elem x, const Mod &m)
    {
        const uint32_t r = x - __umulhi(x, m.one_s) * m.q;        // [0, 2q)
        return csub32(r, m.q);
    }
    D2_DEV static uint64_t canon_fwd(elem x, const Mod &m) { return canon_lazy(x, m); }
    D2_DEV static uint64_t canon_inv(elem x, const Mod &m) { return csub32(x, m.q); }
    // finished forward transform ([0, 2q)) + one lazy product ([0, 2q))
    D2_DEV static uint64_t canon_acc(elem x, const Mod &m) { return canon_lazy(x, m); }
};

// ---------------------------------------------------------------------------------------
// ArithP, ArithQ: moduli q = 2^b - c with a small c (b < 56 / b <= 60), the form in which RNS primes are
// usually searched.  2^(b+1) = 2c (mod q), so the part of a product above bit b + 1 folds down with one
// multiply-add and no quotient is ever estimated.
//
// A multiplicand w is kept as w and W = w 2^32 mod q, each split at bit s = b - 31:
//     w = w01 2^s + w00,   W = w11 2^s + w10,   w01, w11 < 2^31.
// For y = y1 2^32 + y0:  w y = w y0 + W y1 = A + B 2^s (mod q),  A = w00 y0 + w10 y1,  B = w01 y0 + w11 y1 < 2^64,
// and B 2^s = B_lo 2^s + B_hi 2^(b+1) = B_lo 2^s + B_hi 2c.  Six multiply-adds in all; an addend u rides on the
// first.  With kappa = y / 2^64 and gamma = c 2^32 / 2^b the result is below
//     T = ((2 + gamma)(1 + kappa) + 2) 2^b <= G q,
// G computed at context creation (8 for ArithP's 55-bit and 6 for ArithQ's 60-bit moduli; larger when c is).
// The kernels are bound by instruction issue.  Measured, with the Shoup quotients and with this: round of 34,272
// ciphertexts, N = 2^13, four 54-bit limbs, 28.7 -> 22.6 ms; N = 2^14, eight limbs, 20.7 -> 17.5 ms; transforms of
// N = 2^16, 16 60-bit limbs, batch 64: forward 0.509 -> 0.431 ms, inverse 0.516 -> 0.437 ms.
// ---------------------------------------------------------------------------------------
struct ModPm {
    uint64_t q;
    uint64_t k;         // G q: what a difference adds to stay positive
    uint64_t c64;       // c as a 64-bit addend
    uint32_t c, c2;     // c, 2c
    uint32_t p2s;       // 2^s
    uint32_t sh;        // b - 32: bit b of a value as a bit of its high word
};
struct TwPm {
    uint32_t w00, w01, w10, w11;
};

// Written as C: the compiler selects one v_mad_u64_u32 for each of these multiply-adds and interleaves independent
// butterflies.  (As single-instruction assembly statements every dependent pair cost a wait state on top,
// 762 in k_encrypt for N = 2^13 instead of 118, and 116 registers instead of 90.)
D2_DEV ModPm pm_mod(uint64_t q, uint64_t k)
{
    const uint32_t b = 64u - (uint32_t)__builtin_clzll(q);
    const uint32_t c = (uint32_t)(((uint64_t)1 << b) - q);
    uint32_t p2s = 1u << (b - 31);
#if D2_GCN_ASM
    asm("" : "+s"(p2s));        // or a multiplication by it becomes a shift, a move and an addition
#endif
    return ModPm{q, k, c, c, 2 * c, p2s, b - 32};
}
D2_DEV TwPm pm_tw(const Tw &t) { return TwPm{lo32(t.w), hi32(t.w), lo32(t.ws), hi32(t.ws)}; }

// w y + u in u + [0, G q), any y the policy's ranges allow; the low 64 bits are the value (nothing wraps)
D2_DEV uint64_t pm_mul_add(uint64_t y, const TwPm &w, uint64_t u, const ModPm &m)
{
    const uint64_t a = mul32(w.w10, hi32(y)) + (mul32(w.w00, lo32(y)) + u);
    const uint64_t b = mul32(w.w11, hi32(y)) + mul32(w.w01, lo32(y));
    return mul32(m.c2, hi32(b)) + (mul32(m.p2s, lo32(b)) + a);
}
D2_DEV uint64_t pm_mul(uint64_t y, const TwPm &w, const ModPm &m) { return pm_mul_add(y, w, 0, m); }
// 2u + k, as the one instruction it is (as C it comes back as a shift and an addition in half of the butterflies:
// the compiler moves the constant past the subtraction that follows)
D2_DEV uint64_t pm_twice_plus(uint64_t u, uint64_t k)
{
#if D2_GCN_ASM
    uint64_t d;
    asm("v_lshl_add_u64 %0, %1, 1, %2" : "=v"(d) : "v"(u), "s"(k));
    return d;
#else
    return 2 * u + k;
#endif
}
// the same for a 32-bit y (a plaintext coefficient)
D2_DEV uint64_t pm_mul_u32(uint32_t y, const TwPm &w, const ModPm &m)
{
    const uint64_t b = mul32(w.w01, y);
    return mul32(m.c2, hi32(b)) + (mul32(m.p2s, lo32(b)) + mul32(w.w00, y));
}
// s[0] + sum of +-w[j] s[j], |s| <= 32 and at most three products, as pm_mul with signed multiply-adds: the sums of the
// halves are A and B, |B| < 2^38, and 2^40 added to B keeps it positive; 2^40 2^s = 2^(b + 9) = 512 c is taken off
// again.  The result is in (0, 4q).
struct SmallPm {
    int32_t w0, w1;     // the halves of +-w
};
D2_DEV SmallPm pm_small(const TwPm &w, bool neg)
{
    return neg ? SmallPm{-(int32_t)w.w00, -(int32_t)w.w01} : SmallPm{(int32_t)w.w00, (int32_t)w.w01};
}
template <int SS>
D2_DEV uint64_t pm_sum_small(const int32_t (&s)[SS], const SmallPm (&c)[SS], const ModPm &m)
{
    int64_t a = (int64_t)(m.q - 512 * m.c64) + s[0], b = (int64_t)1 << 40;
#pragma unroll
    for (int j = 1; j < SS; ++j) {
        a = (int64_t)c[j].w0 * s[j] + a;
        b = (int64_t)c[j].w1 * s[j] + b;
    }
    return mul32(m.c2, hi32((uint64_t)b)) + (mul32(m.p2s, lo32((uint64_t)b)) + (uint64_t)a);
}
// +-lam m[0] + e[0] +- I (+-lam m[1] + e[1]), m below 2^30, |e| <= 32, in the same way (the signs are in lam, lam_i and
// c): here |B| < 2^62 + 2^37, 2^63 is added, and 2^63 2^s = 2^(b + 32) = 2^32 c is less than k = G q.  The result is
// below (G + 3 + gamma / 2) q.
D2_DEV uint64_t pm_sum_encoded(const uint32_t (&mm)[2], const int32_t (&e)[2], const SmallPm &lam, const SmallPm &lam_i,
                               const SmallPm &c, const ModPm &m)
{
    uint64_t a = (m.k - (m.c64 << 32)) + (uint64_t)(int64_t)e[0], b = (uint64_t)1 << 63;
    a = (uint64_t)((int64_t)c.w0 * e[1]) + a;
    b = (uint64_t)((int64_t)c.w1 * e[1]) + b;
    a = (uint64_t)((int64_t)lam.w0 * (int32_t)mm[0]) + a;
    b = (uint64_t)((int64_t)lam.w1 * (int32_t)mm[0]) + b;
    a = (uint64_t)((int64_t)lam_i.w0 * (int32_t)mm[1]) + a;
    b = (uint64_t)((int64_t)lam_i.w1 * (int32_t)mm[1]) + b;
    return mul32(m.c2, hi32(b)) + (mul32(m.p2s, lo32(b)) + a);
}
// bit b and above folded down: x < 2^64 -> below 2^b + (x >> b) c
D2_DEV uint64_t pm_fold(uint64_t x, const ModPm &m)
{
    const uint32_t h = hi32(x) >> m.sh, top = hi32(x) & ((1u << m.sh) - 1u);
    return mul32(m.c, h) + (((uint64_t)top << 32) | lo32(x));
}
// x -> [0, q) for x + (x / 2^b + 1) c < 2^64: the quotient is h = x >> b or h + 1, and h + 1 exactly when
// x >= (h + 1) q, i.e. when x + (h + 1) c reaches (h + 1) 2^b
D2_DEV uint64_t pm_canon(uint64_t x, const ModPm &m)
{
    const uint32_t h = hi32(x) >> m.sh;
    const uint64_t z = mul32(m.c, h) + (x + m.c64);
    const uint64_t r = mul32(m.c, hi32(z) >> m.sh) + x;
    return ((uint64_t)(hi32(r) & ((1u << m.sh) - 1u)) << 32) | lo32(r);
}
// A canonical value as a multiplicand: W = w 2^32 = w01 2^(b+1) + w00 2^32 = w01 2c + w00 2^32, folded once.
D2_DEV TwPm pm_split(uint64_t w, const ModPm &m)
{
    const uint32_t s = m.sh + 1, mask = m.p2s - 1u;
    TwPm t;
    t.w00 = lo32(w) & mask;
    t.w01 = (uint32_t)(w >> s);
    const uint64_t W = pm_fold(mul32(m.c2, t.w01) + ((uint64_t)t.w00 << 32), m);
    t.w10 = lo32(W) & mask;
    t.w11 = (uint32_t)(W >> s);
    return t;
}

// A lazy value as a multiplicand of canonical ones: folded to 2^b + (x >> b) c, then split like a canonical one.  With
// e = (x >> b) c / 2^b < 1 its halves are below 2^31 (1 + e), and a product with y < q is below
// ((2 + gamma) (1 + e) + 2) 2^b, less than 2 G q (4 to 5 q for the moduli a prime search gives).
D2_DEV TwPm pm_factor(uint64_t x, const ModPm &m) { return pm_split(pm_fold(x, m), m); }

// ---------------------------------------------------------------------------------------
// ArithP: nothing is corrected inside a forward transform.  In units of q: a forward value is at most 64 + 16 G
// (small first stage, 15 further stages, one product with a key); an inverse pass of at most four stages takes
// values up to 8 G, folds the sums of its first stage (the first pass of all starts from canonical values and
// folds nothing) and leaves at most 8 G.  All of it stays below 2^63.
// A forward butterfly is 9 instructions (ArithS 15), an inverse one 11 (ArithS 20).
// ---------------------------------------------------------------------------------------
struct ArithP {
    typedef uint64_t elem;
    typedef uint64_t word;          // LDS word of an exchange
    typedef ModPm Mod;
    typedef TwPm Twid;
    static constexpr int KIND = 4;
    // bounds of inverse values in units of q (G = 8): a product, and what a pass takes and leaves
    static constexpr int INV_PROD = 8, INV_LIM = 64;

    D2_DEV static Mod mod(uint64_t q, uint64_t k) { return pm_mod(q, k); }
    D2_DEV static Twid tw(const Tw &t) { return pm_tw(t); }
    // element of a prepared key: only the value is read, its split form costs 9 instructions and saves
    // half of the bytes
    typedef uint64_t Key;
    D2_DEV static Key key_of(uint64_t v, uint64_t) { return v; }
    D2_DEV static Key key(const uint64_t *v, const uint64_t *, uint32_t lane_off, uint32_t slot_off)
    {
        return ld64(v, lane_off, slot_off);
    }
    static constexpr bool SCALAR_TW = true;
    D2_DEV static Twid load_v(const Tw *table, uint32_t i)
    {
        const U128 e = ld128(table, 16u * i, 0);
        return TwPm{lo32(e.lo), hi32(e.lo), lo32(e.hi), hi32(e.hi)};
    }
    D2_DEV static Twid load_u(const Tw *table, uint32_t i)
    {
        return pm_tw(Tw{const_ld64(table, 16u * i), const_ld64(table, 16u * i + 8u)});
    }
    template <bool SC = false>
    D2_DEV static elem mul(elem y, const Twid &w, const Mod &m) { return pm_mul(y, w, m); }
    D2_DEV static elem mul_u32(uint32_t y, const Twid &w, const Mod &m) { return pm_mul_u32(y, w, m); }
    D2_DEV static elem mul_key_add(elem u, Key k, elem x, const Mod &m) { return pm_mul_add(u, pm_split(k, m), x, m); }
    // a value that several keys multiply: split once instead of a key each time (4 + 9 instructions for 9 per key)
    typedef TwPm Factor;
    D2_DEV static Factor factor(elem u, const Mod &m) { return pm_factor(u, m); }
    D2_DEV static elem factor_key_add(const Factor &u, Key k, elem x, const Mod &m) { return pm_mul_add(k, u, x, m); }
    D2_DEV static elem renorm(elem x, const Mod &) { return x; }
    // sums of canonical words (at most 65 of them), left unreduced until sum_end
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t) { return a + b; }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &m) { return pm_canon(s, m); }
    D2_DEV static elem from_small(int32_t v, const Mod &m)
    {
        return v >= 0 ? (uint64_t)v : m.q - (uint64_t)(uint32_t)(-v);
    }
    D2_DEV static elem from_canon(uint64_t v, const Mod &) { return v; }
    D2_DEV static elem add(elem a, elem b) { return a + b; }
    D2_DEV static elem neg(elem x, const Mod &m) { return m.k - x; }               // minus a product
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &m) { return x + (m.q + (uint64_t)(int64_t)v); }
    static constexpr bool SUM_SMALL = true;
    typedef SmallPm Small;
    D2_DEV static Small small(const Twid &t, bool neg, const Mod &) { return pm_small(t, neg); }
    template <int SS>
    D2_DEV static elem sum_small(const int32_t (&s)[SS], const Small (&c)[SS], const Mod &m) { return pm_sum_small(s, c, m); }
    D2_DEV static elem sum_encoded(const uint32_t (&mm)[2], const int32_t (&e)[2], const Twid &lam, const Twid &lam_i, bool n0,
                                   bool n1, const Small (&c)[2], const Mod &m)
    {
        return pm_sum_encoded(mm, e, pm_small(lam, n0), pm_small(lam_i, n1), c[1], m);
    }
    // x' = u + t comes out of the multiply-adds, y' = u + G q - t = (2u + G q) - x'
    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int = 0)
    {
        const elem u = x;
        x = pm_mul_add(y, w, u, m);
        y = pm_twice_plus(u, m.k) - x;
    }
    // first stage on small signed inputs (|v| <= 32): w yv is an exact 64-bit product, both results in (0, 64q + 32)
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &m)
    {
        const uint64_t wv = ((uint64_t)w.w01 << (m.sh + 1)) + w.w00;
        const int64_t t = (int64_t)wv * (int64_t)yv;
        const uint64_t base = 32 * m.q + (uint64_t)(int64_t)xv;
        x = base + (uint64_t)t;
        y = base - (uint64_t)t;
    }
    D2_DEV static void fwd_end(elem &, const Mod &) {}
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool fold = true)
    {
        const elem s = x + y, d = x + 8 * m.k - y;
        x = fold ? pm_fold(s, m) : s;
        y = pm_mul(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x + 8 * m.k - y;
        x = pm_mul(s, ninv, m);
        y = pm_mul(d, wn, m);
    }
    D2_DEV static void inv_pass_begin(elem &, const Mod &) {}
    D2_DEV static elem inv_input(uint64_t canon, const Mod &) { return canon; }
    D2_DEV static uint64_t canon_wide(elem x, const Mod &m) { return pm_canon(x, m); }
    D2_DEV static uint64_t canon_lazy(elem x, const Mod &m) { return pm_canon(x, m); }
    D2_DEV static uint64_t canon_fwd(elem x, const Mod &m) { return pm_canon(x, m); }
    D2_DEV static uint64_t canon_inv(elem x, const Mod &m) { return pm_canon(x, m); }
    D2_DEV static uint64_t canon_acc(elem x, const Mod &m) { return pm_canon(x, m); }
};

// ---------------------------------------------------------------------------------------
// ArithQ: the same with 16 multiples of q or fewer in a word.  The odd stages of a forward transform fold u
// first: values are at most 1 + G (and a bit) after them and 1 + 2 G after an even stage; the inputs of stage 0
// may reach 1 + G.  Inverse values are at most G between the stages: a sum of two products is folded, sums
// of folded values are not before they reach G.  A forward butterfly is 10.5 instructions on average, an inverse
// one 12 (ArithB 21 and 22).
// ---------------------------------------------------------------------------------------
struct ArithQ : ArithP {
    static constexpr int KIND = 5;
    static constexpr int INV_PROD = 6, INV_LIM = 6;

    // x may come from an even last stage (1 + 2 G): folded before the product is added
    D2_DEV static elem mul_key_add(elem u, Key k, elem x, const Mod &m)
    {
        return pm_mul_add(u, pm_split(k, m), pm_fold(x, m), m);
    }
    D2_DEV static elem factor_key_add(const Factor &u, Key k, elem x, const Mod &m) { return pm_mul_add(k, u, pm_fold(x, m), m); }
    D2_DEV static elem renorm(elem x, const Mod &m) { return pm_fold(x, m); }
    template <bool SC = false>
    D2_DEV static void ct(elem &x, elem &y, const Twid &w, const Mod &m, int stage = 1)
    {
        const elem u = (stage & 1) ? pm_fold(x, m) : x;
        x = pm_mul_add(y, w, u, m);
        y = pm_twice_plus(u, m.k) - x;
    }
    template <bool SC = false>
    D2_DEV static void ct_small(int32_t xv, int32_t yv, elem &x, elem &y, const Twid &w, const Mod &m)
    {
        x = from_small(xv, m);
        y = from_small(yv, m);
        ct<SC>(x, y, w, m, 0);
    }
    // sums of canonical words, canonical at every step
    D2_DEV static uint64_t sum(uint64_t a, uint64_t b, uint64_t q) { return csub(a + b, q); }
    D2_DEV static uint64_t sum_end(uint64_t s, const Mod &) { return s; }
    D2_DEV static elem add_small(elem x, int32_t v, const Mod &m) { return x + from_small(v, m); }
    template <bool SC = false>
    D2_DEV static void gs(elem &x, elem &y, const Twid &w, const Mod &m, bool fold = true)
    {
        const elem s = x + y, d = x + m.k - y;
        x = fold ? pm_fold(s, m) : s;
        y = pm_mul(d, w, m);
    }
    template <bool SC = false>
    D2_DEV static void gs_last(elem &x, elem &y, const Twid &ninv, const Twid &wn, const Mod &m)
    {
        const elem s = x + y, d = x + m.k - y;
        x = pm_mul(s, ninv, m);
        y = pm_mul(d, wn, m);
    }
};

// Which sums of an inverse pass a policy has to fold (bit 16 * stage + slot), from the bounds of its values in
// units of q: a pass starts from canonical values (FIRST) or from values up to A::INV_LIM, a product is at
// most A::INV_PROD, a sum at most the sum of its operands' bounds, and a sum that could exceed
// A::INV_LIM is folded to 1.  INV_LIM = 0: the policy corrects its sums by itself.
template <class A>
constexpr uint64_t inv_folds(bool first, int stages, int slots, int bit0 = 0 /* slot bit of the first stage */)
{
    uint64_t mask = 0;
    if (A::INV_LIM == 0) return mask;
    int bound[16] = {};
    for (int k = 0; k < slots; ++k) bound[k] = first ? 1 : A::INV_LIM;
    for (int i = 0; i < stages; ++i)
        for (int k = 0; k < slots; ++k) {
            const int other = k | (1 << (bit0 + i));
            if (other == k) continue;
            int s = bound[k] + bound[other];
            if (s > A::INV_LIM) {
                s = 1;
                mask |= (uint64_t)1 << (16 * i + k);
            }
            bound[k] = s;
            bound[other] = A::INV_PROD;
        }
    return mask;
}

// A multiplicand in vector registers that a loop keeps: nothing is derived from it outside the loop (the compiler
// would hold its words zero-extended to 64 bits there, twice the registers).
template <class T>
D2_DEV void pin_multiplicand(T &) {}
template <>
D2_DEV void pin_multiplicand<TwPm>(TwPm &w)
{
#if D2_GCN_ASM
    asm volatile("" : "+v"(w.w00), "+v"(w.w01), "+v"(w.w10), "+v"(w.w11));
#else
    (void)w;
#endif
}

// canonical u64 helpers used outside the transforms
D2_DEV uint64_t add_mod(uint64_t a, uint64_t b, uint64_t q) { return csub(a + b, q); }
// w*y mod q, canonical, with the 64-bit Shoup quotient ws64 = floor(w 2^64 / q); any 64-bit y
D2_DEV uint64_t mul_shoup64(uint64_t y, uint64_t w, uint64_t ws64, uint64_t q)
{
    const uint64_t r = w * y - __umul64hi(ws64, y) * q;
    return csub(r, q);
}

// uint64 <-> element bit patterns for lazily stored intermediates and 8-byte LDS words; a policy with
// 4-byte LDS words (Arith32) stores its elements as they are
template <class A>
D2_DEV uint64_t to_bits(typename A::elem v);
template <>
D2_DEV uint64_t to_bits<ArithS>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t to_bits<ArithB>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t to_bits<ArithP>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t to_bits<ArithQ>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t to_bits<ArithF>(double v) { return (uint64_t)__double_as_longlong(v); }

template <>
D2_DEV uint64_t to_bits<Arith32>(uint32_t v) { return v; }

template <class A>
D2_DEV typename A::elem from_bits(uint64_t v);
template <>
D2_DEV uint32_t from_bits<Arith32>(uint64_t v) { return (uint32_t)v; }
template <>
D2_DEV uint64_t from_bits<ArithS>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t from_bits<ArithB>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t from_bits<ArithP>(uint64_t v) { return v; }
template <>
D2_DEV uint64_t from_bits<ArithQ>(uint64_t v) { return v; }
template <>
D2_DEV double from_bits<ArithF>(uint64_t v) { return __longlong_as_double((long long)v); }

template <class A>
D2_DEV typename A::word to_word(typename A::elem v)
{
    if constexpr (sizeof(typename A::word) == 8) return to_bits<A>(v);
    else return v;
}
template <class A>
D2_DEV typename A::elem from_word(typename A::word v)
{
    if constexpr (sizeof(typename A::word) == 8) return from_bits<A>(v);
    else return v;
}

}  // namespace d2
