// HIP kernels of the exchange round.  One workgroup owns one polynomial (or one ciphertext
// and walks over its RNS limbs); transforms run in registers + LDS (ntt_engine.hpp).
#pragma once
#include "ntt_engine.hpp"
#include "philox.hpp"
#include <stddef.h>
#include <type_traits>

// no fused multiply-add unless written out: float results here are compared bit for bit
#pragma clang fp contract(off)

namespace d2 {

constexpr int MAX_LIMBS = 16;
constexpr int MAX_GROUP = 64;

// Per-modulus constants; entry L of the table array describes the plaintext modulus t.
// Tw entries are in the context's arithmetic format ({w, floor(w 2^63/q)} for ArithS and ArithB, the split
// multiplicands for ArithP and ArithQ, {bits of the double w, -} for the floating-point policy, {w | floor(w 2^32/q) << 32, -} for
// the 32-bit policy; the entry of the plaintext modulus is always in the 32-bit format), except
// `pow64`, which is always {w, floor(w 2^64/q)} (it works on 64-bit integers).
struct LimbTab {
    uint64_t q;
    uint64_t one_s;     // floor(2^63 / q); floating-point policy: bits of the double 1/q; 32-bit policy: floor(2^32 / q);
                        // ArithP, ArithQ: G q
    Tw ninv;            // N^-1 mod q
    Tw wn;              // (inverse twiddle 1) * N^-1 mod q
    Tw lambda;          // floor(Q/t) mod q
    Tw lambda_i;        // that times forward twiddle 1
    Tw ninvg, wng;      // ninv and wn times (Q/q)^-1 mod q: an inverse transform scaled for the rounding of a decryption
    uint64_t theta_hi;  // floor(t * 2^128 / q), high and low words
    uint64_t theta_lo;
    Tw pow64;           // 2^64 mod q, integer pair (reduction of 128-bit uniform blocks)
    uint64_t inv64;     // floor(2^64 / q)
    const Tw *fwd;      // forward twiddles, N entries
    const Tw *inv;      // inverse twiddles, N entries
};

// Entry i (uniform over the workgroup) of the table array, fetched with scalar loads so that the
// constants and the table pointers stay in scalar registers.
D2_DEV LimbTab load_tab(const LimbTab *tabs, uint32_t i)
{
    const LimbTab *e = tabs + i;
    LimbTab r;
    r.q = const_ld64(e, offsetof(LimbTab, q));
    r.one_s = const_ld64(e, offsetof(LimbTab, one_s));
    r.ninv = Tw{const_ld64(e, offsetof(LimbTab, ninv)), const_ld64(e, offsetof(LimbTab, ninv) + 8)};
    r.wn = Tw{const_ld64(e, offsetof(LimbTab, wn)), const_ld64(e, offsetof(LimbTab, wn) + 8)};
    r.lambda_i = Tw{const_ld64(e, offsetof(LimbTab, lambda_i)), const_ld64(e, offsetof(LimbTab, lambda_i) + 8)};
    r.lambda = Tw{const_ld64(e, offsetof(LimbTab, lambda)), const_ld64(e, offsetof(LimbTab, lambda) + 8)};
    r.ninvg = Tw{const_ld64(e, offsetof(LimbTab, ninvg)), const_ld64(e, offsetof(LimbTab, ninvg) + 8)};
    r.wng = Tw{const_ld64(e, offsetof(LimbTab, wng)), const_ld64(e, offsetof(LimbTab, wng) + 8)};
    r.theta_hi = const_ld64(e, offsetof(LimbTab, theta_hi));
    r.theta_lo = const_ld64(e, offsetof(LimbTab, theta_lo));
    r.pow64 = Tw{const_ld64(e, offsetof(LimbTab, pow64)), const_ld64(e, offsetof(LimbTab, pow64) + 8)};
    r.inv64 = const_ld64(e, offsetof(LimbTab, inv64));
    r.fwd = (const Tw *)const_ld64(e, offsetof(LimbTab, fwd));
    r.inv = (const Tw *)const_ld64(e, offsetof(LimbTab, inv));
    return r;
}

// The 128-bit little-endian value of a Philox block reduced mod q (uniform sampling): its high half times 2^64 mod q and its
// low half times 1, both prepared multiplicands that take any 64-bit word.  (Word by word it was seven such products: refresh of 153
// ciphertexts by seven members, N = 8192, 54 bits, four limbs 616 / 574 us, masks modulo t and alpha modulo q.)
D2_DEV uint64_t uniform_mod(const Block4 &b, const LimbTab &tb)
{
    const uint64_t q = tb.q, lo = ((uint64_t)b.w[1] << 32) | b.w[0], hi = ((uint64_t)b.w[3] << 32) | b.w[2];
    return add_mod(mul_shoup64(hi, tb.pow64.w, tb.pow64.ws, q), mul_shoup64(lo, 1, tb.inv64, q), q);
}

// The same modulo the plaintext modulus (below 2^30): the words times 2^96, 2^64, 2^32 and 1 modulo t add up to less than 2^64.
// The masks of refresh shares: 575.6 -> 563.7 us for the refresh above.
struct UniformT {
    uint64_t t, inv64;
    uint32_t p32, p64, p96;
    D2_DEV explicit UniformT(const LimbTab &tt) : t(tt.q), inv64(tt.inv64)
    {
        const uint32_t a = 0u - (uint32_t)tt.one_s * (uint32_t)t;              // one_s = floor(2^32 / t)
        const uint32_t b = (uint32_t)mul_shoup64((uint64_t)a * a, 1, inv64, t);
        p32 = wave_uniform(a);
        p64 = wave_uniform(b);
        p96 = wave_uniform((uint32_t)mul_shoup64((uint64_t)a * b, 1, inv64, t));
    }
    D2_DEV uint32_t operator()(const Block4 &b) const
    {
        const uint64_t s = mul32(b.w[3], p96) + (mul32(b.w[2], p64) + (mul32(b.w[1], p32) + b.w[0]));
        return (uint32_t)mul_shoup64(s, 1, inv64, t);
    }
};

struct RoundConst {
    uint64_t t;
    uint32_t L;
    uint32_t eta_mask;   // low eta bits set
    int32_t clamp;       // floor(((t-1)/2) / K_max)
    float scale;         // 2^f
    float inv_scale;     // 2^-f
    PhiloxKey key;
    uint32_t coeff_packing;   // 0: value j of a ciphertext is slot j (default); 1: it is coefficient j
};

struct PtrList {
    const void *p[MAX_GROUP];
};

// Job tables passed by value in the kernel arguments; grid.y indexes the job.
constexpr int JOB_CHUNK = 112;   // 112 * 32 B of table + the other arguments stay under the 4 KB argument limit
// Jobs of Encrypt and of the decryption shares: one job = one (party, group) pair, its C results at out + job * stride.
// What belongs to a party or to a group is listed once and a job is two indices, so that one launch takes a whole
// round: with a row of pointers per job (112 to a launch) the 2,060 jobs of 100 users in 100 groups were 19 launches of
// barely more than one chip's worth of workgroups each.
// Measured, that round (N = 4096, 5 indices, 2 limbs of 54 bits), with the vectors encoded ahead: 1.98 -> 1.42 ms.
// Launches of few jobs list each in a row of its own, entry i of every array, so that a workgroup requests all it needs at
// once: two dependent reads of the arguments cost
// 0.3 to 0.5 us of a launch (a share of 60 indices, N = 1024, 30 bits 5.0 -> 4.8 us; N = 2048, 60 bits 10.3 -> 10.0 us).
constexpr int RJ_PARTIES = 112, RJ_GROUPS = 112, RJ_JOBS = 880, RJ_ROWS = 112;      // 4,016 bytes
struct RoundJobs {
    const void *src[RJ_PARTIES];       // gradient, plaintext polynomials or prepared secret share of a party
    const uint64_t *key[RJ_GROUPS];    // prepared public key or aggregate of a group
    uint64_t *out;
    size_t stride;                     // words
    uint32_t party[RJ_PARTIES / 2];    // ids, two to a word (scalar loads come in words)
    uint32_t group[RJ_GROUPS / 2];
    uint32_t job[RJ_JOBS / 2];         // index into src | index into key << 8, two to a word

    static constexpr uint32_t half(uint32_t v, uint32_t i, uint32_t old) { return i & 1 ? (old & 0xffffu) | (v << 16) : v; }
    void set_party(uint32_t i, const void *p, uint32_t id) { src[i] = p; party[i / 2] = half(id, i, party[i / 2]); }
    void set_group(uint32_t i, const uint64_t *p, uint32_t id) { key[i] = p; group[i / 2] = half(id, i, group[i / 2]); }
    void set_job(uint32_t i, uint32_t si, uint32_t ki) { job[i / 2] = half(si | (ki << 8), i, job[i / 2]); }
    void set_row(uint32_t i, const void *s, uint32_t party_id, const uint64_t *k, uint32_t group_id)
    {
        set_party(i, s, party_id);
        set_group(i, k, group_id);
        set_job(i, i, i);
    }
};
static_assert(sizeof(RoundJobs) <= 4016, "with the other arguments of a launch under 4 KB");
struct RoundJob {                      // one entry, uniform over the workgroup
    const void *src;
    const uint64_t *key;
    uint64_t *out;
    uint32_t party, group;
};
D2_DEV uint32_t half_word(uint32_t w, uint32_t i) { return (w >> (16 * (i & 1))) & 0xffffu; }
// ROWS: look at row i together with the job's entry.  The branch costs as much as the second read where the kernel
// has more to wait for (rows and not: encryption of 60 indices, N = 4096, 36 bits 18.9 / 18.5 us, N = 2048, 60 bits, quotients
// 23.9 / 23.5; share, N = 4096, 36 bits 8.7 / 8.5; but N = 8192, 54 bits 69.5 / 70.2 and 29.1 / 29.3).  Shares in halves of
// N = 2^14 on doubles gain 0.2 us by rows on an empty chip and lose by them over several turns (1,040 shares of eight limbs,
// 36 bits 689 / 675; 54 bits 714 both).
template <bool ROWS>
D2_DEV RoundJob round_job(const RoundJobs &t, uint32_t i)
{
    if constexpr (!ROWS) {
        const uint32_t e = half_word(t.job[i >> 1], i), si = e & 0xffu, ki = e >> 8;
        return RoundJob{t.src[si], t.key[ki], t.out + (size_t)i * t.stride, half_word(t.party[si >> 1], si),
                        half_word(t.group[ki >> 1], ki)};
    }
    const uint32_t row = i < (uint32_t)RJ_ROWS ? i : 0;
    uint32_t job = t.job[i >> 1], party = t.party[row >> 1], group = t.group[row >> 1];
    RoundJob r = {t.src[row], t.key[row], t.out, 0, 0};
    size_t stride = t.stride;
#if D2_GCN_ASM
    // all requested here: the compiler would move them below the branch
    asm volatile("" : "+s"(job), "+s"(party), "+s"(group), "+s"(r.src), "+s"(r.key), "+s"(r.out), "+s"(stride));
#endif
    const uint32_t e = half_word(job, i);
    r.out += (size_t)i * stride;
    r.party = half_word(party, row);
    r.group = half_word(group, row);
    if (e != (row | row << 8)) {
        const uint32_t si = e & 0xffu, ki = e >> 8;
        r.src = t.src[si];
        r.key = t.key[ki];
        r.party = half_word(t.party[si >> 1], si);
        r.group = half_word(t.group[ki >> 1], ki);
    }
    return r;
}
enum { FROM_WORDS64 = 0, FROM_WORDS32 = 1, FROM_VECTOR = 2 };   // what Encrypt reads
constexpr int ENCODE_CHUNK = 448;
struct EncodeJobs {                    // one job = one party's vector
    const float *src[ENCODE_CHUNK];
};
// Conversion shares in the same way: one job = one member's shares towards one receiver, three indices.
// Measured, 80 rows of pointers to a launch and this: 100 users in neighbourhoods of some 20, N = 4096, 5 indices, 2 limbs
// 2.35 -> 2.15 ms; 32 nodes of 7, N = 8192, 37 indices (three launches anyway full) 7.20 ms both.
constexpr int CJ_PARTIES = 104, CJ_GROUPS = 64, CJ_JOBS = 320, CJ_ROWS = 64;       // 4,016 bytes
struct ConvJobs {
    const uint64_t *sk[CJ_PARTIES];    // prepared secret share of a member
    const uint64_t *pk[CJ_PARTIES];    // prepared public key of a receiver
    const uint64_t *ct[CJ_GROUPS];     // aggregate of a group [C][2][L][N]
    uint64_t *out;                     // shares [C][2][L][N] of the first job
    size_t stride;                     // words
    uint32_t member[CJ_PARTIES / 2];   // ids, two to a word
    uint32_t receiver[CJ_PARTIES / 2];
    uint32_t group[CJ_GROUPS / 2];
    uint32_t job[CJ_JOBS];             // index into sk | into pk << 8 | into ct << 16

    void set_member(uint32_t i, const uint64_t *p, uint32_t id) { sk[i] = p; member[i / 2] = RoundJobs::half(id, i, member[i / 2]); }
    void set_receiver(uint32_t i, const uint64_t *p, uint32_t id) { pk[i] = p; receiver[i / 2] = RoundJobs::half(id, i, receiver[i / 2]); }
    void set_group(uint32_t i, const uint64_t *p, uint32_t id) { ct[i] = p; group[i / 2] = RoundJobs::half(id, i, group[i / 2]); }
    void set_job(uint32_t i, uint32_t si, uint32_t pi, uint32_t gi) { job[i] = si | pi << 8 | gi << 16; }
    void set_row(uint32_t i, const uint64_t *s, uint32_t member_id, const uint64_t *p, uint32_t receiver_id, const uint64_t *c,
                 uint32_t group_id)
    {
        set_member(i, s, member_id);
        set_receiver(i, p, receiver_id);
        set_group(i, c, group_id);
        set_job(i, i, i, i);
    }
};
static_assert(sizeof(ConvJobs) <= 4016, "with the other arguments of a launch under 4 KB");
struct ConvJob {                       // one entry, uniform over the workgroup
    const uint64_t *sk, *pk, *ct;
    uint64_t *out;
    uint32_t who, group;               // member | receiver << 16: the party word of the counters
};
D2_DEV ConvJob conv_job(const ConvJobs &t, uint32_t i)
{
    const uint32_t row = i < (uint32_t)CJ_ROWS ? i : 0;
    uint32_t e = t.job[i], member = t.member[row >> 1], receiver = t.receiver[row >> 1], group = t.group[row >> 1];
    ConvJob r = {t.sk[row], t.pk[row], t.ct[row], t.out, 0, 0};
    size_t stride = t.stride;
#if D2_GCN_ASM
    asm volatile("" : "+s"(e), "+s"(member), "+s"(receiver), "+s"(group), "+s"(r.sk), "+s"(r.pk), "+s"(r.ct), "+s"(r.out),
                      "+s"(stride));
#endif
    r.out += (size_t)i * stride;
    r.who = half_word(member, row) | half_word(receiver, row) << 16;
    r.group = half_word(group, row);
    if (e != (row | row << 8 | row << 16)) {
        const uint32_t si = e & 0xffu, pi = (e >> 8) & 0xffu, gi = e >> 16;
        r.sk = t.sk[si];
        r.pk = t.pk[pi];
        r.ct = t.ct[gi];
        r.who = half_word(t.member[si >> 1], si) | half_word(t.receiver[pi >> 1], pi) << 16;
        r.group = half_word(t.group[gi >> 1], gi);
    }
    return r;
}
struct GroupJobs {                     // one job = one group: K buffers laid out at a fixed stride
    const uint64_t *first[JOB_CHUNK];  // buffer of the group's first member
    const uint64_t *ct[JOB_CHUNK];     // aggregate (combine) / unused (sum)
    void *out[JOB_CHUNK];              // aggregate (sum) / decoded floats (combine)
    uint32_t K[JOB_CHUNK];
};
constexpr int FIN_PARTIES = 128, FIN_MEMBERS = 1400, FIN_GROUPS = 64;   // 3.6 KB of table; any group fits
struct FinishJobs {                    // one job = one group
    const uint64_t *sk[FIN_PARTIES];   // prepared secret shares of the parties of this launch
    float *out[FIN_GROUPS];            // decoded floats
    uint16_t party[FIN_PARTIES];
    uint16_t group[FIN_GROUPS];
    uint16_t first[FIN_GROUPS + 2];    // members of group g: entries [first[g], first[g + 1]) of
    uint8_t member[FIN_MEMBERS];       // indices into sk and party
};
constexpr int CONV_CHUNK = 80;         // 80 * 36 B of table
struct RecvJobs {                      // one job = one receiver of one group (MBFV.Convert)
    const uint64_t *first[CONV_CHUNK]; // conversion shares of the group's first member for this receiver
    const uint64_t *ct[CONV_CHUNK];    // aggregate
    const uint64_t *sk[CONV_CHUNK];    // the receiver's prepared secret key
    void *out[CONV_CHUNK];             // decoded floats
    uint32_t K[CONV_CHUNK];
};

D2_DEV uint32_t bitrev(uint32_t v, int bits) { return __brev(v) >> (32 - bits); }

// Returns v unchanged but opaque to the optimiser.  Used at the top of per-limb loops so that
// per-thread addresses and sample conversions are recomputed per iteration (a few
// instructions) instead of being hoisted and kept in ~100 registers across the whole loop.
D2_DEV int opaque(int v)
{
#if D2_GCN_ASM
    asm volatile("" : "+v"(v));
#endif
    return v;
}
D2_DEV uint32_t opaque(uint32_t v) { return (uint32_t)opaque((int)v); }

// The loads above are issued before anything below.
D2_DEV void requested()
{
#if D2_GCN_ASM
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// A value that is the same in every lane, in a scalar register from here on.  The compiler may keep a loop's counter, and the
// pointers it derives from it, in vector registers although all lanes agree, and then wraps every buffer access in a loop over the lanes' values
// (32 of them in k_share<ArithS>: 152 shares, N = 8192, two limbs, 24.7 us; without 21.6).
D2_DEV uint32_t scalar(uint32_t v)
{
#if D2_GCN_ASM
    asm("" : "+s"(v));
#endif
    return v;
}
// The counter of a loop over limbs: only with Shoup quotients (ArithS, ArithB) does the compiler move it; the other kernels are as good with it as
// without (92 launches of 30 to 60 bits: 0.94 to 1.03 of the time, 1.00 in the mean) and keep their own.
template <class A>
D2_DEV uint32_t limb_counter(uint32_t l)
{
    return A::KIND == 1 || A::KIND == 2 ? scalar(l) : l;
}

// The limbs [first, end) of a workgroup where a launch splits every polynomial over gridDim.z workgroups: `split` holds
// the limbs of part 0 and, from bit 16, those of each further part.
struct LimbRange {
    uint32_t first, end;
};
D2_DEV uint32_t launch_part()
{
#if D2_GCN_ASM
    return __builtin_amdgcn_workgroup_id_z();
#else
    return 0;                           // the arithmetic's host check includes this file and launches nothing
#endif
}
D2_DEV LimbRange limb_range(uint32_t split, uint32_t L, uint32_t z)
{
    const uint32_t head = split & 0xffffu, rest = split >> 16;
    const uint32_t first = z ? head + (z - 1) * rest : 0, end = first + (z ? rest : head);
    return LimbRange{first, end < L ? end : L};
}

// -------------------------------------------------------------------------------------
// Plain batched transforms: polys [B][L][N] in place, one workgroup per (b, limb).
// -------------------------------------------------------------------------------------
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_ntt_forward(uint64_t *polys, const LimbTab *tabs, uint32_t L)
{
    typedef typename ENG::A A;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const LimbTab tb = load_tab(tabs, blockIdx.x % L);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    uint64_t *p = polys + (size_t)blockIdx.x * ENG::NB;
    typename A::elem x[ENG::E];
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) x[k] = A::from_canon(p[ENG::coef_pos(k, tid)], md);
    ENG::forward(x, lds, tid, 0, tb.fwd, md);
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) p[ENG::eval_pos(k, tid)] = A::canon_fwd(x[k], md);
}

template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_ntt_inverse(uint64_t *polys, const LimbTab *tabs, uint32_t L)
{
    typedef typename ENG::A A;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const LimbTab tb = load_tab(tabs, blockIdx.x % L);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    uint64_t *p = polys + (size_t)blockIdx.x * ENG::NB;
    typename A::elem x[ENG::E];
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) x[k] = A::inv_input(p[ENG::eval_pos(k, tid)], md);
    ENG::template inverse<true>(x, lds, tid, 0, tb.inv, md, A::tw(tb.ninv), A::tw(tb.wn));
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) p[ENG::coef_pos(k, tid)] = A::canon_inv(x[k], md);
}

// The same where there is more than one polynomial to a workgroup and one workgroup fills a compute unit: without a
// second one nothing overlaps loads with butterflies, so every workgroup walks through the polynomials of its limb with the
// next one's words already requested.  grid: a multiple of L.  See the rule in Launch::ntt.
template <class ENG, bool INV>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_ntt_walk(uint64_t *polys, const LimbTab *tabs, uint32_t L, uint32_t total)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t lane = 8u * (uint32_t)tid;
    const LimbTab tb = load_tab(tabs, blockIdx.x % L);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    const size_t stride = (size_t)gridDim.x * ENG::NB;
    uint64_t *p = polys + (size_t)blockIdx.x * ENG::NB;
    uint64_t nx[E];
#pragma unroll
    for (int k = 0; k < E; ++k) nx[k] = ld64(p, lane, 8u * ENG::T * k);
    for (uint32_t i = blockIdx.x; i < total; i += gridDim.x, p += stride) {
        typename A::elem x[E];
#pragma unroll
        for (int k = 0; k < E; ++k) x[k] = INV ? A::inv_input(nx[k], md) : A::from_canon(nx[k], md);
        if (total - i > gridDim.x) {
#pragma unroll
            for (int k = 0; k < E; ++k) nx[k] = ld64(p + stride, lane, 8u * ENG::T * k);
        }
        if constexpr (INV) ENG::template inverse<true>(x, lds, tid, 0, tb.inv, md, A::tw(tb.ninv), A::tw(tb.wn));
        else ENG::forward(x, lds, tid, 0, tb.fwd, md);
#pragma unroll
        for (int k = 0; k < E; ++k) st64(p, lane, 8u * ENG::T * k, INV ? A::canon_inv(x[k], md) : A::canon_fwd(x[k], md));
    }
}

// -------------------------------------------------------------------------------------
// Transforms longer than one workgroup can hold: the top LOGH = LOGN - LOGB stages couple
// the 2^LOGH blocks of NB coefficients ("head", register-only, strided global access); the
// remaining LOGB stages are independent per block ("tail", the engine with a block id).
// Between the two kernels the data stays in the policy's lazy representation.
// -------------------------------------------------------------------------------------
template <class A, int LOGN, int LOGH>
__global__ void __launch_bounds__(256) k_head_forward(uint64_t *polys, const LimbTab *tabs, uint32_t L,
                                                        uint32_t poly0)
{
    constexpr int H = 1 << LOGH;
    constexpr int STRIDE = 1 << (LOGN - LOGH);
    const uint32_t poly = blockIdx.y;
    const LimbTab tb = load_tab(tabs, (poly0 + poly) % L);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    const Tw *tw = tb.fwd;
    uint64_t *p = polys + ((size_t)poly << LOGN) + (size_t)blockIdx.x * 256 + threadIdx.x;
    typename A::elem x[H];
#pragma unroll
    for (int k = 0; k < H; ++k) x[k] = A::from_canon(p[(size_t)k * STRIDE], md);
#pragma unroll
    for (int kb = LOGH - 1; kb >= 0; --kb) {
        const int s = LOGH - 1 - kb;
#pragma unroll
        for (int g = 0; g < (H >> (kb + 1)); ++g) {
            const typename A::Twid w = load_tw_uniform<A>(tw, (1u << s) + g);
#pragma unroll
            for (int j = 0; j < (1 << kb); ++j) {
                const int k0 = (g << (kb + 1)) | j;
                A::template ct<A::SCALAR_TW>(x[k0], x[k0 | (1 << kb)], w, md, s);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < H; ++k) p[(size_t)k * STRIDE] = to_bits<A>(x[k]);   // stays lazy
}

template <class A, int LOGN, int LOGH>
__global__ void __launch_bounds__(256) k_head_inverse(uint64_t *polys, const LimbTab *tabs, uint32_t L,
                                                        uint32_t poly0)
{
    constexpr int H = 1 << LOGH;
    constexpr int STRIDE = 1 << (LOGN - LOGH);
    const uint32_t poly = blockIdx.y;
    const LimbTab tb = load_tab(tabs, (poly0 + poly) % L);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    const Tw *tw = tb.inv;
    uint64_t *p = polys + ((size_t)poly << LOGN) + (size_t)blockIdx.x * 256 + threadIdx.x;
    constexpr uint64_t folds = inv_folds<A>(false, LOGH, H);
    typename A::elem x[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        x[k] = from_bits<A>(p[(size_t)k * STRIDE]);               // lazy, from the tail kernel
        A::inv_pass_begin(x[k], md);
    }
#pragma unroll
    for (int kb = 0; kb < LOGH; ++kb) {
        const int s = LOGH - 1 - kb;
        if (kb == LOGH - 1) {                                    // last stage: fold N^-1
#pragma unroll
            for (int j = 0; j < (1 << kb); ++j) A::template gs_last<true>(x[j], x[j | (1 << kb)], A::tw(tb.ninv), A::tw(tb.wn), md);
        } else {
#pragma unroll
            for (int g = 0; g < (H >> (kb + 1)); ++g) {
                const typename A::Twid w = load_tw_uniform<A>(tw, (1u << s) + g);
#pragma unroll
                for (int j = 0; j < (1 << kb); ++j) {
                    const int k0 = (g << (kb + 1)) | j;
                    A::template gs<A::SCALAR_TW>(x[k0], x[k0 | (1 << kb)], w, md, (folds >> (16 * kb + k0)) & 1);
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < H; ++k) p[(size_t)k * STRIDE] = A::canon_inv(x[k], md);
}

// Tail of a long transform over polys [B][L][N].  Tiles that share twiddles -- the same (limb, block)
// of every polynomial of the batch, a "group" of B members -- are given to one workgroup `tiles`
// members at a time: it fetches the twiddles once (scalar registers for the uniform passes, 56
// vector registers for the rest with 16-byte entries) and walks its members with the next member's
// coefficients already requested.  Without this the twiddles are twice the bytes of the data.
// Workgroups are handed to the 8 XCDs round-robin by linear id: XCD x = i % 8 walks the contiguous
// slot range [x * grid/8, (x+1) * grid/8), so that the workgroups of a group also share an L2.

struct TailTile {
    uint32_t limb, blk, m0, m1;       // members [m0, m1) of group (limb, blk)
};
D2_DEV TailTile tail_tile(uint32_t i, uint32_t grid, uint32_t B, uint32_t tiles, uint32_t wpg, uint32_t nblk)
{
    uint32_t slot = i;
    if ((grid & 7u) == 0) slot = (i & 7u) * (grid >> 3) + (i >> 3);
    const uint32_t group = slot / wpg, part = slot % wpg;
    // the same in every lane (they depend on the workgroup id only): keep them in scalar registers,
    // the divisions above went through the vector ALU
    TailTile t;
    t.limb = scalar(wave_uniform(group / nblk));
    t.blk = scalar(wave_uniform(group % nblk));
    t.m0 = scalar(wave_uniform(part * tiles));
    t.m1 = t.m0 + tiles < B ? t.m0 + tiles : B;
    return t;
}

// grid = L * 2^(LOGN - LOGB) * wpg, wpg = ceil(B / tiles) workgroups per group
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_tail_forward(uint64_t *polys, const LimbTab *tabs, uint32_t L,
                                                        uint32_t B, uint32_t tiles, uint32_t wpg)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const TailTile tt = tail_tile(blockIdx.x, gridDim.x, B, tiles, wpg, 1u << (ENG::LOGN - ENG::LOGB));
    if (tt.limb >= L || tt.m0 >= tt.m1) return;
    const LimbTab tb = load_tab(tabs, tt.limb);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    typename ENG::Twiddles tw;
    ENG::template load_all<false, false>(tw, tid, tt.blk, tb.fwd);
    const size_t stride = (size_t)L << ENG::LOGN;        // words between members
    uint64_t *p = polys + (((size_t)tt.m0 * L + tt.limb) << ENG::LOGN) + ((size_t)tt.blk << ENG::LOGB);
    uint64_t nx[E];
#pragma unroll
    for (int k = 0; k < E; ++k) nx[k] = ld64(p, 8u * (uint32_t)tid, 8u * ENG::T * k);
    for (uint32_t m = tt.m0; m < tt.m1; ++m, p += stride) {
        ENG::pin(tw);
        typename A::elem x[E];
#pragma unroll
        for (int k = 0; k < E; ++k) x[k] = from_bits<A>(nx[k]);
        if (m + 1 < tt.m1) {
#pragma unroll
            for (int k = 0; k < E; ++k) nx[k] = ld64(p + stride, 8u * (uint32_t)tid, 8u * ENG::T * k);
        }
        ENG::forward(x, lds, tid, tw, md);
#pragma unroll
        for (int k = 0; k < E; ++k) st64(p, 8u * (uint32_t)tid, 8u * ENG::T * k, A::canon_fwd(x[k], md));
    }
}

template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_tail_inverse(uint64_t *polys, const LimbTab *tabs, uint32_t L,
                                                        uint32_t B, uint32_t tiles, uint32_t wpg)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const TailTile tt = tail_tile(blockIdx.x, gridDim.x, B, tiles, wpg, 1u << (ENG::LOGN - ENG::LOGB));
    if (tt.limb >= L || tt.m0 >= tt.m1) return;
    const LimbTab tb = load_tab(tabs, tt.limb);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    typename ENG::Twiddles tw;
    ENG::template load_all<true, false>(tw, tid, tt.blk, tb.inv);
    const typename A::Twid ninv = A::tw(tb.ninv), wn = A::tw(tb.wn);
    const size_t stride = (size_t)L << ENG::LOGN;
    uint64_t *p = polys + (((size_t)tt.m0 * L + tt.limb) << ENG::LOGN) + ((size_t)tt.blk << ENG::LOGB);
    uint64_t nx[E];
#pragma unroll
    for (int k = 0; k < E; ++k) nx[k] = ld64(p, 8u * (uint32_t)tid, 8u * ENG::T * k);
    for (uint32_t m = tt.m0; m < tt.m1; ++m, p += stride) {
        ENG::pin(tw);
        typename A::elem x[E];
#pragma unroll
        for (int k = 0; k < E; ++k) x[k] = A::inv_input(nx[k], md);
        if (m + 1 < tt.m1) {
#pragma unroll
            for (int k = 0; k < E; ++k) nx[k] = ld64(p + stride, 8u * (uint32_t)tid, 8u * ENG::T * k);
        }
        ENG::template inverse<false>(x, lds, tid, tw, md, ninv, wn);
#pragma unroll
        for (int k = 0; k < E; ++k) st64(p, 8u * (uint32_t)tid, 8u * ENG::T * k, to_bits<A>(x[k]));   // lazy, head finishes
    }
}

// -------------------------------------------------------------------------------------
// Sampling helpers: small polynomials are drawn block by block, staged in LDS as packed
// words (one per coefficient, natural order) and then picked up by their pass-0 owners.
// -------------------------------------------------------------------------------------
// mu (ternary) in byte 0, e0 in byte 1, e1 in byte 2 (two's complement bytes); their domains are
// dom, dom + 1, dom + 2 (DOM_ENC_U for Encrypt, DOM_CVT_U for a conversion share)
template <class ENG>
D2_DEV void stage_encrypt_samples(uint32_t *lds32, int tid, uint32_t dom, uint32_t party, uint32_t group,
                                  uint32_t ct, const RoundConst &rc)
{
    for (int j = tid; j < ENG::N / 4; j += ENG::T) {
        int32_t mu[4], e0[4], e1[4];
        ternary4(philox4x32_10(j, ct, party, counter_tag(dom, 0, group), rc.key), mu);
        cbd2(philox4x32_10(2 * j, ct, party, counter_tag(dom + 1, 0, group), rc.key), rc.eta_mask, e0);
        cbd2(philox4x32_10(2 * j + 1, ct, party, counter_tag(dom + 1, 0, group), rc.key), rc.eta_mask, e0 + 2);
        cbd2(philox4x32_10(2 * j, ct, party, counter_tag(dom + 2, 0, group), rc.key), rc.eta_mask, e1);
        cbd2(philox4x32_10(2 * j + 1, ct, party, counter_tag(dom + 2, 0, group), rc.key), rc.eta_mask, e1 + 2);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lds32[4 * j + i] = ((uint32_t)mu[i] & 0xffu) | (((uint32_t)e0[i] & 0xffu) << 8) |
                               (((uint32_t)e1[i] & 0xffu) << 16);
    }
}

template <class ENG>
D2_DEV void stage_cbd(uint32_t *lds32, int tid, uint32_t domain, uint32_t party, uint32_t group, uint32_t ct,
                      const RoundConst &rc)
{
    for (int j = tid; j < ENG::NB / 2; j += ENG::T) {
        int32_t e[2];
        cbd2(philox4x32_10(j, ct, party, counter_tag(domain, 0, group), rc.key), rc.eta_mask, e);
        lds32[2 * j] = (uint32_t)e[0];
        lds32[2 * j + 1] = (uint32_t)e[1];
    }
}

// v of the neighbouring lane (lane ^ 1)
D2_DEV int32_t lane_xor1(int32_t v)
{
#if D2_GCN_ASM
    return __builtin_amdgcn_update_dpp(0, v, 0xb1 /* quad_perm [1,0,3,2] */, 0xf, 0xf, true);
#else
    return __shfl_xor(v, 1);
#endif
}

D2_DEV int32_t sbyte(uint32_t w, int i) { return (int32_t)(int8_t)(w >> (8 * i)); }

// The samples of a small polynomial that a thread's part of a transform starts from: packed bytes where they are more than
// its coefficients (FUSE).
template <class ENG, bool PACKED = (ENG::FUSE > 0)>
struct SmallPoly {
    static_assert(ENG::E == 8, "one 8-byte word per part");
    uint32_t w[ENG::SS][2];
    D2_DEV void set(int j, int k, uint32_t byte)
    {
        if (k % 4 == 0) w[j][k / 4] = byte & 0xffu;
        else w[j][k / 4] |= (byte & 0xffu) << (8 * (k % 4));
    }
    D2_DEV void get(int32_t (&v)[ENG::SS][ENG::E]) const
    {
#pragma unroll
        for (int j = 0; j < ENG::SS; ++j)
#pragma unroll
            for (int k = 0; k < ENG::E; k += 4) {
                const uint32_t b = opaque(w[j][k / 4]);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][k + i] = sbyte(b, i);
            }
    }
    D2_DEV uint64_t word(int j) const { return ((uint64_t)w[j][1] << 32) | w[j][0]; }
    D2_DEV void set_word(int j, uint64_t v)
    {
        w[j][0] = lo32(v);
        w[j][1] = hi32(v);
    }
};
template <class ENG>
struct SmallPoly<ENG, false> {
    int32_t v[ENG::E];
    D2_DEV void set(int, int k, uint32_t sample) { v[k] = (int32_t)sample; }
    D2_DEV void get(int32_t (&out)[1][ENG::E]) const
    {
#pragma unroll
        for (int k = 0; k < ENG::E; ++k) out[0][k] = opaque(v[k]);
    }
    D2_DEV uint64_t word(int) const            // 8 coefficients per thread
    {
        uint32_t w[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k / 4] |= ((uint32_t)v[k] & 0xffu) << (8 * (k % 4));
        return ((uint64_t)w[1] << 32) | w[0];
    }
    D2_DEV void set_word(int, uint64_t w)
    {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = sbyte(k < 4 ? lo32(w) : hi32(w), k % 4);
    }
};
// The three small polynomials of an encryption or a conversion share (mu, e0, e1), as stage_encrypt_samples left them
template <class ENG, bool PACKED = (ENG::FUSE > 0)>
struct SmallTriple {
    SmallPoly<ENG> p[3];
    D2_DEV void load(const uint32_t *stage, int tid)
    {
#pragma unroll
        for (int k = 0; k < ENG::E; ++k)
#pragma unroll
            for (int j = 0; j < ENG::SS; ++j) {
                const uint32_t v = stage[ENG::small_pos(j, k, tid)];
                p[0].set(j, k, v);
                p[1].set(j, k, v >> 8);
                p[2].set(j, k, v >> 16);
            }
    }
    template <int I>
    D2_DEV void get(int32_t (&v)[ENG::SS][ENG::E]) const { p[I].get(v); }
};
template <class ENG>
struct SmallTriple<ENG, false> {
    uint32_t w[ENG::E];
    D2_DEV void load(const uint32_t *stage, int tid)
    {
#pragma unroll
        for (int k = 0; k < ENG::E; ++k) w[k] = stage[ENG::coef_pos(k, tid)];
    }
    template <int I>
    D2_DEV void get(int32_t (&v)[1][ENG::E]) const
    {
#pragma unroll
        for (int k = 0; k < ENG::E; ++k) v[0][k] = sbyte(opaque(w[k]), I);
    }
};
// words of LDS that small_cbd exchanges samples through
template <class ENG>
constexpr int SMALL_LDS_WORDS = ENG::FUSE > 0 ? ENG::N / 8 : 0;

// Centred-binomial coefficients of a polynomial, drawn once by the workgroup.  A block holds two adjacent
// coefficients, i.e. the same slot of two adjacent lanes: of two slots the even lane draws the block of the first,
// the odd lane that of the second, and each hands over the half that is not its own.  A thread draws one or two of
// the SS parts that it needs (draw_part); the rest comes from the threads with the same positions in the other
// parts, which pass their bytes through `buf` (SMALL_LDS_WORDS; barriers in front of the write and of the read, none
// after it).
template <class ENG>
D2_DEV void small_cbd(SmallPoly<ENG> &s, uint64_t *buf, int tid, uint32_t domain, uint32_t party, uint32_t group,
                      uint32_t ct, const RoundConst &rc)
{
    const int odd = tid & 1;
    if constexpr (ENG::FUSE > 0) __syncthreads();        // readers of an earlier polynomial
    constexpr int ROW = ENG::PART / ENG::E;              // threads per part
#pragma unroll
    for (int r = 0; r < ENG::DRAW; ++r) {
        const int part = ENG::draw_part(r, tid);
#pragma unroll
        for (int k = 0; k < ENG::E; k += 2) {
            int32_t e[2];
            const uint32_t j = (uint32_t)(part * ENG::PART + (ENG::small_pos(0, k + odd, tid & ~1))) / 2;
            cbd2(philox4x32_10(j, ct, party, counter_tag(domain, 0, group), rc.key), rc.eta_mask, e);
            const int32_t mine = odd ? e[1] : e[0], got = lane_xor1(odd ? e[0] : e[1]);
            s.set(r, k, (uint32_t)(odd ? got : mine));
            s.set(r, k + 1, (uint32_t)(odd ? mine : got));
        }
        if constexpr (ENG::FUSE > 0) buf[part * ROW + tid % ROW] = s.word(r);
    }
    if constexpr (ENG::FUSE > 0) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ENG::SS; ++j) s.set_word(j, buf[j * ROW + tid % ROW]);
    }
}

// -------------------------------------------------------------------------------------
// Fixed point + slots (encode) as a device step: leaves the plaintext polynomial of
// ciphertext index c in registers in pass-0 (natural) ownership, values in [0, t).
// With rc.coeff_packing the values are the coefficients themselves (an addition-only workload
// never needs the slot structure): no transform on either side.
// `lds` must not have been used by the workgroup yet (no wave may still be reading it).
// -------------------------------------------------------------------------------------
template <class ENG>
D2_DEV void encode_to_regs(uint32_t (&m)[ENG::E], uint64_t *lds, int tid, const float *grad, uint64_t first,
                           uint64_t n_values, const LimbTab &tt, const RoundConst &rc)
{
    // the plaintext modulus is below 2^30: its transform runs on 32-bit residues whatever the context's
    // own arithmetic is (same thread shape and ownership)
    typedef typename ENG::template Rebind<Arith32> TE;
    typedef Arith32 A;
    const uint64_t t = tt.q;
    const typename A::Mod md = A::mod(t, tt.one_s);
    auto fixed = [&](uint64_t gi) -> uint64_t {          // value gi as a residue mod t
        float v = gi < n_values ? grad[gi] : 0.0f;
        float r = (v != v) ? 0.0f : __builtin_rintf(v * rc.scale);
        // The clamp bound (< 2^30) need not be a float once it exceeds 2^24: bring the rounded value into
        // the int32 range first (2^30 is a float), then compare as integers.
        r = r > 0x1p30f ? 0x1p30f : r;
        r = r < -0x1p30f ? -0x1p30f : r;
        int32_t z = (int32_t)r;
        z = z > rc.clamp ? rc.clamp : z;
        z = z < -rc.clamp ? -rc.clamp : z;
        return z >= 0 ? (uint64_t)z : t - (uint64_t)(uint32_t)(-z);
    };
    if (rc.coeff_packing) {                              // coefficient packing: no transform
#pragma unroll
        for (int k = 0; k < ENG::E; ++k) m[k] = (uint32_t)fixed(first + (uint64_t)ENG::coef_pos(k, tid));
        return;
    }
    // (no barrier in front of these writes: the callers have not used this buffer before)
    for (int j = tid; j < ENG::NB; j += ENG::T) lds[ENG::phys(j)] = fixed(first + (uint64_t)j);
    __syncthreads();
    // slot j is the evaluation xhat[j], which the engine keeps at block index bitrev(j)
    typename A::elem x[ENG::E];
#pragma unroll
    for (int k = 0; k < ENG::E; ++k)
        x[k] = A::inv_input(lds[ENG::phys((int)bitrev((uint32_t)(tid * ENG::E + k), ENG::LOGB))], md);
    TE::template inverse<true>(x, lds, tid, 0, tt.inv, md, A::tw(tt.ninv), A::tw(tt.wn));
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) m[k] = (uint32_t)A::canon_inv(x[k], md);
}

// registers hold a plaintext polynomial (natural ownership, [0,t)) -> floats
template <class ENG>
D2_DEV void decode_from_regs(uint32_t (&m)[ENG::E], uint64_t *lds, int tid, float *out, uint64_t first,
                             uint64_t n_values, const LimbTab &tt, const RoundConst &rc)
{
    typedef typename ENG::template Rebind<Arith32> TE;       // as in encode_to_regs
    typedef Arith32 A;
    const uint64_t t = tt.q;
    const typename A::Mod md = A::mod(t, tt.one_s);
    if (rc.coeff_packing) {                              // coefficient packing: no transform
#pragma unroll
        for (int k = 0; k < ENG::E; ++k) {
            const uint64_t gi = first + (uint64_t)ENG::coef_pos(k, tid), z = m[k];
            if (gi < n_values) {
                const int32_t c = z > (t - 1) / 2 ? (int32_t)((int64_t)z - (int64_t)t) : (int32_t)z;
                out[gi] = (float)c * rc.inv_scale;
            }
        }
        return;
    }
    typename A::elem x[ENG::E];
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) x[k] = A::from_canon((uint64_t)m[k], md);
    TE::forward(x, lds, tid, 0, tt.fwd, md);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ENG::E; ++k)
        lds[ENG::phys((int)bitrev((uint32_t)(tid * ENG::E + k), ENG::LOGB))] = A::canon_fwd(x[k], md);
    __syncthreads();
    for (int j = tid; j < ENG::NB; j += ENG::T) {
        uint64_t gi = first + (uint64_t)j;
        if (gi < n_values) {
            uint64_t z = lds[ENG::phys(j)];
            int32_t c = z > (t - 1) / 2 ? (int32_t)((int64_t)z - (int64_t)t) : (int32_t)z;
            out[gi] = (float)c * rc.inv_scale;
        }
    }
}

template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_encode(const float *grad, uint64_t n_values, uint64_t *pt,
                                                   const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    uint32_t m[ENG::E];
    encode_to_regs<ENG>(m, lds, tid, grad, (uint64_t)c * ENG::NB, n_values, load_tab(tabs, rc.L), rc);
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) pt[(size_t)c * ENG::NB + ENG::coef_pos(k, tid)] = m[k];
}

// The plaintexts of a whole round: grid = (C, parties), one 32-bit word per coefficient.  A party encrypts the same
// vector for every group it is in; encoding it in k_encrypt (an inverse transform modulo t and four barriers) repeats
// the work per group.  See the rule in run_round.
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_encode_parties(EncodeJobs jobs, uint64_t n_values, uint32_t *pt,
                                                                       const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    uint32_t m[ENG::E];
    encode_to_regs<ENG>(m, lds, tid, jobs.src[blockIdx.y], (uint64_t)c * ENG::NB, n_values, load_tab(tabs, rc.L), rc);
    pt += ((size_t)blockIdx.y * gridDim.x + c) * ENG::NB;
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) pt[ENG::coef_pos(k, tid)] = m[k];
}

template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_decode(const uint64_t *pt, uint64_t n_values, float *out,
                                                   const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    uint32_t m[ENG::E];
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) m[k] = (uint32_t)pt[(size_t)c * ENG::NB + ENG::coef_pos(k, tid)];
    decode_from_regs<ENG>(m, lds, tid, out, (uint64_t)c * ENG::NB, n_values, load_tab(tabs, rc.L), rc);
}

// -------------------------------------------------------------------------------------
// Set-up: one party's key share.  grid = L (one workgroup per limb).
//   sk (prepared): NTT(s) and Shoup quotients;  pk0 = -(p1 s + e) in evaluation form.
// p1 is the prepared common random polynomial.
// -------------------------------------------------------------------------------------
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_keygen(uint32_t party, uint64_t *sk, uint64_t *pk0, const uint64_t *p1,
                                                   const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    uint32_t *lds32 = (uint32_t *)lds;
    const int tid = threadIdx.x;
    const uint32_t limb = blockIdx.x, L = rc.L;
    const LimbTab tb = load_tab(tabs, limb);
    const uint64_t q = tb.q;
    const typename A::Mod md = A::mod(q, tb.one_s);
    const size_t LN = (size_t)L * ENG::NB, off = (size_t)limb * ENG::NB;
    typename A::elem s[ENG::E], e[ENG::E];
    // secret share: ternary, counter (block, 0, party, SK)
    for (int j = tid; j < ENG::NB / 4; j += ENG::T) {
        int32_t v[4];
        ternary4(philox4x32_10(j, 0, party, counter_tag(DOM_SK, 0, 0), rc.key), v);
#pragma unroll
        for (int i = 0; i < 4; ++i) lds32[4 * j + i] = (uint32_t)v[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) s[k] = A::from_small((int32_t)lds32[ENG::coef_pos(k, tid)], md);
    __syncthreads();
    stage_cbd<ENG>(lds32, tid, DOM_PK_E, party, 0, 0, rc);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) e[k] = A::from_small((int32_t)lds32[ENG::coef_pos(k, tid)], md);
    ENG::forward(s, lds, tid, 0, tb.fwd, md);
    ENG::forward(e, lds, tid, 0, tb.fwd, md);
#pragma unroll
    for (int k = 0; k < ENG::E; ++k) {
        const int pos = ENG::eval_pos(k, tid);
        const uint64_t sv = A::canon_fwd(s[k], md);
        sk[off + pos] = sv;
        sk[LN + off + pos] = shoup_quotient(sv, q);
        const typename A::Key pv = A::key_of(p1[off + pos], p1[LN + off + pos]);
        const uint64_t sum = A::canon_acc(A::mul_key_add(A::from_canon(sv, md), pv, e[k], md), md);      // p1 s + e
        pk0[off + pos] = sum == 0 ? 0 : q - sum;
    }
}

// -------------------------------------------------------------------------------------
// dst = u * key + x, canonical, for the E slots of a thread (evaluation form, one limb).  u comes
// from registers (SRC_REGS: the lazy output of a transform), from raw bits parked at `src`
// (SRC_PARKED: such an output written out earlier; `src` may be `dst` itself) or from canonical
// words at `src` (SRC_CANON: a ciphertext component); x is a transform's lazy output; the key is a
// prepared polynomial (values kp, quotients kps).
// The order of the memory instructions is written out.  A wait for vector memory counts loads and
// stores together, in issue order: a load issued after a store cannot be waited for without also
// waiting for that store to reach memory, and the compiler never moves a load in front of a store
// that might alias it.  So the slots go in batches (sixteen key values and source words at once
// exceed the register budget), and the loads of a batch are issued before the stores of the
// previous one.
// -------------------------------------------------------------------------------------
// NEG (canonical u): dst = x - u * key instead, as x + (q - u) key, so that nothing but the product is added to x: the
// ranges of ArithQ leave no room for more.
enum { SRC_REGS = 0, SRC_PARKED = 1, SRC_CANON = 2 };
template <class ENG, int SRC, bool NEG = false>
D2_DEV void mul_add_store(uint64_t *dst, const uint64_t *kp, const uint64_t *kps, const uint64_t *src,
                          const typename ENG::A::Factor (&u)[ENG::E], const typename ENG::A::elem (&x)[ENG::E], int tl,
                          const typename ENG::A::Mod &md, uint64_t q = 0 /* the modulus, for NEG */)
{
    typedef typename ENG::A A;
    static_assert(!NEG || SRC == SRC_CANON, "q - u");
    constexpr int E = ENG::E, BATCH = E < 8 ? E : 8, NB = E / BATCH;
    const uint32_t lo = 8u * (uint32_t)tl;
    typename A::Key kv[BATCH];
    uint64_t ub[BATCH];
#pragma unroll
    for (int k = 0; k < BATCH; ++k) {
        kv[k] = A::key(kp, kps, lo, 8u * ENG::T * k);
        if constexpr (SRC != SRC_REGS) ub[k] = ld64(src, lo, 8u * ENG::T * k);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        uint64_t r[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const typename A::elem xx = x[b * BATCH + k];
            if constexpr (SRC == SRC_REGS) {
                r[k] = A::canon_acc(A::factor_key_add(u[b * BATCH + k], kv[k], xx, md), md);
            } else {
                typename A::elem uu;
                if constexpr (SRC == SRC_PARKED) uu = from_bits<A>(ub[k]);
                else uu = A::from_canon(NEG ? q - ub[k] : ub[k], md);
                r[k] = A::canon_acc(A::mul_key_add(uu, kv[k], xx, md), md);
            }
        }
        if (b + 1 < NB) {
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                kv[k] = A::key(kp, kps, lo, 8u * ENG::T * ((b + 1) * BATCH + k));
                if constexpr (SRC != SRC_REGS) ub[k] = ld64(src, lo, 8u * ENG::T * ((b + 1) * BATCH + k));
            }
        }
#pragma unroll
        for (int k = 0; k < BATCH; ++k) st64_stream(dst, lo, 8u * ENG::T * (b * BATCH + k), r[k]);
    }
}

// -------------------------------------------------------------------------------------
// BFV.Encrypt in evaluation form.  grid = (C, jobs); one workgroup per ciphertext.
//   c0 = NTT(Lambda m + e0) + NTT(mu) * p0,   c1 = NTT(e1) + NTT(mu) * p1.
// FROM says what a job's source is: plaintext polynomials [C][N], the same in 32-bit words (k_encode_parties), or the
// member's gradient, encoded on the fly.
// -------------------------------------------------------------------------------------
// One component, of the limbs in part `part`.
template <class ENG, int FROM, bool FIRST>
D2_DEV void encrypt_component(uint64_t *lds, const RoundJobs &jobs, uint32_t ct_base, uint32_t split, uint32_t part, uint64_t n_values,
                              const LimbTab *tabs, const RoundConst &rc)
{
    constexpr bool SECOND = !FIRST;
#include "encrypt_body.inc"
}
template <class ENG, int FROM>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_encrypt(RoundJobs jobs, uint32_t ct_base, uint32_t split, uint64_t n_values,
                                                    const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    constexpr bool FIRST = true, SECOND = true;
    const uint32_t part = launch_part();
#include "encrypt_body.inc"
}

// A workgroup for either component, two to a part.  Both make NTT(mu), but only the first encodes the vector and neither does
// three transforms: for launches that leave every workgroup a compute unit of its own.  One workgroup / two: N = 1024, 30 bits,
// 16 indices 7.2 / 5.7 us, N = 4096, 36 bits, 3 limbs, 32 12.1 / 9.5; but 60 of N = 4096 (360 workgroups) 12.2 / 14.8.
// A body for each: both in one, with the component a run-time switch, kept the other's registers (from 54 bits up to 41 spilled, now 16).
// Switch / bodies: N = 8192, 54 bits, 3 limbs, 25 indices 24.2 / 17.8 us, N = 2^14, 54 bits, 40 32.1 / 23.6, N = 1024, 60 bits,
// 4 limbs, 30 10.3 / 7.4;  N = 4096, 60 bits, 2 limbs, 16 12.5 / 13.0, the only ones slower.
template <class ENG, int FROM>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_encrypt_components(RoundJobs jobs, uint32_t ct_base, uint32_t split,
                                                                           uint64_t n_values, const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    const uint32_t z = launch_part();
    if (z & 1u) encrypt_component<ENG, FROM, false>(lds, jobs, ct_base, split, z >> 1, n_values, tabs, rc);
    else encrypt_component<ENG, FROM, true>(lds, jobs, ct_base, split, z >> 1, n_values, tabs, rc);
}

// -------------------------------------------------------------------------------------
// Decryption share h = s c1 + e in evaluation form.  grid = (C, jobs).
// -------------------------------------------------------------------------------------
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_share(RoundJobs jobs, uint32_t ct_base, uint32_t split,
                                                                    const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    uint32_t turn = 0;
    constexpr int E = ENG::E;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x >> ENG::LOGP, blk = blockIdx.x & ((1u << ENG::LOGP) - 1u), L = rc.L;
    const RoundJob job = round_job<(ENG::LOGN != 12 && !(ENG::A::KIND == 0 && ENG::LOGP > 0))>(jobs, blockIdx.y);
    const size_t LN = (size_t)L * ENG::N;
    const uint64_t *sk = (const uint64_t *)job.src;
    const uint64_t *c1 = job.key + ((size_t)c * 2 + 1) * LN;
    uint64_t *out = job.out + (size_t)c * LN;
    SmallPoly<ENG> e;
    static_assert(SMALL_LDS_WORDS<ENG> <= ENG::LDS_WORDS, "in the buffer the first transform leaves alone");
    small_cbd<ENG>(e, lds, tid, DOM_DEC_E, job.party, job.group, ct_base + c, rc);
    if (ENG::WAVE_CHAIN) __syncthreads();
    const LimbRange lr = limb_range(split, L, launch_part());
    // (a fresh counter for every limb or one for all: five members of 256 indices, N = 2^14, 60 bits, three limbs 331 / 317 us, N = 1024, 54 bits,
    // two limbs, 1,024 indices 38.6 / 39.3)
    constexpr bool ONE = ENG::LOGN == 14;
    for (uint32_t l = ONE ? limb_counter<A>(lr.first) : lr.first; l < lr.end; ++l) {
        const uint32_t limb = ONE ? l : limb_counter<A>(l);
        const LimbTab tb = load_tab(tabs, limb);
        const typename A::Mod md = A::mod(tb.q, tb.one_s);
        const size_t off = (size_t)limb * ENG::N;
        const int tl = opaque(tid);
        typename A::elem x[E];
        int32_t sv[ENG::SS][E];
        const typename A::Factor none[E] = {};
        e.get(sv);
        ENG::forward_chained_small(sv, x, lds, turn, tl, blk, tb.fwd, md);
        mul_add_store<ENG, SRC_CANON>(out + off, sk + off, sk + LN + off, c1 + off, none, x, ENG::eval_lane(tl, blk), md);
    }
}

// -------------------------------------------------------------------------------------
// Sums over members.  A sum does not care which thread adds which word, so its loads are of 16 bytes: of two slots whose
// words lie side by side in two lanes (eval_lane), the even lane takes both words of the first, the odd lane those of the
// second, and only the finished sum goes back to its owners.  One compute unit reads 70 bytes/ns from its L2 with 8-byte loads
// and 127 with these, 40 and 49 from memory while half of the units read.
// -------------------------------------------------------------------------------------
template <class ENG>
struct Pairs {
    static constexpr int E = ENG::E, BIT = 1 << ENG::LOGP, B = 8;       // slots go in batches, or more than 8 spill
    static_assert(E % B == 0, "whole batches");
    // byte offset of a thread's two words of slots 0 and 1
    D2_DEV static uint32_t lane(int tid, uint32_t blk)
    {
        return 8u * (uint32_t)(ENG::eval_lane(tid & ~BIT, blk) + (tid & BIT ? ENG::T : 0));
    }
    template <bool STREAM>
    D2_DEV static void load(uint64_t (&v)[B], const uint64_t *p, uint32_t lo, int k0)
    {
#pragma unroll
        for (int k = 0; k < B; k += 2) {
            const U128 w = STREAM ? ld128_stream(p, lo, 8u * ENG::T * (k0 + k)) : ld128(p, lo, 8u * ENG::T * (k0 + k));
            v[k] = w.lo;
            v[k + 1] = w.hi;
        }
    }
    D2_DEV static void store(uint64_t *p, const uint64_t (&v)[B], uint32_t lo, int k0)
    {
#pragma unroll
        for (int k = 0; k < B; k += 2) st128_stream(p, lo, 8u * ENG::T * (k0 + k), U128{v[k], v[k + 1]});
    }
    // v of the other lane of a pair
    D2_DEV static uint32_t other(uint32_t v)
    {
#if D2_GCN_ASM
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, BIT == 1 ? 0xb1 /* quad_perm [1,0,3,2] */ : 0x4e /* [2,3,0,1] */, 0xf,
                                                     0xf, true);
#else
        return (uint32_t)__shfl_xor((int)v, BIT);
#endif
    }
    // from the loaded order to the owners', and back
    D2_DEV static void swap(uint64_t (&v)[B], int tid)
    {
        const bool odd = (tid & BIT) != 0;
#pragma unroll
        for (int k = 0; k < B; k += 2) {
            const uint64_t give = odd ? v[k] : v[k + 1];
            const uint64_t got = ((uint64_t)other(hi32(give)) << 32) | other(lo32(give));
            v[k] = odd ? got : v[k];
            v[k + 1] = odd ? v[k + 1] : got;
        }
    }
    // a sum of K + 1 canonical words made canonical
    D2_DEV static void reduce(uint64_t (&s)[B], uint32_t K, const typename ENG::A::Mod &md, uint64_t q)
    {
        typedef typename ENG::A A;
        if (A::KIND == 0 && K >= (uint32_t)MAX_GROUP) {      // 65 terms: one more than ArithF's sum_end takes
#pragma unroll
            for (int k = 0; k < B; ++k) s[k] = csub(s[k], 32 * q);
        }
#pragma unroll
        for (int k = 0; k < B; ++k) s[k] = A::sum_end(s[k], md);
    }
    // s + the sum of K polynomials, at(j) being the j-th, all canonical and in loaded order (s: up to 65 terms, not reduced
    // where the policy puts that off).  RING: the words of two members are always under way; else those of DEPTH are requested
    // together and then added, for kernels that have no registers for the other.  RING against three together, combine of
    // N = 4096, 36 bits, 3 limbs: 512 indices, two members 41.0 / 40.5 us, twelve 113.6 / 112.2; 400, five 51.5 / 54.1; N = 8192,
    // 54 bits, 4 limbs, 400 of two 112.9 / 120.5 us.
    template <bool STREAM, bool RING, int DEPTH = (ENG::E > 8 ? 2 : 3), class AT>
    D2_DEV static void add(uint64_t (&s)[B], AT at, uint32_t K, uint32_t lo, int k0, uint64_t q)
    {
        typedef typename ENG::A A;
        if constexpr (RING) {
            uint64_t v[2][B];
#pragma unroll
            for (int d = 0; d < 2; ++d)
                if ((uint32_t)d < K) load<STREAM>(v[d], at(d), lo, k0);
            for (uint32_t j = 0; j < K; j += 2) {
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    if (j + d < K) {
#pragma unroll
                        for (int k = 0; k < B; ++k) s[k] = A::sum(s[k], v[d][k], q);
                        if (j + d + 2 < K) load<STREAM>(v[d], at(j + d + 2), lo, k0);
                    }
                }
            }
        } else {
            auto batch = [&](uint32_t j, auto n) {
                constexpr int D = decltype(n)::value;
                uint64_t v[D][B];
#pragma unroll
                for (int d = 0; d < D; ++d) load<STREAM>(v[d], at(j + d), lo, k0);
#pragma unroll
                for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int k = 0; k < B; ++k) s[k] = A::sum(s[k], v[d][k], q);
            };
            uint32_t j = 0;
            for (; j + DEPTH <= K; j += DEPTH) batch(j, std::integral_constant<int, DEPTH>());
            if (DEPTH > 2 && K - j == 2) batch(j, std::integral_constant<int, 2>());
            else if (DEPTH > 1 && j < K) batch(j, std::integral_constant<int, 1>());
        }
    }
};

// -------------------------------------------------------------------------------------
// Combine: y = c0 + sum_k h_k, back to coefficient form, then pt = round(t y / Q) mod t
// by summing t * y_i' / q_i over the limbs with y_i' = y_i (Q/q_i)^-1 mod q_i: integer
// parts exactly, fractional parts in 64-bit fixed point (each term is truncated by less
// than 2^-63, so the rounding is exact unless t y / Q lies within L * 2^-63 of a half-integer).
// SH(j) returns the share buffer of member j.
// COMBINE_CONVERT (MBFV.Convert, Eq. (2)): a share is a pair (h0, h1) [C][2][L][N] and the receiver's
// single-key decryption is folded in: y = c0 + sum h0_k + (sum h1_k) sk (the converted ciphertext drops the
// old c1).  aux: the receiver's prepared secret key.
// COMBINE_DECRYPT (BFV.Decrypt): y = c0 + c1 sk; no shares.  aux as above.
// COMBINE_BOOTSTRAP (MBFV.Bootstrap, Eq. (3)): a share is a pair (eta0, eta1); y = c0 + sum eta0_k is rounded
// to x in R_t, and the refreshed ciphertext (Lambda x + sum eta1_k, alpha) goes to ct_out.
// aux: alpha [C][L][N] in evaluation form.
// -------------------------------------------------------------------------------------
// One limb's term of round(t y / Q) = round(sum_i t y_i' / q_i) with y_i' = y_i (Q/q_i)^-1 mod q_i, which the inverse
// transform delivers (ninvg, wng): y_i' * theta / 2^128 = integer part, next 64 bits = fraction (theta =
// floor(t 2^128 / q_i)); added to the running integer part (kept below t) and 64-bit fraction of a coefficient.
D2_DEV void scale_term(uint64_t yi, const LimbTab &tb, uint32_t t, uint32_t &acc_int, uint64_t &acc_frac)
{
    const uint64_t hi_lo = yi * tb.theta_hi, hi_hi = __umul64hi(yi, tb.theta_hi);
    const uint64_t frac = hi_lo + __umul64hi(yi, tb.theta_lo), nf = acc_frac + frac;
    const uint32_t v = acc_int + (uint32_t)hi_hi + (frac < hi_lo ? 1u : 0u) + (nf < frac ? 1u : 0u);   // <= 2t
    acc_int = v - t < v ? v - t : v;
    acc_frac = nf;
}
// + 1/2, floor, mod t
D2_DEV uint32_t round_mod_t(uint32_t acc_int, uint64_t acc_frac, uint32_t t)
{
    const uint32_t v = acc_int + (uint32_t)(acc_frac >> 63);
    return v >= t ? v - t : v;
}

enum { COMBINE_COLLECTIVE = 0, COMBINE_CONVERT = 1, COMBINE_BOOTSTRAP = 2, COMBINE_REFRESH = 3, COMBINE_DECRYPT = 4 };

// One limb of a refreshed ciphertext from the rounded plaintext, which sits where a forward transform takes its input:
// c0' = NTT(Lambda x) + sum eta1_k, c1' = alpha.  second(j): this limb of the j-th member's eta1.
template <class ENG, class SH>
D2_DEV void refresh_limb(uint64_t *lds, const uint32_t (&m)[ENG::E], int tl, const LimbTab &tb, SH second, uint32_t K,
                         const uint64_t *alpha, uint64_t *c0, uint64_t *c1, bool stream)
{
    typedef typename ENG::A A;
    typedef Pairs<ENG> PR;
    constexpr int E = ENG::E;
    const uint64_t q = tb.q;
    const typename A::Mod md = A::mod(q, tb.one_s);
    const typename A::Twid lam = A::tw(tb.lambda);
    typename A::elem x[E];
#pragma unroll
    for (int k = 0; k < E; ++k) x[k] = A::mul_u32(opaque(m[k]), lam, md);
    ENG::forward(x, lds, tl, 0, tb.fwd, md);
    const uint32_t lp = PR::lane(tl, 0);
#pragma unroll
    for (int k0 = 0; k0 < E; k0 += PR::B) {
        uint64_t v[PR::B];
#pragma unroll
        for (int k = 0; k < PR::B; ++k) v[k] = A::canon_fwd(x[k0 + k], md);
        PR::swap(v, tl);
        if (stream) PR::template add<true, false>(v, second, K, lp, k0, q);
        else PR::template add<false, false>(v, second, K, lp, k0, q);
        PR::reduce(v, K, md, q);
        PR::store(c0, v, lp, k0);
        PR::template load<false>(v, alpha, lp, k0);
        PR::store(c1, v, lp, k0);
    }
}

// FEW: the members' words 8 bytes a lane (see Launch::FEW).
template <class ENG, bool DECODE, int MODE, bool FEW = false, class SH>
D2_DEV void combine_body(uint64_t *lds, const uint64_t *ct, SH share_of, uint32_t K, const uint64_t *aux,
                         uint64_t *pt, float *out, uint64_t n_values, const LimbTab *tabs, const RoundConst &rc)
{
    const uint64_t *skr = aux;
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    const int tid = threadIdx.x;
    // ciphertext indices (and, in the whole-round kernels, jobs) from the last to the first: what the
    // share kernel wrote last is still in the memory-side cache
    const uint32_t c = gridDim.x - 1 - blockIdx.x, L = rc.L;
    const size_t LN = (size_t)L * ENG::NB;
    const size_t share_ct = (MODE == COMBINE_COLLECTIVE ? 1 : 2) * LN;       // words of one share per ciphertext index
    const uint64_t *c0 = ct + (size_t)c * 2 * LN;
    const uint32_t t = (uint32_t)rc.t;
    typedef Pairs<ENG> PR;
    // Shares that fit the caches may still be there, or be wanted again; a launch that fills the chip is faster without
    // leaving them there.  Kept and streamed, N = 4096, 36 bits, 3 limbs, shares read again / made just before: 25 indices of five
    // members (14 MB) 22.0 / 24.8 and 27.5 / 27.8 us, 128 of twelve (156 MB) 35.8 / 44.2 and 48.6 / 47.8, 256 of twelve (312 MB)
    // 64.4 / 61.2 and 72.5 / 65.6; N = 2048, 256 of two (48 MB) 19.8 / 18.3 and 23.4 / 22.5.  With 16 coefficients per thread the
    // second loop spills (N = 2^14, 60 bits, 160 of five with both 129, streamed only 115 us).
    const uint32_t units = gridDim.x * gridDim.y;
    const bool stream = E > 8 || units > 128 || (uint64_t)units * (K + 1) * share_ct > (192u << 20) / 8;
    // (a zero of its own: shared with the limb counter's it would move the counter, and with it every buffer
    // descriptor, to vector registers)
    const uint32_t zero = opaque(0u);
    uint32_t acc_int[E];
    uint64_t acc_frac[E];
#pragma unroll
    for (int k = 0; k < E; ++k) { acc_int[k] = zero; acc_frac[k] = 0; }
    for (uint32_t limb = 0; limb < L; ++limb) {
        const LimbTab tb = load_tab(tabs, limb);
        const uint64_t q = tb.q;
        const typename A::Mod md = A::mod(q, tb.one_s);
        const size_t off = (size_t)limb * ENG::NB;
        const int tl = opaque(tid);
        const uint32_t lo = 8u * (uint32_t)tl, lp = PR::lane(tl, 0);
        auto share = [&](uint32_t j) { return share_of(j) + (size_t)c * share_ct + off; };
        // `from` and a polynomial of every member from the first on, 8 bytes a lane
        auto one_by_one = [&](uint64_t (&s)[E], const uint64_t *from, auto at, uint32_t first) {
#pragma unroll
            for (int k = 0; k < E; ++k) s[k] = ld64_stream(from, lo, 8u * ENG::T * k);
            for (uint32_t j = first; j < K; ++j) {
                uint64_t v[E];
#pragma unroll
                for (int k = 0; k < E; ++k) v[k] = ld64_stream(at(j), lo, 8u * ENG::T * k);
#pragma unroll
                for (int k = 0; k < E; ++k) s[k] = add_mod(s[k], v[k], q);
            }
        };
        // the same in pairs
        auto in_pairs = [&](uint64_t (&s)[E], const uint64_t *from) {
#pragma unroll
            for (int k0 = 0; k0 < E; k0 += PR::B) {
                uint64_t v[PR::B];
                if (from) {                                 // (always; without a branch here the loops of N = 2^14 take 5 % longer)
                    PR::template load<true>(v, from, lp, k0);
                } else {
#pragma unroll
                    for (int k = 0; k < PR::B; ++k) v[k] = 0;
                }
                if (stream) PR::template add<true, (E <= 8)>(v, share, K, lp, k0, q);
                else PR::template add<false, (E <= 8)>(v, share, K, lp, k0, q);
                PR::reduce(v, K, md, q);
                PR::swap(v, tl);
#pragma unroll
                for (int k = 0; k < PR::B; ++k) s[k0 + k] = v[k];
            }
        };
        typename A::elem x[E];
        if constexpr (MODE == COMBINE_DECRYPT) {
            // The ciphertext's words are requested before anything is multiplied: left alone, the compiler spreads the loads over the products to
            // save registers.  Left and requested first, 42 indices, N = 2048, eight limbs of 54 bits (ArithS) 49.2 / 43.5 us.
            // With 16 coefficients per thread they go in batches of eight; there only 32-bit words have registers for more, and ask for two of the
            // keys with them (196 indices of two limbs 54.8 / 51.9 us).
#pragma unroll
            for (int k0 = 0; k0 < E; k0 += 8) {
                uint64_t z[8], y[8];
                typename A::Key kv[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) z[k] = ld64_stream(c0 + LN + off, lo, 8u * ENG::T * (k0 + k));
#pragma unroll
                for (int k = 0; k < 8; ++k) y[k] = ld64_stream(c0 + off, lo, 8u * ENG::T * (k0 + k));
                if constexpr (E <= 8) requested();
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    kv[k] = A::key(skr + off, skr + LN + off, lo, 8u * ENG::T * (k0 + k));
                    if (E > 8 && A::KIND == 3 && k == 1) requested();
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const typename A::elem sum = A::mul_key_add(A::from_canon(z[k], md), kv[k], A::from_canon(y[k], md), md);
                    x[k0 + k] = A::inv_input(A::canon_acc(sum, md), md);
                }
            }
        } else if constexpr (MODE == COMBINE_CONVERT) {
            // Two sums and the keys leave registers for two members at a time, in one loop each (streamed always; three and a second
            // loop spilled).  One at a time where two spill (ArithB, ArithQ below N = 4096) or gain nothing (N = 4096, 36 bits, three limbs, 25
            // indices of 16 receivers 102.2 / 103.6 us); two, N = 2048, 44 bits, two limbs, 60 indices 73.6 / 76.7.  With 16 coefficients per
            // thread there are none left for a second set of addresses: one member, 8 bytes a lane (FEW; the rule for launches that leave most units idle, where
            // spills cost less than narrow loads, is Launch::convert_combine_decode's; four nodes, N = 2^14, 54 bits, eight limbs, 80
            // indices 936 us; the pairs' loads in batches of eight slots 986 with one member and 1,039 with two, of four 1,132).
            auto second = [&](uint32_t j) { return share(j) + LN; };
            constexpr int DEPTH = ENG::LOGN == 12 || (ENG::LOGN < 12 && (A::KIND == 2 || A::KIND == 5)) ? 1 : 2;
            uint64_t y[E], z[E];
            if constexpr (E <= 8) {
                PR::template load<true>(z, second(0), lp, 0);
                PR::template add<true, false, DEPTH>(z, [&](uint32_t j) { return second(j + 1); }, K - 1, lp, 0, q);
                PR::reduce(z, K - 1, md, q);
                PR::swap(z, tl);
                PR::template load<true>(y, c0 + off, lp, 0);
                PR::template add<true, false, DEPTH>(y, share, K, lp, 0, q);
                PR::reduce(y, K, md, q);
                PR::swap(y, tl);
            } else if constexpr (!FEW) {
                auto pairs = [&](uint64_t (&s)[E], const uint64_t *from, auto at, uint32_t n) {
#pragma unroll
                    for (int k0 = 0; k0 < E; k0 += PR::B) {
                        uint64_t v[PR::B];
                        PR::template load<true>(v, from, lp, k0);
                        PR::template add<true, false, DEPTH>(v, at, n, lp, k0, q);
                        PR::reduce(v, n, md, q);
                        PR::swap(v, tl);
#pragma unroll
                        for (int k = 0; k < PR::B; ++k) s[k0 + k] = v[k];
                    }
                };
                pairs(y, c0 + off, share, K);
                pairs(z, second(0), [&](uint32_t j) { return second(j + 1); }, K - 1);
            } else {
                one_by_one(y, c0 + off, share, 0);
                one_by_one(z, second(0), second, 1);
            }
            typename A::Key kv[E];
#pragma unroll
            for (int k = 0; k < E; ++k) kv[k] = A::key(skr + off, skr + LN + off, lo, 8u * ENG::T * k);
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const typename A::elem sum = A::mul_key_add(A::from_canon(z[k], md), kv[k], A::from_canon(y[k], md), md);
                x[k] = A::inv_input(A::canon_acc(sum, md), md);
            }
        } else {
            uint64_t y[E];
            if constexpr (FEW) one_by_one(y, c0 + off, share, 0);
            else in_pairs(y, c0 + off);
#pragma unroll
            for (int k = 0; k < E; ++k) x[k] = A::inv_input(y[k], md);
        }
        ENG::template inverse<true>(x, lds, tl, 0, tb.inv, md, A::tw(tb.ninvg), A::tw(tb.wng));
#pragma unroll
        for (int k = 0; k < E; ++k) scale_term(A::canon_inv(x[k], md), tb, t, acc_int[k], acc_frac[k]);
    }
    uint32_t m[E];
#pragma unroll
    for (int k = 0; k < E; ++k) m[k] = round_mod_t(acc_int[k], acc_frac[k], t);
    if constexpr (MODE == COMBINE_BOOTSTRAP) {
        uint64_t *ct_out = pt + (size_t)c * 2 * LN;
        const uint64_t *alpha = aux + (size_t)c * LN;
        for (uint32_t limb = 0; limb < L; ++limb) {
            const size_t off = (size_t)limb * ENG::NB;
            refresh_limb<ENG>(lds, m, opaque(tid), load_tab(tabs, limb),
                              [&](uint32_t j) { return share_of(j) + (size_t)c * share_ct + LN + off; }, K, alpha + off, ct_out + off,
                              ct_out + LN + off, stream);
        }
    } else if constexpr (MODE == COMBINE_REFRESH) {
        // a copy for the workgroup of every limb, where that will put its c0'
        for (uint32_t limb = 0; limb < L; ++limb) {
            uint32_t *x = (uint32_t *)(pt + (size_t)c * 2 * LN + (size_t)limb * ENG::NB);
#pragma unroll
            for (int k = 0; k < E; ++k) x[ENG::coef_pos(k, tid)] = m[k];
        }
    } else if (DECODE) {
        decode_from_regs<ENG>(m, lds, tid, out, (uint64_t)c * ENG::NB, n_values, load_tab(tabs, L), rc);
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k) pt[(size_t)c * ENG::NB + ENG::coef_pos(k, tid)] = m[k];
    }
}

// one aggregate, K share buffers anywhere in memory, plaintext polynomials out; grid = C
template <class ENG, bool FEW>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_combine(const uint64_t *ct, PtrList shares, uint32_t K, uint64_t *pt,
                                                    const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    combine_body<ENG, false, COMBINE_COLLECTIVE, FEW>(lds, ct, [&](uint32_t j) { return (const uint64_t *)shares.p[j]; }, K,
                                    (const uint64_t *)nullptr, pt, (float *)nullptr, 0, tabs, rc);
}

// whole round: grid = (C, groups); the group's shares lie `stride` words apart; decoded floats out
template <class ENG, bool FEW>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_combine_decode(GroupJobs jobs, size_t stride, uint64_t n_values,
                                                           const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const uint32_t job = gridDim.y - 1 - blockIdx.y;
    const uint64_t *first = jobs.first[job];
    combine_body<ENG, true, COMBINE_COLLECTIVE, FEW>(lds, jobs.ct[job], [&](uint32_t j) { return first + (size_t)j * stride; },
                                   jobs.K[job], (const uint64_t *)nullptr, (uint64_t *)nullptr,
                                   (float *)jobs.out[job], n_values, tabs, rc);
}

// -------------------------------------------------------------------------------------
// Sum, decryption shares, combine and decode of one ciphertext index of one group in one workgroup; grid = (C, groups).
// The separate kernels are bound by memory (sum, combine) or alternate memory and transforms (share), and read
// every aggregate K times and every share once more; here the aggregate's c1 stays in registers for the K shares,
// the shares are added up as they are made, and only what the protocol sends is written.
//   cts: fresh ciphertexts of the first member of the launch's first group, the others ct_words apart; agg and shares:
//   aggregate of the first group, shares of its first member.
// The error samples of a member are drawn once and kept as bytes where its share of the last limb will go.
// Measured (sum + shares + combine, 32 groups of 7, N = 8192, 4 limbs, 153 indices): 10.3 ms as three launches, 7.0 ms
// in one.  The chain of K + 1 transforms per limb in one workgroup needs a full chip: see finish_pays.
// COMBINE = false: the sum and the shares only.  A half of a polynomial can't be transformed back by itself, so N = 2^14
// ends with k_combine_decode (8 nodes, 8 limbs, 684 indices: round 15.33 -> 14.93 ms).
// -------------------------------------------------------------------------------------
template <class ENG, bool COMBINE>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_finish(FinishJobs jobs, const uint64_t *cts, uint64_t *agg,
                                                               uint64_t *shares, size_t ct_words, uint32_t ct_base,
                                                               uint64_t n_values, const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    static_assert(E == 8, "the samples of a thread are kept in SS 8-byte words");
    static_assert(!COMBINE || ENG::LOGP == 0, "the inverse transform takes the whole polynomial");
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    const int tid = threadIdx.x;
    uint32_t turn = 0;
    // from the last to the first: what the encryption wrote last is still in the memory-side cache
    const uint32_t b = gridDim.x - 1 - blockIdx.x, c = b >> ENG::LOGP, blk = b & ((1u << ENG::LOGP) - 1u);
    const uint32_t job = gridDim.y - 1 - blockIdx.y, L = rc.L, t = (uint32_t)rc.t;
    const uint32_t m0 = jobs.first[job], K = jobs.first[job + 1] - m0, group = jobs.group[job];
    const size_t LN = (size_t)L * ENG::N, sh_words = ct_words / 2;
    cts += (size_t)m0 * ct_words + (size_t)c * 2 * LN;
    agg += (size_t)job * ct_words + (size_t)c * 2 * LN;
    shares += (size_t)m0 * sh_words + (size_t)c * LN;
    // (a zero of its own: shared with the limb counter's it would move the counter, and with it every buffer
    // descriptor, to vector registers)
    const uint32_t zero = opaque(0u);
    uint32_t acc_int[E];
    uint64_t acc_frac[E];
#pragma unroll
    for (int k = 0; k < E; ++k) { acc_int[k] = zero; acc_frac[k] = 0; }
    for (uint32_t limb = 0; limb < L; ++limb) {
        const LimbTab tb = load_tab(tabs, limb);
        const uint64_t q = tb.q;
        const typename A::Mod md = A::mod(q, tb.one_s);
        const size_t off = (size_t)limb * ENG::N;
        const uint32_t lo = 8u * (uint32_t)ENG::eval_lane(opaque(tid), blk);
        uint64_t y[E], z[E];                        // sums of c0 (and of the shares) and of c1
        {
            // Three members at once spilled (32-bit words 21 registers, N = 2048, 80 groups' members of 128 indices 557 us; two 536); ArithP has no
            // registers for two either (16 spilled against 8; the same time, 0.2 GB of 34 less for 32 groups of 7, N = 8192, four limbs).  Without
            // the combine (halves of N = 2^14) there is room for three (8 groups of 8, 684 indices, 54 bits, eight limbs: one 5.46 ms, three 5.34).
            constexpr int DEPTH = ENG::LOGP > 0 ? 3 : A::KIND == 4 ? 1 : 2;
            const int tp = opaque(tid);
            const uint32_t lp = Pairs<ENG>::lane(tp, blk);
            auto sum = [&](uint64_t (&s)[E], size_t at) {
                const uint64_t *p = cts + at + off;
                Pairs<ENG>::template load<true>(s, p, lp, 0);
                Pairs<ENG>::template add<true, false, DEPTH>(s, [&](uint32_t j) { return p + (size_t)(j + 1) * ct_words; }, K - 1, lp, 0, q);
#pragma unroll
                for (int k = 0; k < E; ++k) s[k] = A::sum_end(s[k], md);
                Pairs<ENG>::store(agg + at + off, s, lp, 0);
                Pairs<ENG>::swap(s, tp);
            };
            sum(z, LN);
            sum(y, 0);
        }
        for (uint32_t j = 0; j < K; ++j) {
            const uint32_t who = jobs.member[m0 + j];
            uint64_t *share = shares + (size_t)j * sh_words, *kept = share + (size_t)(L - 1) * ENG::N;
            SmallPoly<ENG> e;
            if (limb == 0) {
                // through the buffer that the next transform leaves alone
                small_cbd<ENG>(e, ENG::PINGPONG ? lds + turn * (uint32_t)ENG::LDS_WORDS : lds, opaque(tid), DOM_DEC_E, jobs.party[who], group, ct_base + c, rc);
                if (L > 1) {
#pragma unroll
                    for (int i = 0; i < ENG::SS; ++i)
                        st64(kept, lo, 8u * ENG::T * i, e.word(i));
                }
            } else {
#pragma unroll
                for (int i = 0; i < ENG::SS; ++i) e.set_word(i, ld64(kept, lo, 8u * ENG::T * i));
            }
            int32_t sv[ENG::SS][E];
            e.get(sv);
            typename A::elem x[E];
            ENG::forward_chained_small(sv, x, lds, turn, opaque(tid), blk, tb.fwd, md);
            const uint64_t *sk = jobs.sk[who];
            typename A::Key kv[E];
#pragma unroll
            for (int k = 0; k < E; ++k) kv[k] = A::key(sk + off, sk + LN + off, lo, 8u * ENG::T * k);
            uint64_t h[E];
#pragma unroll
            for (int k = 0; k < E; ++k) h[k] = A::canon_acc(A::mul_key_add(A::from_canon(z[k], md), kv[k], x[k], md), md);
#pragma unroll
            for (int k = 0; k < E; ++k) {
                st64_stream(share + off, lo, 8u * ENG::T * k, h[k]);
                if (COMBINE) y[k] = A::sum(y[k], h[k], q);
            }
            if (COMBINE && j == 31) {                          // a sum never holds more than 33 terms
#pragma unroll
                for (int k = 0; k < E; ++k) y[k] = A::sum_end(y[k], md);
            }
        }
        if constexpr (COMBINE) {
#pragma unroll
            for (int k = 0; k < E; ++k) y[k] = A::sum_end(y[k], md);
            // the inverse side of the table, fetched here so that it is not held in scalar registers across the shares
            const LimbTab ti = load_tab(fresh_table(tabs), limb);
            typename A::elem x[E];
#pragma unroll
            for (int k = 0; k < E; ++k) x[k] = A::inv_input(y[k], md);
            ENG::template inverse<true>(x, ENG::next_buffer(lds, turn), opaque(tid), 0, ti.inv, md, A::tw(ti.ninvg), A::tw(ti.wng));
#pragma unroll
            for (int k = 0; k < E; ++k) scale_term(A::canon_inv(x[k], md), ti, t, acc_int[k], acc_frac[k]);
            if (ENG::WAVE_CHAIN) __syncthreads();       // the next shares' transforms have no barrier of their own
        }
    }
    if constexpr (COMBINE) {
        uint32_t m[E];
#pragma unroll
        for (int k = 0; k < E; ++k) m[k] = round_mod_t(acc_int[k], acc_frac[k], t);
        decode_from_regs<ENG>(m, lds, tid, jobs.out[job], (uint64_t)c * ENG::NB, n_values, load_tab(tabs, L), rc);
    }
}

// -------------------------------------------------------------------------------------
// MBFV.Convert (Sec. 4.2 item 3): key switching of an aggregate to a receiver's own key.
// -------------------------------------------------------------------------------------
// Set-up: a node's own single-key pair (Sec. 3.2 items 1-2).  grid = L.
//   sk (prepared) [2][L][N] = NTT(s), quotients;  pk (prepared) [2][2][L][N] = (p0, quotients,
//   p1, quotients) with p1 = NTT(a), a uniform in R_q, p0 = -(p1 s + e).
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_receiver_keygen(uint32_t party, uint64_t *sk, uint64_t *pk,
                                                            const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    uint32_t *lds32 = (uint32_t *)lds;
    const int tid = threadIdx.x;
    const uint32_t limb = blockIdx.x, L = rc.L;
    const LimbTab tb = load_tab(tabs, limb);
    const uint64_t q = tb.q;
    const typename A::Mod md = A::mod(q, tb.one_s);
    const size_t LN = (size_t)L * ENG::NB, off = (size_t)limb * ENG::NB;
    typename A::elem x[E];
    // secret key: ternary, counter (block, 0, party, RSK)
    for (int j = tid; j < ENG::NB / 4; j += ENG::T) {
        int32_t v[4];
        ternary4(philox4x32_10(j, 0, party, counter_tag(DOM_RSK, 0, 0), rc.key), v);
#pragma unroll
        for (int i = 0; i < 4; ++i) lds32[4 * j + i] = (uint32_t)v[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; ++k) x[k] = A::from_small((int32_t)lds32[ENG::coef_pos(k, tid)], md);
    ENG::forward(x, lds, tid, 0, tb.fwd, md);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int pos = ENG::eval_pos(k, tid);
        const uint64_t sv = A::canon_fwd(x[k], md);
        sk[off + pos] = sv;
        sk[LN + off + pos] = shoup_quotient(sv, q);
    }
    // p1: coefficient n is block n of (RPK_A, limb) reduced mod q
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const uint32_t n = (uint32_t)ENG::coef_pos(k, tid);
        x[k] = A::from_canon(uniform_mod(philox4x32_10(n, 0, party, counter_tag(DOM_RPK_A, limb, 0), rc.key), tb), md);
    }
    ENG::forward(x, lds, tid, 0, tb.fwd, md);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int pos = ENG::eval_pos(k, tid);
        const uint64_t av = A::canon_fwd(x[k], md);
        pk[2 * LN + off + pos] = av;
        pk[3 * LN + off + pos] = shoup_quotient(av, q);
    }
    // error, then p0 = -(p1 s + e) from the values this thread has just stored
    __syncthreads();
    stage_cbd<ENG>(lds32, tid, DOM_RPK_E, party, 0, 0, rc);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; ++k) x[k] = A::from_small((int32_t)lds32[ENG::coef_pos(k, tid)], md);
    ENG::forward(x, lds, tid, 0, tb.fwd, md);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int pos = ENG::eval_pos(k, tid);
        const typename A::Key pv = A::key_of(pk[2 * LN + off + pos], pk[3 * LN + off + pos]);
        const uint64_t sum = A::canon_acc(A::mul_key_add(A::from_canon(sk[off + pos], md), pv, x[k], md), md);      // p1 s + e
        const uint64_t p0 = sum == 0 ? 0 : q - sum;
        pk[off + pos] = p0;
        pk[LN + off + pos] = shoup_quotient(p0, q);
    }
}

// A member's conversion share towards a receiver, Eq. (1), in evaluation form.  grid = (C, jobs).
//   h0 = s_k c1 + NTT(mu) p0_i + NTT(e0),   h1 = NTT(mu) p1_i + NTT(e1)
// mu ternary, e0, e1 from chi, counters (block, ciphertext, member | receiver << 16, domain | group << 16).
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_convert_share(ConvJobs jobs, uint32_t ct_base, uint32_t split,
                                                          const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    typedef typename A::elem elem;
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    uint32_t turn = 0;      // staging uses buffer 0; the transforms then take the two buffers in turn
    uint32_t *lds32 = (uint32_t *)lds;
    constexpr int E = ENG::E;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x >> ENG::LOGP, blk = blockIdx.x & ((1u << ENG::LOGP) - 1u), L = rc.L;
    const ConvJob job = conv_job(jobs, blockIdx.y);
    const size_t LN = (size_t)L * ENG::N;
    const uint64_t *sk = job.sk, *pk = job.pk;
    const uint64_t *c1 = job.ct + ((size_t)c * 2 + 1) * LN;
    uint64_t *out = job.out + (size_t)c * 2 * LN;
    stage_encrypt_samples<ENG>(lds32, tid, DOM_CVT_U, job.who, job.group, ct_base + c, rc);
    __syncthreads();
    SmallTriple<ENG> smp;
    smp.load(lds32, tid);
    if (ENG::WAVE_CHAIN) __syncthreads();   // before a wave's second transform writes where others read samples

    const LimbRange lr = limb_range(split, L, launch_part());
    for (uint32_t l = lr.first; l < lr.end; ++l) {
        const uint32_t limb = limb_counter<A>(l);
        const LimbTab tb = load_tab(tabs, limb);
        const typename A::Mod md = A::mod(tb.q, tb.one_s);
        const size_t off = (size_t)limb * ENG::N;
        const int tl = opaque(tid), el = ENG::eval_lane(tl, blk);
        // as in Encrypt: with 16 coefficients per thread NTT(mu) is parked in the h1 slot of the output
        constexpr bool STASH = E > 8;
        uint64_t *stash = out + LN + off;
        elem u[E];
        int32_t sv[ENG::SS][E];
        smp.template get<0>(sv);
        ENG::forward_chained_small(sv, u, lds, turn, tl, blk, tb.fwd, md);
        if (STASH) {
#pragma unroll
            for (int k = 0; k < E; ++k) st64(stash, 8u * (uint32_t)el, 8u * ENG::T * k, to_bits<A>(u[k]));
        }
        typename A::Factor f[E];
        if (!STASH) {
#pragma unroll
            for (int k = 0; k < E; ++k) f[k] = A::factor(u[k], md);
        }
        elem x[E];
        smp.template get<1>(sv);
        ENG::forward_chained_small(sv, x, lds, turn, opaque(tl), blk, tb.fwd, md);
        // h0: two products per slot, each reduced on its own; first x <- s c1 + x (loads only, eight slots at a time)
        constexpr int BATCH = E < 8 ? E : 8;
#pragma unroll
        for (int k0 = 0; k0 < E; k0 += BATCH) {
            typename A::Key kv[BATCH];
            uint64_t cv[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                kv[k] = A::key(sk + off, sk + LN + off, 8u * (uint32_t)el, 8u * ENG::T * (k0 + k));
                cv[k] = ld64(c1 + off, 8u * (uint32_t)el, 8u * ENG::T * (k0 + k));
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k)
                x[k0 + k] = A::renorm(A::mul_key_add(A::from_canon(cv[k], md), kv[k], x[k0 + k], md), md);
        }
        mul_add_store<ENG, STASH ? SRC_PARKED : SRC_REGS>(out + off, pk + off, pk + LN + off, stash, f, x, el, md);
        smp.template get<2>(sv);
        ENG::forward_chained_small(sv, x, lds, turn, opaque(tl), blk, tb.fwd, md);
        mul_add_store<ENG, STASH ? SRC_PARKED : SRC_REGS>(stash, pk + 2 * LN + off, pk + 3 * LN + off, stash, f, x, el, md);
    }
}

// BFV.Decrypt(sk_i, .) of ciphertexts under a node's own key; grid = C.  Plaintext polynomials out.
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_decrypt(const uint64_t *ct, const uint64_t *skr, uint64_t *pt, const LimbTab *tabs,
                                                    RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    combine_body<ENG, false, COMBINE_DECRYPT>(lds, ct, [](uint32_t) { return (const uint64_t *)nullptr; }, 0, skr, pt, (float *)nullptr,
                                              0, tabs, rc);
}

// The receiver's side of MBFV.Convert fused with BFV.Decrypt(sk_i, .) (Eq. (2)), whole round:
// grid = (C, receivers of all groups); decoded floats out
template <class ENG, bool FEW>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_convert_combine_decode(RecvJobs jobs, size_t stride,
                                                                   uint64_t n_values, const LimbTab *tabs,
                                                                   RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const uint32_t job = gridDim.y - 1 - blockIdx.y;
    const uint64_t *first = jobs.first[job];
    combine_body<ENG, true, COMBINE_CONVERT, FEW>(lds, jobs.ct[job], [&](uint32_t j) { return first + (size_t)j * stride; },
                                  jobs.K[job], jobs.sk[job], (uint64_t *)nullptr, (float *)jobs.out[job],
                                  n_values, tabs, rc);
}

// -------------------------------------------------------------------------------------
// MBFV.Bootstrap (Sec. 4.2 item 4): collective refresh of a ciphertext.
// -------------------------------------------------------------------------------------
// alpha of ciphertext indices ct_base .. ct_base + C - 1 of a group, evaluation form, [C][L][N].
// grid = (C, L).  Coefficient n of limb i = block n of (BS_A, limb i, group) reduced mod q_i.
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_bootstrap_alpha(uint64_t *alpha, uint32_t group, uint32_t ct_base,
                                                            const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x, limb = blockIdx.y, L = rc.L;
    const LimbTab tb = load_tab(tabs, limb);
    const typename A::Mod md = A::mod(tb.q, tb.one_s);
    typename A::elem x[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const uint32_t n = (uint32_t)ENG::coef_pos(k, tid);
        x[k] = A::from_canon(uniform_mod(philox4x32_10(n, ct_base + c, 0, counter_tag(DOM_BS_A, limb, group), rc.key), tb), md);
    }
    ENG::forward(x, lds, tid, 0, tb.fwd, md);
    uint64_t *o = alpha + ((size_t)c * L + limb) * ENG::NB;
#pragma unroll
    for (int k = 0; k < E; ++k) st64(o, 8u * (uint32_t)tid, 8u * ENG::T * k, A::canon_fwd(x[k], md));
}

// A member's refresh share, Eq. (3), in evaluation form.  grid = (C, jobs); jobs.pk holds alpha.
//   eta0 = s_k c1 + NTT(e0 - Lambda M),   eta1 = NTT(Lambda M + e1) - s_k alpha
// M uniform mod t (one block per coefficient), e0, e1 from chi.
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_bootstrap_share(ConvJobs jobs, uint32_t ct_base, uint32_t split,
                                                            const LimbTab *tabs, RoundConst rc)
{
    typedef typename ENG::A A;
    typedef typename A::elem elem;
    __shared__ uint64_t lds[ENG::LDS_CHAIN_WORDS];
    uint32_t turn = 0;      // staging uses buffer 0; the transforms then take the two buffers in turn
    uint32_t *lds32 = (uint32_t *)lds;
    constexpr int E = ENG::E;
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x >> ENG::LOGP, blk = blockIdx.x & ((1u << ENG::LOGP) - 1u), L = rc.L;
    const ConvJob job = conv_job(jobs, blockIdx.y);
    const size_t LN = (size_t)L * ENG::N;
    const uint32_t party = job.who, group = job.group;
    const uint64_t *sk = job.sk;
    const uint64_t *alpha = job.pk + (size_t)c * LN;
    const uint64_t *c1 = job.ct + ((size_t)c * 2 + 1) * LN;
    uint64_t *out = job.out + (size_t)c * 2 * LN;
    // staging: words [0, N) the masks, words [N, 2 N) e0 | e1 << 8 (two's complement bytes)
    const UniformT mask(load_tab(tabs, L));               // the entry of the plaintext modulus
    for (int n = tid; n < ENG::N; n += ENG::T)
        lds32[n] = mask(philox4x32_10(n, ct_base + c, party, counter_tag(DOM_BS_M, 0, group), rc.key));
    for (int j = tid; j < ENG::N / 2; j += ENG::T) {
        int32_t e0[2], e1[2];
        cbd2(philox4x32_10(j, ct_base + c, party, counter_tag(DOM_BS_E0, 0, group), rc.key), rc.eta_mask, e0);
        cbd2(philox4x32_10(j, ct_base + c, party, counter_tag(DOM_BS_E1, 0, group), rc.key), rc.eta_mask, e1);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            lds32[ENG::N + 2 * j + i] = ((uint32_t)e0[i] & 0xffu) | (((uint32_t)e1[i] & 0xffu) << 8);
    }
    __syncthreads();
    static_assert(ENG::N <= ENG::LDS_CHAIN_WORDS, "two words per coefficient");
    // with a fused start (for the shapes that k_encrypt starts its messages so) the two coefficients of every sum, the errors
    // as bytes.  Fused and not: N = 8192, 2 limbs, 900 indices of 36 bits 217 / 173 us; N = 1024, 60 of 30 bits 13.7 / 12.6 us.
    constexpr bool FUSED = ENG::FUSE > 0 && (ENG::LOGP > 0 || A::KIND >= 4);
    constexpr int MS = FUSED ? 2 : 1;
    uint32_t mv[MS][E], ev[MS][E / (FUSED ? 2 : 1)];
#pragma unroll
    for (int j = 0; j < MS; ++j)
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int pos = FUSED ? ENG::encoded_pos(j, k, tid) : ENG::coef_pos(k, tid);
            mv[j][k] = lds32[pos];
            const uint32_t e = lds32[ENG::N + pos];
            if constexpr (!FUSED) ev[j][k] = e;
            else ev[j][k / 2] = k & 1 ? ev[j][k / 2] | e << 16 : e;
        }
    // the transforms overwrite the samples: both buffers hold some, or their transforms have no barrier
    if (2 * ENG::LDS_WORDS < 2 * ENG::N || ENG::WAVE_CHAIN) __syncthreads();
    const LimbRange lr = limb_range(split, L, launch_part());
    for (uint32_t l = lr.first; l < lr.end; ++l) {
        const uint32_t limb = limb_counter<A>(l);
        const LimbTab tb = load_tab(tabs, limb);
        const uint64_t q = tb.q;
        const typename A::Mod md = A::mod(q, tb.one_s);
        const typename A::Twid lam = A::tw(tb.lambda);
        const size_t off = (size_t)limb * ENG::N;
        const int tl = opaque(tid), el = ENG::eval_lane(tl, blk);
        const typename A::Factor none[E] = {};
        elem x[E];
        // coefficient and error `which` of a slot, unpacked where they are used
        auto fetch = [&](int which) {
            return [&, which](int j, int k, uint32_t &m, int32_t &e) {
                m = opaque(mv[j][k]);
                e = FUSED ? sbyte(opaque(ev[j][k / (FUSED ? 2 : 1)]), 2 * (k & 1) + which) : sbyte(opaque(ev[j][k]), which);
            };
        };
        auto transform = [&](auto neg, auto at, int tid0) {
            if constexpr (FUSED) {
                ENG::template forward_chained_encoded<decltype(neg)::value>(at, x, lds, turn, tid0, blk, tb.fwd, lam,
                                                                            A::tw(tb.lambda_i), md);
            } else {
                // the product again for the second transform: kept, its words cost 32 registers across the first (N = 2^14,
                // 2 limbs, 250 indices, ArithS 167 -> 127 us, ArithB 196 -> 152 us)
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    uint32_t m;
                    int32_t e;
                    at(0, k, m, e);
                    const elem v = A::mul_u32(m, lam, md);
                    x[k] = A::add_small(decltype(neg)::value ? A::neg(v, md) : v, e, md);
                }
                ENG::forward_chained(x, lds, turn, tid0, 0, tb.fwd, md);
            }
        };
        transform(std::true_type(), fetch(0), tl);
        mul_add_store<ENG, SRC_CANON>(out + off, sk + off, sk + LN + off, c1 + off, none, x, el, md);
        transform(std::false_type(), fetch(1), opaque(tl));
        // eta1 = Lambda M + e1 - s_k alpha
        mul_add_store<ENG, SRC_CANON, true>(out + LN + off, sk + off, sk + LN + off, alpha + off, none, x, el, md, q);
    }
}

// The receiver's side of MBFV.Bootstrap; grid = C.  ct_out [C][2][L][N].
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_bootstrap_combine(const uint64_t *ct, PtrList shares, uint32_t K,
                                                              const uint64_t *alpha, uint64_t *ct_out,
                                                              const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    combine_body<ENG, false, COMBINE_BOOTSTRAP>(lds, ct, [&](uint32_t j) { return (const uint64_t *)shares.p[j]; }, K,
                                                alpha, ct_out, (float *)nullptr, 0, tabs, rc);
}

// The same in two launches, for batches that leave compute units idle: the sums of eta0 and the rounding, grid = C, then every limb
// of the refreshed ciphertexts by itself, grid = (C, L).  One and two, see the rule in Launch::bootstrap_combine.
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_bootstrap_round(const uint64_t *ct, PtrList shares, uint32_t K,
                                                            uint64_t *ct_out, const LimbTab *tabs, RoundConst rc)
{
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    combine_body<ENG, false, COMBINE_REFRESH>(lds, ct, [&](uint32_t j) { return (const uint64_t *)shares.p[j]; }, K,
                                              (const uint64_t *)nullptr, ct_out, (float *)nullptr, 0, tabs, rc);
}
template <class ENG>
__global__ void __launch_bounds__(ENG::T, ENG::WAVES) k_bootstrap_refresh(PtrList shares, uint32_t K, const uint64_t *alpha,
                                                              uint64_t *ct_out, const LimbTab *tabs, RoundConst rc)
{
    constexpr int E = ENG::E;
    __shared__ uint64_t lds[ENG::LDS_WORDS];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x, limb = blockIdx.y, L = rc.L;
    const size_t LN = (size_t)L * ENG::NB, off = (size_t)limb * ENG::NB, at = (size_t)c * 2 * LN + off;
    uint32_t m[E];
#pragma unroll
    for (int k = 0; k < E; ++k) m[k] = ((const uint32_t *)(ct_out + at))[ENG::coef_pos(k, tid)];
    __syncthreads();                                       // they lie where other threads will store
    refresh_limb<ENG>(lds, m, tid, load_tab(tabs, limb), [&](uint32_t j) { return (const uint64_t *)shares.p[j] + at + LN; }, K,
                      alpha + (size_t)c * LN + off, ct_out + at, ct_out + LN + at, true);
}

}  // namespace d2
