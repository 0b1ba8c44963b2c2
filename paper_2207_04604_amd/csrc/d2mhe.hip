// C-ABI entry points of the d2mhe library (see include/d2mhe.h): parameter validation,
// host-side table construction and kernel launches.  No device memory is allocated here.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "ctx.hpp"
#include "limb_split.hpp"
#include "pm_growth.hpp"
#include "stream_kernels.hpp"

using namespace d2;

namespace {

typedef unsigned __int128 u128;

// ---- host number theory (set-up only) -------------------------------------------------
uint64_t h_mul(uint64_t a, uint64_t b, uint64_t m) { return (uint64_t)((u128)a * b % m); }

uint64_t h_pow(uint64_t base, uint64_t exp, uint64_t m)
{
    uint64_t acc = 1 % m;
    for (base %= m; exp; exp >>= 1, base = h_mul(base, base, m))
        if (exp & 1) acc = h_mul(acc, base, m);
    return acc;
}

uint64_t h_inv(uint64_t a, uint64_t prime) { return h_pow(a, prime - 2, prime); }

// Miller-Rabin with the first twelve primes as witnesses: deterministic below 2^64.
bool h_is_prime(uint64_t n)
{
    const uint64_t wit[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    if (n < 2) return false;
    for (uint64_t p : wit) {
        if (n == p) return true;
        if (n % p == 0) return false;
    }
    int twos = 0;
    uint64_t odd = n - 1;
    while (!(odd & 1)) { odd >>= 1; ++twos; }
    for (uint64_t a : wit) {
        uint64_t y = h_pow(a, odd, n);
        if (y == 1 || y == n - 1) continue;
        bool composite = true;
        for (int i = 1; i < twos && composite; ++i) {
            y = h_mul(y, y, n);
            if (y == n - 1) composite = false;
        }
        if (composite) return false;
    }
    return true;
}

// psi = x^((m-1)/2N) for the smallest x >= 2 such that psi has order exactly 2N.
uint64_t h_root(uint64_t m, uint32_t log2n)
{
    const uint64_t n = 1ull << log2n, e = (m - 1) / (2 * n);
    for (uint64_t x = 2; x < m; ++x) {
        uint64_t psi = h_pow(x, e, m);
        if (h_pow(psi, n, m) == m - 1) return psi;
    }
    return 0;
}

uint64_t h_shoup(uint64_t w, uint64_t m) { return (uint64_t)(((u128)w << 64) / m); }

Tw h_tw(uint64_t w, uint64_t m)
{
    Tw t;
    t.w = w;
    t.ws = h_shoup(w, m);
    return t;
}

uint32_t h_bitrev(uint32_t v, int bits)
{
    uint32_t r = 0;
    for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1u) << (bits - 1 - i);
    return r;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- engine shape per ring degree ----------------------------------------------------------
typedef const EngineOps *(*OpsGetter)();
const OpsGetter OPS_TABLE[6][7] = {
    {ops_f_10, ops_f_11, ops_f_12, ops_f_13, ops_f_14, ops_f_15, ops_f_16},
    {ops_s_10, ops_s_11, ops_s_12, ops_s_13, ops_s_14, ops_s_15, ops_s_16},
    {ops_b_10, ops_b_11, ops_b_12, ops_b_13, ops_b_14, ops_b_15, ops_b_16},
    {ops_w_10, ops_w_11, ops_w_12, ops_w_13, ops_w_14, ops_w_15, ops_w_16},
    {ops_p_10, ops_p_11, ops_p_12, ops_p_13, ops_p_14, ops_p_15, ops_p_16},
    {ops_q_10, ops_q_11, ops_q_12, ops_q_13, ops_q_14, ops_q_15, ops_q_16},
};
constexpr int ARITH_F = 0, ARITH_S = 1, ARITH_B = 2, ARITH_32 = 3, ARITH_P = 4, ARITH_Q = 5;

const EngineOps *engine_ops(const d2mhe_ctx *ctx) { return OPS_TABLE[ctx->arith][ctx->log2n - 10](); }

// Arithmetic back-end from the moduli: 32-bit residues below 2^30, doubles below 2^44 (8 instructions per
// butterfly each); above, moduli just below a power of two take ArithP or ArithQ (9 and 10.5), any
// others the Shoup quotients of ArithS below 2^55 (15) and ArithB (21).
// Transforms modulo the plaintext modulus (< 2^30) always use the 32-bit back-end.
int arith_for(const d2mhe_params *p)
{
    uint64_t qmax = 0;
    bool narrow = true, wide = true;
    for (uint32_t i = 0; i < p->num_limbs; ++i) {
        qmax = p->q[i] > qmax ? p->q[i] : qmax;
        narrow = narrow && pm_growth(p->q[i], false);
        wide = wide && pm_growth(p->q[i], true);
    }
    if (qmax < (1ull << 30)) return ARITH_32;
    if (qmax < (1ull << 44)) return ARITH_F;
    if (narrow) return ARITH_P;
    if (wide) return ARITH_Q;
    if (qmax < (1ull << 55)) return ARITH_S;
    return ARITH_B;
}

// table entry in the format of the back-end
Tw h_entry(int arith, uint64_t w, uint64_t m)
{
    Tw t;
    if (arith == ARITH_F) {
        const double d = (double)w;          // exact: w < 2^44
        std::memcpy(&t.w, &d, sizeof(d));
        t.ws = 0;
    } else if (arith == ARITH_32) {
        t.w = w | ((w << 32) / m) << 32;     // value and floor(w 2^32 / m) in one 8-byte word
        t.ws = 0;
    } else if (arith == ARITH_P || arith == ARITH_Q) {
        const int s = 64 - __builtin_clzll(m) - 31;          // w and w 2^32 mod m, each split at bit s
        const uint64_t low = ((uint64_t)1 << s) - 1, v = (uint64_t)(((u128)w << 32) % m);
        t.w = (w & low) | (w >> s) << 32;
        t.ws = (v & low) | (v >> s) << 32;
    } else {
        t.w = w;
        t.ws = (uint64_t)(((unsigned __int128)w << 63) / m);
    }
    return t;
}

struct Layout {
    size_t tabs_off, tw_off, p1_off, total;
};

Layout layout_of(uint32_t log2n, uint32_t L, bool has_t)
{
    const size_t N = (size_t)1 << log2n;
    const uint32_t moduli = L + (has_t ? 1 : 0);
    Layout lo;
    lo.tabs_off = 0;
    lo.tw_off = align_up(sizeof(LimbTab) * (MAX_LIMBS + 1), 256);
    lo.p1_off = lo.tw_off + (size_t)moduli * 2 * N * sizeof(Tw);
    lo.total = lo.p1_off + (has_t ? (size_t)2 * L * N * sizeof(uint64_t) : 0);
    return lo;
}

bool params_ok(const d2mhe_params *p)
{
    if (!p || !p->q) return false;
    if (p->log2_n < 10 || p->log2_n > 16) return false;
    if (p->num_limbs < 1 || p->num_limbs > (uint32_t)MAX_LIMBS) return false;
    const uint64_t two_n = 2ull << p->log2_n;
    for (uint32_t i = 0; i < p->num_limbs; ++i) {
        const uint64_t q = p->q[i];
        if (q >> 61) return false;
        if (q % two_n != 1 || !h_is_prime(q)) return false;
        for (uint32_t j = 0; j < i; ++j)
            if (p->q[j] == q) return false;
    }
    if (p->t) {
        if (p->t >> 30) return false;
        if (p->t % two_n != 1 || !h_is_prime(p->t)) return false;
        for (uint32_t i = 0; i < p->num_limbs; ++i)
            if (p->t >= p->q[i]) return false;
        if (p->cbd_eta < 1 || p->cbd_eta > 32) return false;
        if (p->frac_bits > 30 || p->max_group < 1) return false;
    }
    return true;
}

}  // namespace

namespace {

bool misaligned(const void *p) { return ((uintptr_t)p & 15u) != 0; }

// the table of a launch for one (party, group) pair
void one_job(RoundJobs &jobs, const void *src, uint32_t party, const uint64_t *key, uint32_t group, uint64_t *out)
{
    jobs.out = out;
    jobs.stride = 0;
    jobs.set_row(0, src, party, key, group);
}

d2mhe_status launch_ntt(d2mhe_ctx *ctx, uint64_t *polys, uint32_t B, bool forward, hipStream_t st)
{
    return engine_ops(ctx)->ntt(ctx, polys, B, forward, st);
}

}  // namespace

// ---- scratch memory of d2mhe_round_group_static ------------------------------------------------
// A device array of the library's own, for callers that may not allocate.  In host code the name
// of a __device__ array is only a stand-in for the symbol, never a device address: its address on
// the current device comes from hipGetSymbolAddress, once per device (every device holds its own
// copy of the array), and only that pointer is ever handed to a kernel or a runtime call.
namespace {

static __device__ __align__(256) uint64_t static_scratch[D2MHE_STATIC_SCRATCH_BYTES / sizeof(uint64_t)];

constexpr int MAX_DEVICES = 64;
std::mutex g_static_lock;
uint64_t *g_static_ptr[MAX_DEVICES];      // address of static_scratch on device i, null until looked up

// Address of the array on the current device (looked up on first use; no allocation).
d2mhe_status static_scratch_ptr(d2mhe_ctx *ctx, uint64_t **out)
{
    int dev = -1;
    D2_HIP(ctx, hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return D2MHE_ERR_RANGE;
    std::lock_guard<std::mutex> hold(g_static_lock);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        D2_HIP(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(static_scratch)));
        if (!p) return D2MHE_ERR_HIP;
        g_static_ptr[dev] = (uint64_t *)p;
    }
    *out = g_static_ptr[dev];
    return D2MHE_OK;
}

}  // namespace

extern "C" {

const char *d2mhe_strerror(d2mhe_status s)
{
    switch (s) {
    case D2MHE_OK: return "ok";
    case D2MHE_ERR_BAD_PARAMS: return "invalid parameters";
    case D2MHE_ERR_NULL: return "null pointer";
    case D2MHE_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case D2MHE_ERR_RANGE: return "index or count out of range";
    case D2MHE_ERR_WORKSPACE: return "workspace or scratch too small";
    case D2MHE_ERR_HIP: return "HIP runtime error";
    case D2MHE_ERR_UNIMPLEMENTED: return "not implemented for these parameters";
    default: return "unknown status";
    }
}

size_t d2mhe_workspace_bytes(const d2mhe_params *p)
{
    if (!params_ok(p)) return 0;
    return layout_of(p->log2_n, p->num_limbs, p->t != 0).total;
}

d2mhe_status d2mhe_create(const d2mhe_params *p, void *dev_workspace, size_t bytes, void *stream,
                          d2mhe_ctx **out)
{
    if (!p || !out) return D2MHE_ERR_NULL;
    *out = nullptr;
    if (!p->q) return D2MHE_ERR_NULL;
    if (!params_ok(p)) return D2MHE_ERR_BAD_PARAMS;
    if (!dev_workspace) return D2MHE_ERR_NULL;
    if (misaligned(dev_workspace)) return D2MHE_ERR_ALIGN;
    const uint32_t L = p->num_limbs, log2n = p->log2_n;
    const size_t N = (size_t)1 << log2n;
    const bool has_t = p->t != 0;
    const Layout lo = layout_of(log2n, L, has_t);
    if (bytes < lo.total) return D2MHE_ERR_WORKSPACE;

    d2mhe_ctx *ctx = new (std::nothrow) d2mhe_ctx();
    if (!ctx) return D2MHE_ERR_HIP;
    ctx->log2n = log2n;
    ctx->L = L;
    ctx->N = N;
    ctx->t = p->t;
    ctx->max_group = p->max_group;
    ctx->arith = arith_for(p);
    ctx->last_hip = 0;
    // Long transforms run as launch pairs over at most 65535 polynomials (grid.y limit).  Smaller
    // chunks (to keep a chunk in the memory-side cache between the two kernels) were measured
    // and bring nothing on MI355X: the strided kernel already runs at copy speed.
    ctx->ntt_chunk_polys = 65535;
    char *ws = (char *)dev_workspace;
    ctx->d_tabs = (const LimbTab *)(ws + lo.tabs_off);
    ctx->d_p1 = has_t ? (uint64_t *)(ws + lo.p1_off) : nullptr;

    const uint32_t moduli = L + (has_t ? 1 : 0);
    std::vector<LimbTab> tabs(MAX_LIMBS + 1);
    std::memset(tabs.data(), 0, sizeof(LimbTab) * tabs.size());
    std::vector<Tw> tw((size_t)moduli * 2 * N);
    std::vector<uint64_t> pw(N);
    uint64_t q_mod_t = 1;
    for (uint32_t i = 0; has_t && i < L; ++i) q_mod_t = h_mul(q_mod_t, p->q[i] % p->t, p->t);
    for (uint32_t i = 0; i < moduli; ++i) {
        // slot L of the table array is the plaintext modulus
        const uint64_t m = i < L ? p->q[i] : p->t;
        const int ar = i < L ? ctx->arith : ARITH_32;      // table format of this modulus
        const uint64_t psi = h_root(m, log2n);
        if (i < L) ctx->q[i] = m;
        ctx->psi[i < L ? i : L] = psi;
        Tw *fwd = tw.data() + (size_t)i * 2 * N, *inv = fwd + N;
        pw[0] = 1;
        for (size_t k = 1; k < N; ++k) pw[k] = h_mul(pw[k - 1], psi, m);
        for (size_t k = 0; k < N; ++k) fwd[k] = h_entry(ar, pw[h_bitrev((uint32_t)k, (int)log2n)], m);
        const uint64_t psi_inv = h_inv(psi, m);
        for (size_t k = 1; k < N; ++k) pw[k] = h_mul(pw[k - 1], psi_inv, m);
        for (size_t k = 0; k < N; ++k) inv[k] = h_entry(ar, pw[h_bitrev((uint32_t)k, (int)log2n)], m);
        LimbTab &tb = tabs[i < L ? i : L];
        tb.q = m;
        if (ar == ARITH_F) {
            const double qinv = 1.0 / (double)m;
            std::memcpy(&tb.one_s, &qinv, sizeof(qinv));
        } else if (ar == ARITH_32) {
            tb.one_s = ((uint64_t)1 << 32) / m;
        } else if (ar == ARITH_P || ar == ARITH_Q) {
            tb.one_s = pm_growth(m, ar == ARITH_Q) * m;
        } else {
            tb.one_s = (uint64_t)(((u128)1 << 63) / m);
        }
        tb.pow64 = h_tw((uint64_t)(((u128)1 << 64) % m), m);
        tb.inv64 = (uint64_t)((((u128)1) << 64) / m);
        const uint64_t ninv = h_inv((uint64_t)N % m, m);
        tb.ninv = h_entry(ar, ninv, m);
        tb.wn = h_entry(ar, h_mul(pw[h_bitrev(1u, (int)log2n)], ninv, m), m);   // inverse twiddle 1 times N^-1
        tb.fwd = (const Tw *)(ws + lo.tw_off) + (size_t)i * 2 * N;
        tb.inv = tb.fwd + N;
        if (i < L && has_t) {
            // floor(Q/t) = (Q - (Q mod t)) / t  and  Q = 0 (mod q_i)  =>  floor(Q/t) = -(Q mod t) t^-1 (mod q_i)
            const uint64_t lam = h_mul((m - q_mod_t % m) % m, h_inv(p->t % m, m), m);
            tb.lambda = h_entry(ar, lam, m);
            tb.lambda_i = h_entry(ar, h_mul(lam, h_pow(psi, N / 2, m), m), m);
            uint64_t others = 1;
            for (uint32_t j = 0; j < L; ++j)
                if (j != i) others = h_mul(others, p->q[j] % m, m);
            const uint64_t gamma = h_inv(others, m);
            tb.ninvg = h_entry(ar, h_mul(ninv, gamma, m), m);
            tb.wng = h_entry(ar, h_mul(h_mul(pw[h_bitrev(1u, (int)log2n)], ninv, m), gamma, m), m);
            const u128 num = (u128)p->t << 64;
            tb.theta_hi = (uint64_t)(num / m);
            tb.theta_lo = (uint64_t)(((num % m) << 64) / m);
        }
    }
    if (has_t && L < (uint32_t)MAX_LIMBS) { /* slot L already filled above */ }

    std::memset(&ctx->rc, 0, sizeof(ctx->rc));
    ctx->rc.t = p->t;
    ctx->rc.L = L;
    ctx->rc.key.k0 = (uint32_t)(p->seed & 0xffffffffu);
    ctx->rc.key.k1 = (uint32_t)(p->seed >> 32);
    if (has_t) {
        ctx->rc.eta_mask = p->cbd_eta >= 32 ? 0xffffffffu : ((1u << p->cbd_eta) - 1u);
        ctx->rc.clamp = (int32_t)(((p->t - 1) / 2) / p->max_group);
        ctx->rc.scale = (float)(1u << p->frac_bits);
        ctx->rc.inv_scale = 1.0f / (float)(1u << p->frac_bits);
    }

    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipMemcpy(ws + lo.tabs_off, tabs.data(), sizeof(LimbTab) * tabs.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(ws + lo.tw_off, tw.data(), tw.size() * sizeof(Tw), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        delete ctx;
        return D2MHE_ERR_HIP;
    }
    if (has_t) {
        // common random polynomial p1: uniform per limb, to evaluation form, with Shoup quotients
        const size_t total = (size_t)L * N;
        hipLaunchKernelGGL(k_uniform, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, ctx->d_p1,
                           ctx->d_tabs, L, log2n, (uint32_t)DOM_CRS, ctx->rc.key, total);
        d2mhe_status s = launch_ntt(ctx, ctx->d_p1, 1, true, st);
        if (s == D2MHE_OK) {
            PtrList src;
            src.p[0] = ctx->d_p1;
            hipLaunchKernelGGL(k_prepare, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, ctx->d_p1, src,
                               1u, ctx->d_tabs, log2n, total);
            if (hipGetLastError() != hipSuccess) s = D2MHE_ERR_HIP;
        }
        if (s == D2MHE_OK && hipStreamSynchronize(st) != hipSuccess) s = D2MHE_ERR_HIP;
        if (s != D2MHE_OK) {
            delete ctx;
            return s;
        }
    }
    // d2mhe_round_group_static's scratch array: look its address up now, with this device current
    uint64_t *own_scratch = nullptr;
    const d2mhe_status ss = static_scratch_ptr(ctx, &own_scratch);
    if (ss != D2MHE_OK) {
        delete ctx;
        return ss;
    }
    *out = ctx;
    return D2MHE_OK;
}

void d2mhe_destroy(d2mhe_ctx *ctx) { delete ctx; }

int d2mhe_last_hip_error(const d2mhe_ctx *ctx) { return ctx ? ctx->last_hip : 0; }

uint64_t d2mhe_root(const d2mhe_ctx *ctx, uint32_t limb)
{
    if (!ctx || limb > ctx->L || (limb == ctx->L && !ctx->t)) return 0;
    return ctx->psi[limb];
}

d2mhe_status d2mhe_ntt_index_map(const d2mhe_ctx *ctx, uint32_t *perm)
{
    if (!ctx || !perm) return D2MHE_ERR_NULL;
    const EngineOps *ops = engine_ops(ctx);
    const int elog = ops->elog, logb = ops->logb;
    const uint32_t T = 1u << (logb - elog), NB = 1u << logb;
    for (uint32_t pos = 0; pos < ctx->N; ++pos) {
        const uint32_t blk = pos >> logb, lp = pos & (NB - 1);
        const uint32_t idx = (blk << logb) | ((lp % T) << elog) | (lp / T);
        perm[pos] = h_bitrev(idx, (int)ctx->log2n);
    }
    return D2MHE_OK;
}

d2mhe_status d2mhe_ntt_forward(d2mhe_ctx *ctx, uint64_t *polys, uint32_t B, void *stream)
{
    if (!ctx || !polys) return D2MHE_ERR_NULL;
    if (misaligned(polys)) return D2MHE_ERR_ALIGN;
    if (B == 0) return D2MHE_OK;
    if ((uint64_t)B * ctx->L > 0x7fffffffull) return D2MHE_ERR_RANGE;
    return launch_ntt(ctx, polys, B, true, (hipStream_t)stream);
}

d2mhe_status d2mhe_ntt_inverse(d2mhe_ctx *ctx, uint64_t *polys, uint32_t B, void *stream)
{
    if (!ctx || !polys) return D2MHE_ERR_NULL;
    if (misaligned(polys)) return D2MHE_ERR_ALIGN;
    if (B == 0) return D2MHE_OK;
    if ((uint64_t)B * ctx->L > 0x7fffffffull) return D2MHE_ERR_RANGE;
    return launch_ntt(ctx, polys, B, false, (hipStream_t)stream);
}

d2mhe_status d2mhe_bench_polys(d2mhe_ctx *ctx, uint64_t *out, uint32_t B, void *stream)
{
    if (!ctx || !out) return D2MHE_ERR_NULL;
    if (misaligned(out)) return D2MHE_ERR_ALIGN;
    if (B == 0) return D2MHE_OK;
    const size_t total = (size_t)B * ctx->L * ctx->N;
    hipLaunchKernelGGL(k_uniform, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, out,
                       ctx->d_tabs, ctx->L, ctx->log2n, (uint32_t)DOM_BENCH, ctx->rc.key, total);
    D2_LAUNCHED(ctx);
    return D2MHE_OK;
}

#define D2_NEED_SCHEME(ctx)                                          \
    do {                                                             \
        if (!(ctx)) return D2MHE_ERR_NULL;                           \
        if (!(ctx)->t) return D2MHE_ERR_BAD_PARAMS;                  \
        if ((ctx)->log2n > 14) return D2MHE_ERR_UNIMPLEMENTED;       \
    } while (0)

d2mhe_status d2mhe_keygen_share(d2mhe_ctx *ctx, uint32_t party, uint64_t *sk_share, uint64_t *pk0_share,
                                void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk_share || !pk0_share) return D2MHE_ERR_NULL;
    if (misaligned(sk_share) || misaligned(pk0_share)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu) return D2MHE_ERR_RANGE;
    return engine_ops(ctx)->keygen(ctx, party, sk_share, pk0_share, (hipStream_t)stream);
}

d2mhe_status d2mhe_aggregate_pk(d2mhe_ctx *ctx, const uint64_t *const *pk0_shares, uint32_t K, uint64_t *pk,
                                void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pk0_shares || !pk) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group) return D2MHE_ERR_RANGE;
    if (misaligned(pk)) return D2MHE_ERR_ALIGN;
    PtrList src;
    for (uint32_t k = 0; k < K; ++k) {
        if (!pk0_shares[k]) return D2MHE_ERR_NULL;
        if (misaligned(pk0_shares[k])) return D2MHE_ERR_ALIGN;
        src.p[k] = pk0_shares[k];
    }
    const size_t total = (size_t)ctx->L * ctx->N;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_prepare, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, pk, src, K, ctx->d_tabs,
                       ctx->log2n, total);
    D2_LAUNCHED(ctx);
    D2_HIP(ctx, hipMemcpyAsync(pk + 2 * total, ctx->d_p1, 2 * total * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    return D2MHE_OK;
}

d2mhe_status d2mhe_encode(d2mhe_ctx *ctx, const float *grad, uint64_t n_values, uint64_t *pt, uint32_t C,
                          void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pt || (!grad && n_values)) return D2MHE_ERR_NULL;
    if (misaligned(pt) || misaligned(grad)) return D2MHE_ERR_ALIGN;
    if (n_values > (uint64_t)C * ctx->N) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    return engine_ops(ctx)->encode(ctx, grad, n_values, pt, C, (hipStream_t)stream);
}

d2mhe_status d2mhe_decode(d2mhe_ctx *ctx, const uint64_t *pt, uint32_t C, uint64_t n_values, float *out,
                          void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pt || (!out && n_values)) return D2MHE_ERR_NULL;
    if (misaligned(pt) || misaligned(out)) return D2MHE_ERR_ALIGN;
    if (n_values > (uint64_t)C * ctx->N) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    return engine_ops(ctx)->decode(ctx, pt, C, n_values, out, (hipStream_t)stream);
}

// Coefficient packing (value j of a ciphertext is coefficient j): the same launchers with the
// packing flag set in a private copy of the context.
d2mhe_status d2mhe_encode_coefficients(d2mhe_ctx *ctx, const float *grad, uint64_t n_values, uint64_t *pt,
                                       uint32_t C, void *stream)
{
    D2_NEED_SCHEME(ctx);
    d2mhe_ctx local = *ctx;
    local.rc.coeff_packing = 1;
    const d2mhe_status s = d2mhe_encode(&local, grad, n_values, pt, C, stream);
    ctx->last_hip = local.last_hip;
    return s;
}

d2mhe_status d2mhe_decode_coefficients(d2mhe_ctx *ctx, const uint64_t *pt, uint32_t C, uint64_t n_values,
                                       float *out, void *stream)
{
    D2_NEED_SCHEME(ctx);
    d2mhe_ctx local = *ctx;
    local.rc.coeff_packing = 1;
    const d2mhe_status s = d2mhe_decode(&local, pt, C, n_values, out, stream);
    ctx->last_hip = local.last_hip;
    return s;
}

d2mhe_status d2mhe_encrypt(d2mhe_ctx *ctx, const uint64_t *pk, const uint64_t *pt, uint32_t C, uint32_t party,
                           uint32_t group, uint32_t ct_base, uint64_t *ct, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pk || !pt || !ct) return D2MHE_ERR_NULL;
    if (misaligned(pk) || misaligned(pt) || misaligned(ct)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu || group > 0xffffu || (uint64_t)ct_base + C > 0xffffffffull) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    RoundJobs jobs;
    one_job(jobs, pt, party, pk, group, ct);
    const bool whole = C == 1 && crosses(ct, 2 * (size_t)ctx->L * ctx->N, pt, ctx->N, 0);
    return engine_ops(ctx)->encrypt(ctx, FROM_WORDS64, jobs, 1, ct_base, 0, C, whole, (hipStream_t)stream);
}

d2mhe_status d2mhe_add(d2mhe_ctx *ctx, uint64_t *ct_acc, const uint64_t *ct_in, uint32_t C, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!ct_acc || !ct_in) return D2MHE_ERR_NULL;
    if (misaligned(ct_acc) || misaligned(ct_in)) return D2MHE_ERR_ALIGN;
    if (C == 0) return D2MHE_OK;
    PtrList src;
    src.p[0] = ct_acc;
    src.p[1] = ct_in;
    const size_t total = (size_t)C * 2 * ctx->L * ctx->N;
    hipLaunchKernelGGL(k_sum, dim3((unsigned)((total / 2 + 255) / 256)), dim3(256), 0, (hipStream_t)stream, ct_acc,
                       src, 2u, ctx->d_tabs, ctx->L, ctx->log2n, total);
    D2_LAUNCHED(ctx);
    return D2MHE_OK;
}

d2mhe_status d2mhe_partial_decrypt(d2mhe_ctx *ctx, const uint64_t *sk_share, const uint64_t *ct, uint32_t C,
                                   uint32_t party, uint32_t group, uint32_t ct_base, uint64_t *share, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk_share || !ct || !share) return D2MHE_ERR_NULL;
    if (misaligned(sk_share) || misaligned(ct) || misaligned(share)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu || group > 0xffffu || (uint64_t)ct_base + C > 0xffffffffull) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    RoundJobs jobs;
    one_job(jobs, sk_share, party, ct, group, share);
    const size_t LN = (size_t)ctx->L * ctx->N;
    const bool whole = C == 1 && crosses(share, LN, ct, 2 * LN, LN);
    return engine_ops(ctx)->share(ctx, jobs, 1, ct_base, C, whole, (hipStream_t)stream);
}

d2mhe_status d2mhe_combine(d2mhe_ctx *ctx, const uint64_t *ct, const uint64_t *const *shares, uint32_t K, uint32_t C,
                           uint64_t *pt, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!ct || !shares || !pt) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group) return D2MHE_ERR_RANGE;
    if (misaligned(ct) || misaligned(pt)) return D2MHE_ERR_ALIGN;
    PtrList sh;
    for (uint32_t k = 0; k < K; ++k) {
        if (!shares[k]) return D2MHE_ERR_NULL;
        if (misaligned(shares[k])) return D2MHE_ERR_ALIGN;
        sh.p[k] = shares[k];
    }
    if (C == 0) return D2MHE_OK;
    return engine_ops(ctx)->combine(ctx, ct, sh, K, C, pt, (hipStream_t)stream);
}

// ---- MBFV.Convert ------------------------------------------------------------------------------

d2mhe_status d2mhe_receiver_keygen(d2mhe_ctx *ctx, uint32_t party, uint64_t *sk, uint64_t *pk, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk || !pk) return D2MHE_ERR_NULL;
    if (misaligned(sk) || misaligned(pk)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu) return D2MHE_ERR_RANGE;
    return engine_ops(ctx)->receiver_keygen(ctx, party, sk, pk, (hipStream_t)stream);
}

d2mhe_status d2mhe_convert_share(d2mhe_ctx *ctx, const uint64_t *sk_share, const uint64_t *pk_recv,
                                 const uint64_t *ct, uint32_t C, uint32_t party, uint32_t receiver, uint32_t group,
                                 uint32_t ct_base, uint64_t *share, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk_share || !pk_recv || !ct || !share) return D2MHE_ERR_NULL;
    if (misaligned(sk_share) || misaligned(pk_recv) || misaligned(ct) || misaligned(share)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu || receiver > 0xffffu || group > 0xffffu || (uint64_t)ct_base + C > 0xffffffffull)
        return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    ConvJobs jobs;
    jobs.out = share;
    jobs.stride = 0;
    jobs.set_row(0, sk_share, party, pk_recv, receiver, ct, group);
    const size_t LN = (size_t)ctx->L * ctx->N;
    const bool whole = C == 1 && crosses(share, 2 * LN, ct, 2 * LN, LN);
    return engine_ops(ctx)->convert_share(ctx, jobs, 1, ct_base, C, whole, (hipStream_t)stream);
}

d2mhe_status d2mhe_convert_combine(d2mhe_ctx *ctx, const uint64_t *ct, const uint64_t *const *shares, uint32_t K,
                                   uint32_t C, uint64_t *ct_out, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!ct || !shares || !ct_out) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group) return D2MHE_ERR_RANGE;
    if (misaligned(ct) || misaligned(ct_out)) return D2MHE_ERR_ALIGN;
    PtrList sh;
    for (uint32_t k = 0; k < K; ++k) {
        if (!shares[k]) return D2MHE_ERR_NULL;
        if (misaligned(shares[k])) return D2MHE_ERR_ALIGN;
        sh.p[k] = shares[k];
    }
    if (C == 0) return D2MHE_OK;
    const size_t LN = (size_t)ctx->L * ctx->N, total = (size_t)C * 2 * LN;
    hipLaunchKernelGGL(k_convert_sum, dim3((unsigned)((total / 2 + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       ct_out, ct, sh, K, ctx->d_tabs, ctx->L, ctx->log2n, LN, total);
    D2_LAUNCHED(ctx);
    return D2MHE_OK;
}

d2mhe_status d2mhe_decrypt(d2mhe_ctx *ctx, const uint64_t *sk, const uint64_t *ct, uint32_t C, uint64_t *pt,
                           void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk || !ct || !pt) return D2MHE_ERR_NULL;
    if (misaligned(sk) || misaligned(ct) || misaligned(pt)) return D2MHE_ERR_ALIGN;
    if (C == 0) return D2MHE_OK;
    return engine_ops(ctx)->decrypt(ctx, ct, sk, C, pt, (hipStream_t)stream);
}

// ---- MBFV.Bootstrap ----------------------------------------------------------------------------

d2mhe_status d2mhe_bootstrap_alpha(d2mhe_ctx *ctx, uint32_t group, uint32_t ct_base, uint32_t C, uint64_t *alpha,
                                   void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!alpha) return D2MHE_ERR_NULL;
    if (misaligned(alpha)) return D2MHE_ERR_ALIGN;
    if (group > 0xffffu || (uint64_t)ct_base + C > 0xffffffffull || C > 0xffffu * 0x10000ull) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    return engine_ops(ctx)->bootstrap_alpha(ctx, group, ct_base, C, alpha, (hipStream_t)stream);
}

d2mhe_status d2mhe_bootstrap_share(d2mhe_ctx *ctx, const uint64_t *sk_share, const uint64_t *ct,
                                   const uint64_t *alpha, uint32_t C, uint32_t party, uint32_t group,
                                   uint32_t ct_base, uint64_t *share, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!sk_share || !ct || !alpha || !share) return D2MHE_ERR_NULL;
    if (misaligned(sk_share) || misaligned(ct) || misaligned(alpha) || misaligned(share)) return D2MHE_ERR_ALIGN;
    if (party > 0xffffu || group > 0xffffu || (uint64_t)ct_base + C > 0xffffffffull) return D2MHE_ERR_RANGE;
    if (C == 0) return D2MHE_OK;
    ConvJobs jobs;
    jobs.out = share;
    jobs.stride = 0;
    jobs.set_row(0, sk_share, party, alpha, 0, ct, group);
    const size_t LN = (size_t)ctx->L * ctx->N;
    const bool whole = C == 1 && (crosses(share, 2 * LN, ct, 2 * LN, LN) || crosses(share, 2 * LN, alpha, LN, LN));
    return engine_ops(ctx)->bootstrap_share(ctx, jobs, 1, ct_base, C, whole, (hipStream_t)stream);
}

d2mhe_status d2mhe_bootstrap_combine(d2mhe_ctx *ctx, const uint64_t *ct, const uint64_t *alpha,
                                     const uint64_t *const *shares, uint32_t K, uint32_t C, uint64_t *ct_out,
                                     void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!ct || !alpha || !shares || !ct_out) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group) return D2MHE_ERR_RANGE;
    if (misaligned(ct) || misaligned(alpha) || misaligned(ct_out)) return D2MHE_ERR_ALIGN;
    PtrList sh;
    for (uint32_t k = 0; k < K; ++k) {
        if (!shares[k]) return D2MHE_ERR_NULL;
        if (misaligned(shares[k])) return D2MHE_ERR_ALIGN;
        sh.p[k] = shares[k];
    }
    if (C == 0) return D2MHE_OK;
    // in two launches the first leaves plaintexts in ct_out: eta1 and alpha are read after that
    const size_t LN = (size_t)ctx->L * ctx->N;
    bool whole = C == 1 && alpha != ct_out + LN && crosses(ct_out, 2 * LN, alpha, LN, 0);
    for (uint32_t k = 0; k < K && C == 1; ++k) whole = whole || (sh.p[k] != ct_out && crosses(ct_out, 2 * LN, sh.p[k], 2 * LN, 0));
    return engine_ops(ctx)->bootstrap_combine(ctx, ct, sh, K, alpha, C, ct_out, whole, (hipStream_t)stream);
}

// ---- the float step of one training iteration (Alg. 2 lines 9-10) -----------------------------

d2mhe_status d2mhe_average_update(const float *sum, uint32_t K, const float *grad, float gamma, uint64_t n,
                                  float *w, void *stream)
{
    if (!sum || !w || (!grad && gamma != 0.0f)) return D2MHE_ERR_NULL;
    if (K == 0) return D2MHE_ERR_RANGE;
    if (n == 0) return D2MHE_OK;
    if (n > 0xffffffffull * 256ull) return D2MHE_ERR_RANGE;
    hipLaunchKernelGGL(k_average_update, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, sum,
                       1.0f / (float)K, grad, gamma, n, w);
    if (hipGetLastError() != hipSuccess) return D2MHE_ERR_HIP;
    return D2MHE_OK;
}

namespace {

// a party listed twice among the (at most MAX_GROUP) members of a group
bool has_duplicates(const uint32_t *members, uint32_t K)
{
    for (uint32_t a = 1; a < K; ++a)
        for (uint32_t b = 0; b < a; ++b)
            if (members[a] == members[b]) return true;
    return false;
}

// words of scratch for J (party, group) jobs, G groups, C ciphertext indices; S conversion shares
// (0: collective decryption, one single-polynomial share per job)
size_t round_words(const d2mhe_ctx *ctx, uint64_t J, uint64_t G, uint64_t S, uint64_t C)
{
    const size_t LN = (size_t)ctx->L * ctx->N;
    const size_t shares = S ? (size_t)S * 2 * LN : (size_t)J * LN;
    return (size_t)C * ((size_t)J * 2 * LN + (size_t)G * 2 * LN + shares);
}

// The different ids of a list in order of their first appearance, and the place of every entry's id among them.  (A
// table by id would cost more than a small round where ids are large.)
struct Places {
    std::vector<uint32_t> ids, place;
    Places(const uint32_t *list, uint32_t n) : place(n)
    {
        int bits = 4;
        while (((uint64_t)1 << bits) < 2 * (uint64_t)n) ++bits;
        std::vector<uint32_t> seen((size_t)1 << bits, 0u);              // 1 + place, open addressing
        for (uint32_t i = 0; i < n; ++i) {
            size_t h = (list[i] * 0x9E3779B1u) >> (32 - bits);
            while (seen[h] && ids[seen[h] - 1] != list[i]) h = (h + 1) & (seen.size() - 1);
            if (!seen[h]) {
                ids.push_back(list[i]);
                seen[h] = (uint32_t)ids.size();
            }
            place[i] = seen[h] - 1;
        }
    }
};

// A round's J jobs in as few launches as their table allows, of equal size.
uint32_t jobs_per_launch(uint32_t J)
{
    const uint32_t launches = (J + RJ_JOBS - 1) / RJ_JOBS;
    return (J + launches - 1) / launches;
}

// The table of a launch over jobs j0, j0 + 1, ..., at most `limit` of them and as far as it holds their parties and
// groups; returns their number (at least one).  src(job) and key(group index): the pointers of a job.  slot: scratch of
// one zero per party (1 + its place in this table).
extern "C++" template <class SRC, class KEY>
uint32_t fill_round_jobs(RoundJobs &jobs, const d2mhe_round_desc *d, const Places &who, uint32_t j0, uint32_t limit,
                         std::vector<uint16_t> &slot, uint64_t *out, size_t stride, SRC src, KEY key)
{
    const uint32_t J = d->group_offsets[d->num_groups];
    const bool rows = J <= (uint32_t)RJ_ROWS;
    uint32_t n = 0, parties = 0, groups = 0, g = 0, listed = d->num_groups;
    std::fill(slot.begin(), slot.end(), (uint16_t)0);
    jobs.out = out;
    jobs.stride = stride;
    for (; n < limit && j0 + n < J; ++n) {
        const uint32_t j = j0 + n, party = d->members[j];
        while (d->group_offsets[g + 1] <= j) ++g;
        const uint32_t id = d->group_ids ? d->group_ids[g] : g;
        if (rows) {
            jobs.set_row(n, src(j), party, key(g), id);
            continue;
        }
        uint16_t &s = slot[who.place[j]];
        if ((g != listed && groups == (uint32_t)RJ_GROUPS) || (!s && parties == (uint32_t)RJ_PARTIES)) break;
        if (g != listed) {
            jobs.set_group(groups++, key(g), id);
            listed = g;
        }
        if (!s) {
            jobs.set_party(parties, src(j), party);
            s = (uint16_t)++parties;
        }
        jobs.set_job(n, s - 1u, groups - 1);
    }
    return n;
}

// The table of a k_finish launch: groups g0, g0 + 1, ..., at most `limit` of them and as far as it holds them; returns
// their number (at least one).  slot: scratch of one zero per party (1 + its place in this table).
uint32_t fill_finish_jobs(FinishJobs &jobs, const d2mhe_round_desc *d, const Places &who, uint32_t g0, uint32_t limit,
                          std::vector<uint16_t> &slot)
{
    static_assert(MAX_GROUP <= FIN_PARTIES && MAX_GROUP <= FIN_MEMBERS, "a group must fit one launch");
    uint32_t n = 0, members = 0, parties = 0;
    std::fill(slot.begin(), slot.end(), (uint16_t)0);
    jobs.first[0] = 0;
    for (; g0 + n < d->num_groups && n < (uint32_t)FIN_GROUPS && n < limit; ++n) {
        const uint32_t g = g0 + n, first = d->group_offsets[g], K = d->group_offsets[g + 1] - first;
        uint32_t fresh = 0;
        for (uint32_t i = 0; i < K; ++i) fresh += slot[who.place[first + i]] == 0;
        if (members + K > (uint32_t)FIN_MEMBERS || parties + fresh > (uint32_t)FIN_PARTIES) break;
        for (uint32_t i = 0; i < K; ++i) {
            uint16_t &s = slot[who.place[first + i]];
            if (!s) {
                const uint32_t party = d->members[first + i];
                jobs.sk[parties] = d->sk_shares[party];
                jobs.party[parties] = (uint16_t)party;
                s = (uint16_t)++parties;
            }
            jobs.member[members + i] = (uint8_t)(s - 1);
        }
        members += K;
        jobs.first[n + 1] = (uint16_t)members;
        jobs.out[n] = d->out_sums[g];
        jobs.group[n] = (uint16_t)(d->group_ids ? d->group_ids[g] : g);
    }
    return n;
}

// Whether a k_finish launch over `groups` groups of `members` members in all is faster than the separate launches.  One
// of its workgroups walks through the K + 1 transforms of every limb of its ciphertext index, so the launch has to fill
// the chip and to leave few units idle at its end: W workgroups take W / 256 turns of the 256 compute units, rounded up.
// How much of the last one may be missing depends on what else a unit has to do: a workgroup of N = 8192 has it for
// itself, two of N = 4096 and four of N = 2048 share it.  With few members the launches saved weigh more.
// Measured (30 to 60 bits, one or two limbs, groups of K = 2 / 4 / 8 to 32), three launches' time over one's:
//   N = 8192   W = 256 1.02-1.09 / 1.05-1.12 / 1.05-1.13,  290 0.98-1.02 / 0.93-0.98 / 0.90-0.96,  350 0.99-1.04 / 0.98-1.02 /
//              0.95-1.00,  384 1.00-1.07 / 0.99-1.05 / 0.99-1.05,  420 1.04-1.06 / 1.01-1.05 / 0.99-1.05,  512 1.05-1.13,
//              576 1.02-1.06 / 1.00-1.04 / 0.98-1.03,  640 and more 1.01-1.12
//   N = 4096   256 1.06-1.15 / 1.03-1.09 / 0.99-1.07,  320 1.01-1.07 / 0.96-0.98 / 0.91-0.96,  384 1.03-1.09 / 1.00-1.04 /
//              0.98-1.03,  400 (K = 5, 36 bits) 1.06,  448 1.06-1.11 / 1.03-1.08 / 1.00-1.06,  512 1.06-1.12 / 1.04-1.09 / 1.03-1.08,
//              576 1.03-1.06 / 0.98-1.02 / 0.94-1.00,  640 and more 1.00-1.12
//   N = 2048   256 1.04-1.16 / 0.99-1.08 / 0.84-1.00,  320 1.00-1.06 / 0.93-0.99 / 0.86-0.93,  372 (K = 3, 44 bits) 1.03,  384
//              1.01-1.08 / 0.97-1.02 / 0.90-0.98,  448 1.06-1.09 / 1.02-1.05 / 0.97-1.04,  512 1.06-1.14 / 1.03-1.09 / 0.99-1.05,
//              576 1.04-1.10 / 0.99-1.06 / 0.94-0.99,  640 and more 0.98-1.15
//   N = 1024   1024 1.09-1.17 / 1.00-1.08 / 0.91-1.01,  1280 1.08-1.14 / 1.05-1.07 / 0.98-1.04,  1536 1.03-1.15 / 1.02-1.07 /
//              0.97-1.04,  1792 1.07-1.12 / 1.04-1.07 / 1.04-1.06
//   N = 2^14   (halves: twice the workgroups; sums and shares only, against a sum and shares in halves or whole, see
//              engine_inst.hpp) eight limbs 256 1.02-1.06, 512 1.02-1.08, 896 1.02-1.05;  four 512 0.96-1.05, 768 1.00-1.05,
//              896 (7/8) 0.97-1.04, 1024 0.99-1.07, 1280 1.04-1.05;  three 512 0.98-1.03, 896 0.96-1.02, 1024 1.01-1.05, 1536
//              1.02-1.05;  one and two 512 0.96-1.02, 1024 0.95-1.01, 1800 0.96-1.01
// One of several such launches (`several`) ends by itself and makes the next one wait, where the separate ones go over all
// groups at once: twice the workgroups, and 7/8 of all turns.  Measured, one kind of launch's time over the other's: 300
// groups of three, N = 2048, five launches of 240 / 360 workgroups 0.91-0.96 / 0.94; N = 4096, five of 240 1.01-1.03; 150 of 17,
// N = 2048, three of 400 0.96-0.98.
bool finish_pays(const d2mhe_ctx *ctx, uint32_t groups, uint32_t members, uint32_t C, bool several)
{
    const bool few = members <= 4 * groups && !several;
    uint64_t W = (uint64_t)groups * C, least;
    uint32_t sixteenths = 12;               // of all turns, to be used by more than that
    switch (ctx->log2n) {
    case 14:
        if (ctx->L < 3) return false;
        W *= 2;
        least = ctx->L >= 8 ? 256 : ctx->L >= 4 ? 512 : 1024;
        break;
    case 13:
        least = 256;
        sixteenths = 11;
        break;
    case 12:
        least = 256;
        if (W <= 512) sixteenths = 11;
        break;
    case 11: least = few ? 256 : 512; break;
    default: least = few ? 1024 : 1792;
    }
    if (few) sixteenths = members <= 3 * groups ? 10 : 11;
    if (several) least *= 2;
    if (several || ctx->log2n == 14) sixteenths = 14;
    return W >= least && 16 * W > sixteenths * 256 * ((W + 255) / 256);
}

// One exchange round; conv == nullptr: collective decryption of every aggregate, otherwise key
// switching to every receiver (MBFV.Convert) and single-key decryption.
d2mhe_status run_round(d2mhe_ctx *ctx, const d2mhe_round_desc *d, const d2mhe_convert_desc *conv, void *scratch,
                       size_t scratch_bytes, void *const *phase_events, void *stream)
{
    if (!d || !scratch) return D2MHE_ERR_NULL;
    if (!d->group_offsets || !d->members || !d->pks || !d->sk_shares || !d->grads) return D2MHE_ERR_NULL;
    if (!conv && !d->out_sums) return D2MHE_ERR_NULL;
    if (conv && (!conv->recv_offsets || !conv->receivers || !conv->recv_pks || !conv->recv_sks || !conv->out_recv))
        return D2MHE_ERR_NULL;
    const uint32_t G = d->num_groups;
    if (G == 0 || G > 0xffffu) return D2MHE_ERR_RANGE;
    if (d->group_offsets[0] != 0) return D2MHE_ERR_RANGE;
    const uint32_t J = d->group_offsets[G];
    for (uint32_t g = 0; g < G; ++g) {
        if (d->group_offsets[g + 1] <= d->group_offsets[g]) return D2MHE_ERR_RANGE;
        const uint32_t K = d->group_offsets[g + 1] - d->group_offsets[g];
        if (K > (uint32_t)MAX_GROUP || K > ctx->max_group) return D2MHE_ERR_RANGE;
        if (!d->pks[g]) return D2MHE_ERR_NULL;
        if (misaligned(d->pks[g])) return D2MHE_ERR_ALIGN;
        if (!conv) {
            if (!d->out_sums[g]) return D2MHE_ERR_NULL;
            if (misaligned(d->out_sums[g])) return D2MHE_ERR_ALIGN;
        }
    }
    // The Philox counters hold 16 bits of group id and of party id, and a (party, group id) pair names one
    // stream of randomness: ids beyond 16 bits, two groups with one id or a member listed twice in a group
    // would make two encryptions share their mu, e0, e1.
    if (d->group_ids) {
        std::vector<uint32_t> ids(d->group_ids, d->group_ids + G);
        std::sort(ids.begin(), ids.end());
        if (ids.back() > 0xffffu) return D2MHE_ERR_RANGE;
        if (std::adjacent_find(ids.begin(), ids.end()) != ids.end()) return D2MHE_ERR_RANGE;
    }
    for (uint32_t g = 0; g < G; ++g)
        if (has_duplicates(d->members + d->group_offsets[g], d->group_offsets[g + 1] - d->group_offsets[g]))
            return D2MHE_ERR_RANGE;
    for (uint32_t j = 0; j < J; ++j) {
        const uint32_t party = d->members[j];
        if (party >= d->num_parties || party > 0xffffu) return D2MHE_ERR_RANGE;
        if (!d->sk_shares[party] || !d->grads[party]) return D2MHE_ERR_NULL;
        if (misaligned(d->sk_shares[party]) || misaligned(d->grads[party])) return D2MHE_ERR_ALIGN;
    }
    uint64_t S = 0;          // conversion shares
    uint32_t R = 0;          // (group, receiver) pairs
    if (conv) {
        if (conv->recv_offsets[0] != 0) return D2MHE_ERR_RANGE;
        for (uint32_t g = 0; g < G; ++g) {
            if (conv->recv_offsets[g + 1] <= conv->recv_offsets[g]) return D2MHE_ERR_RANGE;
            S += (uint64_t)(conv->recv_offsets[g + 1] - conv->recv_offsets[g]) *
                 (d->group_offsets[g + 1] - d->group_offsets[g]);
        }
        R = conv->recv_offsets[G];
        if (S > 0xffffffffull) return D2MHE_ERR_RANGE;
        for (uint32_t r = 0; r < R; ++r) {
            const uint32_t party = conv->receivers[r];
            if (party >= d->num_parties || party > 0xffffu) return D2MHE_ERR_RANGE;
            if (!conv->recv_pks[party] || !conv->recv_sks[party] || !conv->out_recv[r]) return D2MHE_ERR_NULL;
            if (misaligned(conv->recv_pks[party]) || misaligned(conv->recv_sks[party]) || misaligned(conv->out_recv[r]))
                return D2MHE_ERR_ALIGN;
        }
    }
    if (misaligned(scratch)) return D2MHE_ERR_ALIGN;
    if (d->n_values == 0) return D2MHE_OK;
    const uint64_t C64 = (d->n_values + ctx->N - 1) / ctx->N;
    if (C64 > 0x7fffffffull || (uint64_t)d->ct_base + C64 > 0xffffffffull) return D2MHE_ERR_RANGE;
    const uint32_t C = (uint32_t)C64;
    if (scratch_bytes < round_words(ctx, J, G, S, C) * sizeof(uint64_t)) return D2MHE_ERR_WORKSPACE;

    const size_t LN = (size_t)ctx->L * ctx->N;
    const size_t ct_words = (size_t)C * 2 * LN, sh_words = (size_t)C * LN;
    uint64_t *cts = (uint64_t *)scratch;
    uint64_t *agg = cts + (size_t)J * ct_words;
    uint64_t *shares = agg + (size_t)G * ct_words;
    hipStream_t st = (hipStream_t)stream;
    const EngineOps *ops = engine_ops(ctx);
    hipEvent_t *ev = (hipEvent_t *)phase_events;
    if (ev && ev[0]) D2_HIP(ctx, hipEventRecord(ev[0], st));

    // phase 1: every member of every group encodes and encrypts its gradient.  A party in many groups encrypts one
    // vector many times: its plaintexts are then made first, in the space the shares take later, and read from there.
    // Measured, encoded per group and ahead: 32 parties in 7 groups each, N = 8192, 4 limbs 20.2 / 19.1 ms; 16 in 5, N =
    // 4096, 3 limbs 0.391 / 0.375 ms.  Below two groups per party, or where the launches do not fill the chip, the
    // extra launch costs what it saves: N = 2048 with 960 / 1080 / 1920 jobs times indices 0.97-1.00 / 1.00-1.02 / 1.00-1.02 times
    // as fast, N = 1024 with 1600 / 1920 / 2880 0.97-0.99 / 0.96-1.00 / 1.00-1.03.
    const Places who(d->members, J);
    const size_t V = who.ids.size();                     // parties that take part
    std::vector<uint16_t> slot(V);
    const bool ahead = ops->halves || (!ctx->rc.coeff_packing && J >= 2 * V && (uint64_t)J * C >= (ctx->log2n == 10 ? 2560u : 1024u));
    uint32_t *pt = (uint32_t *)shares;
    if (ahead) {
        for (size_t p0 = 0; p0 < V; p0 += ENCODE_CHUNK) {
            const uint32_t n = (uint32_t)std::min(V - p0, (size_t)ENCODE_CHUNK);
            EncodeJobs jobs;
            for (uint32_t i = 0; i < n; ++i) jobs.src[i] = d->grads[who.ids[p0 + i]];
            d2mhe_status s = ops->encode_parties(ctx, jobs, n, d->n_values, pt + p0 * C * ctx->N, C, st);
            if (s != D2MHE_OK) return s;
        }
    }
    const uint32_t per_launch = jobs_per_launch(J);
    for (uint32_t j0 = 0, n; j0 < J; j0 += n) {
        RoundJobs jobs;
        n = fill_round_jobs(jobs, d, who, j0, per_launch, slot, cts + j0 * ct_words, ct_words,
                            [&](uint32_t j) -> const void * {
                                return ahead ? (const void *)(pt + (size_t)who.place[j] * C * ctx->N) : d->grads[d->members[j]];
                            },
                            [&](uint32_t g) { return d->pks[g]; });
        d2mhe_status s = ops->encrypt(ctx, ahead ? FROM_WORDS32 : FROM_VECTOR, jobs, n, d->ct_base, d->n_values, C, false, st);
        if (s != D2MHE_OK) return s;
    }
    if (ev && ev[1]) D2_HIP(ctx, hipEventRecord(ev[1], st));

    // Phases 2 to 4 in one launch, unless the caller wants an event between them: see finish_pays.  Groups that its table
    // does not hold go in several launches of equal size, each of which has to pay by itself.
    const bool split = ev && (ev[2] || ev[3]);
    bool shared = false;            // sums and shares are done
    if (!conv && ops->finish && !split && finish_pays(ctx, G, J, C, false)) {
        FinishJobs jobs;
        uint32_t n = fill_finish_jobs(jobs, d, who, 0, G, slot), launches = 1, limit = G;
        shared = true;
        if (n < G) {
            for (uint32_t g0 = n; g0 < G; ++launches) g0 += fill_finish_jobs(jobs, d, who, g0, G, slot);
            limit = (G + launches - 1) / launches;
            for (uint32_t g0 = 0; shared && g0 < G; g0 += n) {
                n = fill_finish_jobs(jobs, d, who, g0, limit, slot);
                shared = finish_pays(ctx, n, d->group_offsets[g0 + n] - d->group_offsets[g0], C, true);
            }
        }
        for (uint32_t g0 = 0; shared && g0 < G; g0 += n) {
            if (limit < G) n = fill_finish_jobs(jobs, d, who, g0, limit, slot);
            const size_t j0 = d->group_offsets[g0];
            d2mhe_status s = ops->finish(ctx, jobs, n, cts + j0 * ct_words, agg + (size_t)g0 * ct_words,
                                         shares + j0 * sh_words, d->ct_base, C, d->n_values, st);
            if (s != D2MHE_OK) return s;
        }
        if (shared && !ops->halves) {
            if (ev && ev[4]) D2_HIP(ctx, hipEventRecord(ev[4], st));
            return D2MHE_OK;
        }
    }

    // phase 2: homomorphic sum per group
    for (uint32_t g0 = 0; !shared && g0 < G; g0 += JOB_CHUNK) {
        const uint32_t n = G - g0 < (uint32_t)JOB_CHUNK ? G - g0 : (uint32_t)JOB_CHUNK;
        GroupJobs jobs;
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t g = g0 + i;
            jobs.first[i] = cts + (size_t)d->group_offsets[g] * ct_words;
            jobs.ct[i] = nullptr;
            jobs.out[i] = agg + (size_t)g * ct_words;
            jobs.K[i] = d->group_offsets[g + 1] - d->group_offsets[g];
        }
        hipLaunchKernelGGL(k_sum_groups, dim3((unsigned)((ct_words / 2 + 255) / 256), n), dim3(256), 0, st, jobs,
                           ct_words, ctx->d_tabs, ctx->L, ctx->log2n, ct_words);
        D2_LAUNCHED(ctx);
    }
    if (ev && ev[2]) D2_HIP(ctx, hipEventRecord(ev[2], st));

    if (!conv) {
        // phase 3: every member's decryption share of its group's aggregate
        for (uint32_t j0 = 0, n; !shared && j0 < J; j0 += n) {
            RoundJobs jobs;
            n = fill_round_jobs(jobs, d, who, j0, per_launch, slot, shares + j0 * sh_words, sh_words,
                                [&](uint32_t j) -> const void * { return d->sk_shares[d->members[j]]; },
                                [&](uint32_t g) { return agg + (size_t)g * ct_words; });
            d2mhe_status s = ops->share(ctx, jobs, n, d->ct_base, C, false, st);
            if (s != D2MHE_OK) return s;
        }
        if (ev && ev[3]) D2_HIP(ctx, hipEventRecord(ev[3], st));

        // phase 4: combine the shares, round, decode
        for (uint32_t g0 = 0; g0 < G; g0 += JOB_CHUNK) {
            const uint32_t n = G - g0 < (uint32_t)JOB_CHUNK ? G - g0 : (uint32_t)JOB_CHUNK;
            GroupJobs jobs;
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t g = g0 + i;
                jobs.first[i] = shares + (size_t)d->group_offsets[g] * sh_words;
                jobs.ct[i] = agg + (size_t)g * ct_words;
                jobs.out[i] = d->out_sums[g];
                jobs.K[i] = d->group_offsets[g + 1] - d->group_offsets[g];
            }
            d2mhe_status s = ops->combine_decode(ctx, jobs, n, sh_words, C, d->n_values, st);
            if (s != D2MHE_OK) return s;
        }
        if (ev && ev[4]) D2_HIP(ctx, hipEventRecord(ev[4], st));
        return D2MHE_OK;
    }

    // phase 3 (Convert): one share per (group, receiver, member), in that order
    struct ShareRef {
        uint32_t g, r, j;      // group, index into receivers, index into members
    };
    std::vector<ShareRef> refs;
    refs.reserve((size_t)S);
    std::vector<size_t> first_share(R);     // position of the first share of a (group, receiver) pair
    for (uint32_t g = 0; g < G; ++g)
        for (uint32_t r = conv->recv_offsets[g]; r < conv->recv_offsets[g + 1]; ++r) {
            first_share[r] = refs.size();
            for (uint32_t j = d->group_offsets[g]; j < d->group_offsets[g + 1]; ++j) refs.push_back(ShareRef{g, r, j});
        }
    const Places to(conv->receivers, R);
    std::vector<uint16_t> rslot(to.ids.size());          // as slot, for receivers
    const size_t launches = (refs.size() + CJ_JOBS - 1) / CJ_JOBS, limit = (refs.size() + launches - 1) / launches;
    const bool rows = refs.size() <= (size_t)CJ_ROWS;
    for (size_t s0 = 0; s0 < refs.size();) {
        ConvJobs jobs;
        jobs.out = shares + s0 * ct_words;
        jobs.stride = ct_words;
        std::fill(slot.begin(), slot.end(), (uint16_t)0);
        std::fill(rslot.begin(), rslot.end(), (uint16_t)0);
        uint32_t n = 0, members = 0, receivers = 0, groups = 0, listed = G;
        for (; n < limit && s0 + n < refs.size(); ++n) {
            const ShareRef &f = refs[s0 + n];
            const uint32_t member = d->members[f.j], receiver = conv->receivers[f.r];
            const uint32_t id = d->group_ids ? d->group_ids[f.g] : f.g;
            const uint64_t *sk = d->sk_shares[member], *pk = conv->recv_pks[receiver], *ct = agg + (size_t)f.g * ct_words;
            if (rows) {
                jobs.set_row(n, sk, member, pk, receiver, ct, id);
                continue;
            }
            uint16_t &ms = slot[who.place[f.j]], &rs = rslot[to.place[f.r]];
            if ((!ms && members == (uint32_t)CJ_PARTIES) || (!rs && receivers == (uint32_t)CJ_PARTIES) ||
                (f.g != listed && groups == (uint32_t)CJ_GROUPS))
                break;
            if (!ms) {
                jobs.set_member(members, sk, member);
                ms = (uint16_t)++members;
            }
            if (!rs) {
                jobs.set_receiver(receivers, pk, receiver);
                rs = (uint16_t)++receivers;
            }
            if (f.g != listed) {
                jobs.set_group(groups++, ct, id);
                listed = f.g;
            }
            jobs.set_job(n, ms - 1u, rs - 1u, groups - 1);
        }
        d2mhe_status s = ops->convert_share(ctx, jobs, n, d->ct_base, C, false, st);
        if (s != D2MHE_OK) return s;
        s0 += n;
    }
    if (ev && ev[3]) D2_HIP(ctx, hipEventRecord(ev[3], st));

    // phase 4 (Convert): every receiver forms its ciphertext, decrypts with its own key, decodes
    for (uint32_t r0 = 0; r0 < R; r0 += CONV_CHUNK) {
        const uint32_t n = R - r0 < (uint32_t)CONV_CHUNK ? R - r0 : (uint32_t)CONV_CHUNK;
        RecvJobs jobs;
        uint32_t g = 0;
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t r = r0 + i;
            while (conv->recv_offsets[g + 1] <= r) ++g;
            jobs.first[i] = shares + first_share[r] * ct_words;
            jobs.ct[i] = agg + (size_t)g * ct_words;
            jobs.sk[i] = conv->recv_sks[conv->receivers[r]];
            jobs.out[i] = conv->out_recv[r];
            jobs.K[i] = d->group_offsets[g + 1] - d->group_offsets[g];
        }
        d2mhe_status s = ops->convert_combine_decode(ctx, jobs, n, ct_words, C, d->n_values, st);
        if (s != D2MHE_OK) return s;
    }
    if (ev && ev[4]) D2_HIP(ctx, hipEventRecord(ev[4], st));
    return D2MHE_OK;
}

}  // namespace

size_t d2mhe_round_scratch_bytes(const d2mhe_ctx *ctx, uint32_t num_jobs, uint32_t num_groups, uint64_t n_values)
{
    if (!ctx || !ctx->t || num_jobs == 0 || num_groups == 0) return 0;
    const uint64_t C = (n_values + ctx->N - 1) / ctx->N;
    return round_words(ctx, num_jobs, num_groups, 0, C) * sizeof(uint64_t);
}

size_t d2mhe_round_convert_scratch_bytes(const d2mhe_ctx *ctx, uint32_t num_jobs, uint32_t num_groups,
                                         uint32_t num_shares, uint64_t n_values)
{
    if (!ctx || !ctx->t || num_jobs == 0 || num_groups == 0 || num_shares == 0) return 0;
    const uint64_t C = (n_values + ctx->N - 1) / ctx->N;
    return round_words(ctx, num_jobs, num_groups, num_shares, C) * sizeof(uint64_t);
}

// The packing of the round travels in a private copy of the context (the launchers read the
// per-context constants from it).
d2mhe_status run_round_packed(d2mhe_ctx *ctx, const d2mhe_round_desc *d, const d2mhe_convert_desc *conv,
                              void *scratch, size_t scratch_bytes, void *const *phase_events, void *stream)
{
    if (!d) return D2MHE_ERR_NULL;
    if (d->packing > 1) return D2MHE_ERR_RANGE;
    d2mhe_ctx local = *ctx;
    local.rc.coeff_packing = d->packing;
    const d2mhe_status s = run_round(&local, d, conv, scratch, scratch_bytes, phase_events, stream);
    ctx->last_hip = local.last_hip;
    return s;
}

d2mhe_status d2mhe_round(d2mhe_ctx *ctx, const d2mhe_round_desc *d, void *scratch, size_t scratch_bytes,
                         void *const *phase_events, void *stream)
{
    D2_NEED_SCHEME(ctx);
    return run_round_packed(ctx, d, nullptr, scratch, scratch_bytes, phase_events, stream);
}

d2mhe_status d2mhe_round_convert(d2mhe_ctx *ctx, const d2mhe_round_desc *d, const d2mhe_convert_desc *conv,
                                 void *scratch, size_t scratch_bytes, void *const *phase_events, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!conv) return D2MHE_ERR_NULL;
    return run_round_packed(ctx, d, conv, scratch, scratch_bytes, phase_events, stream);
}

d2mhe_status d2mhe_round_group(d2mhe_ctx *ctx, const uint64_t *pk, const uint64_t *const *sk_shares,
                               const float *const *grads, const uint32_t *members, uint32_t K, uint32_t group,
                               uint64_t n_values, float *out_sum, void *scratch, size_t scratch_bytes, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pk || !sk_shares || !grads || !members || !out_sum || !scratch) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group || group > 0xffffu) return D2MHE_ERR_RANGE;
    // a one-group round
    uint32_t offsets[2] = {0, K};
    for (uint32_t k = 0; k < K; ++k)
        if (members[k] > 0xffffu) return D2MHE_ERR_RANGE;
    if (has_duplicates(members, K)) return D2MHE_ERR_RANGE;
    // pointer tables indexed by party id: build sparse views of size max id + 1
    uint32_t max_id = 0;
    for (uint32_t k = 0; k < K; ++k) max_id = members[k] > max_id ? members[k] : max_id;
    std::vector<const uint64_t *> sk_by_party(max_id + 1, nullptr);
    std::vector<const float *> grad_by_party(max_id + 1, nullptr);
    for (uint32_t k = 0; k < K; ++k) {
        sk_by_party[members[k]] = sk_shares[k];
        grad_by_party[members[k]] = grads[k];
    }
    d2mhe_round_desc d;
    d.num_groups = 1;
    d.group_offsets = offsets;
    d.members = members;
    d.group_ids = &group;
    d.pks = &pk;
    d.num_parties = max_id + 1;
    d.sk_shares = sk_by_party.data();
    d.grads = grad_by_party.data();
    d.out_sums = &out_sum;
    d.n_values = n_values;
    d.ct_base = 0;
    d.packing = 0;
    return d2mhe_round(ctx, &d, scratch, scratch_bytes, nullptr, stream);
}

// d2mhe_round_group for callers that may not allocate: the same four launches on the library's own
// scratch array.  Nothing here touches the heap or the device allocator: the job tables are on the
// stack (K <= 64 fits one launch per phase) and travel in the kernel arguments.
d2mhe_status d2mhe_round_group_static(d2mhe_ctx *ctx, const uint64_t *pk, const uint64_t *const *sk_shares,
                                      const float *const *grads, const uint32_t *members, uint32_t K,
                                      uint32_t group, uint64_t n_values, float *out_sum, void *stream)
{
    D2_NEED_SCHEME(ctx);
    if (!pk || !sk_shares || !grads || !members || !out_sum) return D2MHE_ERR_NULL;
    if (K == 0 || K > (uint32_t)MAX_GROUP || K > ctx->max_group || group > 0xffffu) return D2MHE_ERR_RANGE;
    static_assert(MAX_GROUP <= RJ_ROWS && MAX_GROUP <= JOB_CHUNK, "a group must fit one launch");
    if (misaligned(pk) || misaligned(out_sum)) return D2MHE_ERR_ALIGN;
    for (uint32_t k = 0; k < K; ++k) {
        if (members[k] > 0xffffu) return D2MHE_ERR_RANGE;
        if (!sk_shares[k] || !grads[k]) return D2MHE_ERR_NULL;
        if (misaligned(sk_shares[k]) || misaligned(grads[k])) return D2MHE_ERR_ALIGN;
    }
    if (has_duplicates(members, K)) return D2MHE_ERR_RANGE;
    if (n_values == 0) return D2MHE_OK;
    const uint64_t C64 = (n_values + ctx->N - 1) / ctx->N;
    if (C64 > 0x7fffffffull) return D2MHE_ERR_RANGE;
    const uint32_t C = (uint32_t)C64;
    // the limit: the scratch of this round must fit the array
    const size_t LN = (size_t)ctx->L * ctx->N;
    if (C64 > D2MHE_STATIC_SCRATCH_BYTES / sizeof(uint64_t) / ((size_t)(3 * K + 2) * LN)) return D2MHE_ERR_WORKSPACE;
    uint64_t *base = nullptr;
    const d2mhe_status ps = static_scratch_ptr(ctx, &base);       // the device address, never the array's name
    if (ps != D2MHE_OK) return ps;

    const size_t ct_words = (size_t)C * 2 * LN, sh_words = (size_t)C * LN;
    uint64_t *cts = base, *agg = cts + (size_t)K * ct_words, *shares = agg + ct_words;
    hipStream_t st = (hipStream_t)stream;
    const EngineOps *ops = engine_ops(ctx);
    d2mhe_ctx local = *ctx;                  // slot packing, whatever a concurrent call sets in its own copy
    local.rc.coeff_packing = 0;

    RoundJobs enc, shr;
    enc.out = cts;
    enc.stride = ct_words;
    shr.out = shares;
    shr.stride = sh_words;
    uint32_t *pt = (uint32_t *)shares;       // plaintexts made ahead wait in the space of the shares (see run_round)
    for (uint32_t k = 0; k < K; ++k) {
        enc.set_row(k, ops->halves ? (const void *)(pt + (size_t)k * C * ctx->N) : grads[k], members[k], pk, group);
        shr.set_row(k, sk_shares[k], members[k], agg, group);
    }
    d2mhe_status s = D2MHE_OK;
    if (ops->halves) {
        static_assert(MAX_GROUP <= ENCODE_CHUNK, "a group must fit one launch");
        EncodeJobs vectors;
        std::copy(grads, grads + K, vectors.src);
        s = ops->encode_parties(&local, vectors, K, n_values, pt, C, st);
    }
    if (s == D2MHE_OK)
        s = ops->encrypt(&local, ops->halves ? FROM_WORDS32 : FROM_VECTOR, enc, K, 0, n_values, C, false, st);
    if (s == D2MHE_OK) {
        GroupJobs sum;
        sum.first[0] = cts;
        sum.ct[0] = nullptr;
        sum.out[0] = agg;
        sum.K[0] = K;
        hipLaunchKernelGGL(k_sum_groups, dim3((unsigned)((ct_words / 2 + 255) / 256), 1), dim3(256), 0, st, sum,
                           ct_words, ctx->d_tabs, ctx->L, ctx->log2n, ct_words);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            local.last_hip = (int)e;
            s = D2MHE_ERR_HIP;
        }
    }
    if (s == D2MHE_OK) s = ops->share(&local, shr, K, 0, C, false, st);
    if (s == D2MHE_OK) {
        GroupJobs cmb;
        cmb.first[0] = shares;
        cmb.ct[0] = agg;
        cmb.out[0] = out_sum;
        cmb.K[0] = K;
        s = ops->combine_decode(&local, cmb, 1, sh_words, C, n_values, st);
    }
    ctx->last_hip = local.last_hip;
    return s;
}

}  // extern "C"
