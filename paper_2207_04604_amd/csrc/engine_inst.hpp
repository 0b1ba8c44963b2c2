// Launchers for one engine shape; included by inst_<log2n>.hip, which instantiates them.
#pragma once
#include "ctx.hpp"
#include "limb_split.hpp"

namespace d2 {

// HALF: the engine of the kernels that only transform forward, which may take a polynomial in two halves.  N = 2^14 does
// where the policy can take the stage that couples the halves as a sum of samples: with 16 coefficients per thread one
// workgroup filled a CU without room for a second exchange buffer (two barriers per transform, NTT(mu) parked in memory)
// and kept the vector ALU busy 55 % of the time.  Measured, 8 nodes, 8 limbs, 684 indices: 16.83 -> 15.40 ms.
//
// Either half draws all samples of its polynomial, which costs most where a kernel does little else, and n polynomials
// take turns(2n) turns of half workgroups on the chip instead of turns(n) of whole ones.  Measured, us for whole / halves
// (54 bits unless stated; one kernel):
//   n = 60 (one turn of either)  encrypt 52 / 29, share 19.5 / 14.1, conversion 53 / 32, refresh 56 / 45 with one limb;
//                                172 / 86, 64 / 39, 181 / 96, 147 / 100 with four
//   n = 300 (two and three)      encrypt 113 / 88, 397 / 256;  share 42.4 / 41.4, 156 / 114;  refresh 116 / 133, 338 / 325
//   n = 160 (one and two)        share 20.3 / 26.7, 65 / 75;  refresh 57 / 88, 150 / 196;  encrypt 55 / 59, 176 / 167
//   n = 900 (four and eight)     share 88 / 106, 328 / 344;  refresh 237 / 349, 749 / 875;  encrypt 238 / 233, 811 / 702
//   36 bits, eight limbs         share 148 / 133 (n = 160), 276 / 225 (300);  refresh 338 / 412 (160), 684 / 850 (400)
//   44 bits, one limb            encrypt 52 / 58 (160), 212 / 223 (900), 103 / 86 (300);  conversion 55 / 60, 234 / 235
template <class ENG, class HALF = ENG>
struct Launch {
    static constexpr bool HALVES = HALF::LOGP > 0;
    static uint64_t turns(uint64_t workgroups) { return (workgroups + 255) / 256; }
    // the turns of halves take less time than those of whole polynomials, a turn of halves being two thirds as long
    static bool turns_pay(uint64_t n) { return 2 * turns(2 * n) <= 3 * turns(n); }
    static bool encrypt_in_halves(const d2mhe_ctx *ctx, uint64_t n) { return ENG::A::KIND != 0 || ctx->L > 1 || turns_pay(n); }
    // Where the last turn of whole polynomials is at most half full, halves save half of it: with limbs enough that is
    // more than the samples drawn twice cost.  Measured shares, us for whole / halves, n = 520 (three turns and five),
    // 780 (four, seven), 1040 (five, nine), 1300 (six, eleven):
    //   36 bits  two limbs 106 / 103, 154 / 144, 198 / 187, 242 / 246;
    //            three limbs 148 / 141, 226 / 221, 290 / 293, 346 / 356;  four 219 / 186, 299 / 285, 377 / 366, 455 / 448;
    //            seven 378 / 333, 508 / 480, 637 / 602, 765 / 734
    //   54 bits  two limbs 107 / 108, 141 / 150, 182 / 196, 239 / 261;  four 205 / 196, 304 / 297, 391 / 390, 472 / 469;
    //            six 339 / 308, 455 / 436, 583 / 548, 688 / 689
    // and with that turn fuller, n = 660, seven limbs of 36 bits: 388 / 400.
    static bool share_in_halves(const d2mhe_ctx *ctx, uint64_t n)
    {
        const uint64_t most = ctx->L > 3 ? UINT64_MAX : ctx->L == 3 ? 4 : ctx->L == 2 && ENG::A::KIND == 0 ? 5 : 0;
        return ctx->L >= 8 || turns_pay(n) || (turns(2 * n) < 2 * turns(n) && turns(n) <= most);
    }
    static bool refresh_in_halves(uint64_t n) { return turns(2 * n) == 1; }
    template <class E>
    struct Shape {
        typedef E type;
    };
    // What every part of a split polynomial repeats, in limbs: the samples (all of them for either half of a polynomial),
    // for an encryption of a vector also its encoding.  Fitted to the choices that are fastest, as the model leaves out what else a part costs:
    // by itself the fixed work is less (256 indices of N = 8192, one to four limbs: refresh shares 27.4, 46.1, 62.6, 80.5 us, decryption shares
    // 11.8, 21.5, 28.4, 36.0; a launch 2.5), but with 0.15 limbs shares take up to 15 % longer, refresh shares 24 %.  Time of 28 shapes
    // (54 and 36 bits, N = 1024 to 2^14, two to eight limbs, 40 to 1,500 indices) with 0.15, 0.3, 0.4, 0.5, 0.7 against 0.5 (refresh shares 0.7):
    // shares 1.010, 1.002, 0.996, 1.000, 1.004;  encryptions 1.003, 0.997, 0.994, 0.993, 1.002;  conversion shares 0.993, 0.992, 0.993, 0.995,
    // 1.004;  refresh shares 1.032, 1.014, 0.996, 0.996, 0.997;  two runs with the same value differ by 0.7 %.
    static constexpr float SAMPLES = 0.5f, ENCODING = 0.7f, MASKS = 0.7f;
    template <class E>
    static LimbSplit split(const d2mhe_ctx *ctx, uint64_t n, float fixed, bool whole)
    {
        if (whole) return LimbSplit{1, ctx->L};
        return split_limbs(ctx->L, n << E::LOGP, 1024 / E::T, E::LOGP ? 2 * fixed : fixed);
    }
    // launch(Shape<engine>) with the one to take
    template <bool BOTH, class F>
    static void choose(bool half, F launch)
    {
        if constexpr (BOTH) {
            if (half) launch(Shape<HALF>());
            else launch(Shape<ENG>());
        } else {
            launch(Shape<HALF>());
        }
    }

    // Members that a workgroup of the tail takes in turn, for `groups` groups of B.  The twiddles it fetches first cost about two
    // members' time; the workgroups take ceil(W / places) turns of the chip, and where there are more than two, W / places + 1/2 as they
    // drift apart (L = 15, B = 37, inverse: sevens, 1,440 workgroups, 225 us, eights, 1,200, 222).  Always eight and this, N = 2^16, 60 bits, us:
    // L = 1, B = 8 32.6 / 12.8;  4, 8 43.9 / 27.8;  4, 16 41.0 / 31.3;  4, 24 46.7 / 41.7;  16, 2 26.0 / 25.5;  N = 2^15, 60 bits:
    // 1, 32 36.0 / 16.2;  4, 16 37.9 / 21.2;  7, 48 75.8 / 67.8.  More than eight gain where they fill a turn of the chip, of N =
    // 2^16 also two, if all are equal (L = 16: B = 32 194 / 176, 48 286 / 273, 64 398 / 383; in part of two, L = 4, B = 200 305 / 317; N = 2^15, L = 16,
    // B = 128 397 / 420).  What nearly fills two turns otherwise (L = 14, B = 64;  L = 16, B = 62) was not measured and stays with eights.
    static uint32_t tail_tiles(uint32_t groups, uint32_t B)
    {
        constexpr uint64_t PLACES = 256 * (1024 / ENG::T);
        uint32_t best = 1;
        uint64_t least = ~(uint64_t)0;
        for (uint32_t m = 1; m <= 16 && m <= B; ++m) {
            const uint64_t W = (uint64_t)groups * ((B + m - 1) / m), n = (W + PLACES - 1) / PLACES;
            if (m > 8 && n > 1 && !(ENG::LOGN == 16 && n == 2 && B % m == 0 && 16 * W >= 15 * 2 * PLACES)) continue;
            const uint64_t time = (n > 2 ? 2 * W + PLACES : 2 * n * PLACES) * (m + 2);
            if (time <= least) {
                least = time;
                best = m;
            }
        }
        return best;
    }

    static d2mhe_status ntt(d2mhe_ctx *ctx, uint64_t *polys, uint32_t B, bool forward, hipStream_t st)
    {
        const uint32_t L = ctx->L, polys_n = B * L;
        if constexpr (ENG::LOGB == ENG::LOGN) {
            // One workgroup to a compute unit: N = 8192 with multiplicands of four registers (more than 64 registers to a
            // thread), N = 2^14 always, where those of two leave room for the next polynomial.  One by one and walking, us, 537 MB and
            // 134 MB:  N = 8192, 54 bits forward 278 / 261, 68.4 / 61.4, inverse 385 / 336, 85 / 79;  60 bits 302 / 298, 73.4 / 70.3,
            // 405 / 345, 90 / 81;  N = 2^14, 36 bits 278 / 254, 71.7 / 60.6, 344 / 326, 86 / 76;  30 bits 267 / 245, 67.6 / 56.4,
            // 415 / 289, 80 / 67.  Two to a unit (N = 8192, 36 bits) 261 / 266, 254 / 314; spilling (N = 2^14, 54 bits) 288 / 365, 360 / 449.
            // Forward transforms with Shoup quotients gain nothing (54 bits, 300 polynomials 19.4 / 19.2, 420 20.3 / 21.2; inverse 25.9 /
            // 24.3, 27.5 / 26.6).  What walking costs within the same turns: forward, N = 8192, seven limbs, batch of 60 3 %.
            // A workgroup keeps its limb, so up to eight units stay idle, and just below a multiple of 256 polynomials that takes
            // a turn more, which only many turns make up for.  One by one / walking, seven limbs, N = 8192 54 bits inverse, 60 bits forward,
            // N = 2^14 36 bits forward and inverse, batch of
            //   73 (two turns / three) 24.0 / 30.6, 21.2 / 25.4, 37.8 / 42.8, 46.4 / 55.4;  109 35.6 / 40.3, 30.5 / 32.0, 55.5 / 56.0, 68.2 / 73.6
            //   145 (four / five) 47.0 / 50.7, 39.3 / 41.2, 73.0 / 68.8, 90.0 / 91.0;  182 57.8 / 60.3, 49.0 / 51.0, 91.5 / 84.1, 111.6 / 109.4
            //   218 (six / seven) 68.1 / 69.6, 58.2 / 57.8;  254 77.8 / 78.2, 65.3 / 65.4;  292 (eight / nine) 87.6 / 87.0, 72.8 / 70.8
            constexpr bool WALK_INV = (ENG::LOGN == 13 && sizeof(typename ENG::Twid) > 8) || (ENG::LOGN == 14 && sizeof(typename ENG::Twid) <= 8);
            constexpr bool WALK_FWD = WALK_INV && (ENG::LOGN == 14 || ENG::A::KIND >= 4);
            constexpr uint32_t MAKE_UP = ENG::LOGN == 14 ? 4 : 7;      // turns of 256
            const uint32_t grid = 256 / L * L, full = (polys_n + 255) / 256;
            const bool walks = polys_n > 256 && (full >= MAKE_UP || (polys_n + grid - 1) / grid == full);
            const dim3 walk(grid), block(ENG::T);
            if constexpr (WALK_FWD) {
                if (forward && walks) {
                    hipLaunchKernelGGL((k_ntt_walk<ENG, false>), walk, block, 0, st, polys, ctx->d_tabs, L, polys_n);
                    D2_LAUNCHED(ctx);
                    return D2MHE_OK;
                }
            }
            if constexpr (WALK_INV) {
                if (!forward && walks) {
                    hipLaunchKernelGGL((k_ntt_walk<ENG, true>), walk, block, 0, st, polys, ctx->d_tabs, L, polys_n);
                    D2_LAUNCHED(ctx);
                    return D2MHE_OK;
                }
            }
            if (forward)
                hipLaunchKernelGGL(k_ntt_forward<ENG>, dim3(polys_n), block, 0, st, polys, ctx->d_tabs, L);
            else
                hipLaunchKernelGGL(k_ntt_inverse<ENG>, dim3(polys_n), block, 0, st, polys, ctx->d_tabs, L);
            D2_LAUNCHED(ctx);
        } else {
            // head: top stages across blocks; tail: the block-local stages.  The batch is walked in
            // chunks of whole batches that fit the second grid dimension of the head kernel.
            constexpr int LOGN = ENG::LOGN, LOGH = LOGN - ENG::LOGB;
            const uint32_t chunk_b = ctx->ntt_chunk_polys / L ? ctx->ntt_chunk_polys / L : 1;
            for (uint32_t b0 = 0; b0 < B; b0 += chunk_b) {
                const uint32_t nb = B - b0 < chunk_b ? B - b0 : chunk_b, n = nb * L;
                uint64_t *base = polys + ((size_t)b0 * L << LOGN);
                dim3 hgrid((1u << (LOGN - LOGH)) / 256, n);
                const uint32_t tiles = tail_tiles(L << LOGH, nb);
                const uint32_t wpg = (nb + tiles - 1) / tiles;
                dim3 tgrid(L * (1u << LOGH) * wpg);
                if (forward) {
                    hipLaunchKernelGGL((k_head_forward<typename ENG::A, LOGN, LOGH>), hgrid, dim3(256), 0, st, base,
                                       ctx->d_tabs, L, 0u);
                    D2_LAUNCHED(ctx);
                    hipLaunchKernelGGL(k_tail_forward<ENG>, tgrid, dim3(ENG::T), 0, st, base, ctx->d_tabs, L, nb, tiles, wpg);
                } else {
                    hipLaunchKernelGGL(k_tail_inverse<ENG>, tgrid, dim3(ENG::T), 0, st, base, ctx->d_tabs, L, nb, tiles, wpg);
                    D2_LAUNCHED(ctx);
                    hipLaunchKernelGGL((k_head_inverse<typename ENG::A, LOGN, LOGH>), hgrid, dim3(256), 0, st, base,
                                       ctx->d_tabs, L, 0u);
                }
                D2_LAUNCHED(ctx);
            }
        }
        return D2MHE_OK;
    }

    static d2mhe_status keygen(d2mhe_ctx *ctx, uint32_t party, uint64_t *sk, uint64_t *pk0, hipStream_t st)
    {
        hipLaunchKernelGGL(k_keygen<ENG>, dim3(ctx->L), dim3(ENG::T), 0, st, party, sk, pk0,
                           (const uint64_t *)ctx->d_p1, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status encode(d2mhe_ctx *ctx, const float *grad, uint64_t n_values, uint64_t *pt, uint32_t C,
                               hipStream_t st)
    {
        hipLaunchKernelGGL(k_encode<ENG>, dim3(C), dim3(ENG::T), 0, st, grad, n_values, pt, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status encode_parties(d2mhe_ctx *ctx, const EncodeJobs &jobs, uint32_t nparties, uint64_t n_values,
                                       uint32_t *pt, uint32_t C, hipStream_t st)
    {
        hipLaunchKernelGGL(k_encode_parties<ENG>, dim3(C, nparties), dim3(ENG::T), 0, st, jobs, n_values, pt, ctx->d_tabs,
                           ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status decode(d2mhe_ctx *ctx, const uint64_t *pt, uint32_t C, uint64_t n_values, float *out,
                               hipStream_t st)
    {
        hipLaunchKernelGGL(k_decode<ENG>, dim3(C), dim3(ENG::T), 0, st, pt, n_values, out, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    template <class E, int FROM>
    static void launch_encrypt(d2mhe_ctx *ctx, const RoundJobs &jobs, uint32_t njobs, uint32_t ct_base, uint64_t n_values, uint32_t C,
                               float fixed, bool whole, hipStream_t st)
    {
        const uint64_t n = (uint64_t)C * njobs;
        if constexpr (E::E == 8) {
            const uint32_t L = ctx->L;
            if (!whole && (n << E::LOGP) * 2 * L <= 256) {
                hipLaunchKernelGGL((k_encrypt_components<E, FROM>), dim3(C << E::LOGP, njobs, 2 * L), dim3(E::T), 0, st, jobs, ct_base,
                                   1u | 1u << 16, n_values, ctx->d_tabs, ctx->rc);
                return;
            }
        }
        const LimbSplit sp = split<E>(ctx, n, fixed, whole);
        hipLaunchKernelGGL((k_encrypt<E, FROM>), dim3(C << E::LOGP, njobs, sp.parts), dim3(E::T), 0, st, jobs, ct_base, sp.word, n_values,
                           ctx->d_tabs, ctx->rc);
    }

    static d2mhe_status encrypt(d2mhe_ctx *ctx, int from, const RoundJobs &jobs, uint32_t njobs,
                                uint32_t ct_base, uint64_t n_values, uint32_t C, bool whole, hipStream_t st)
    {
        if (from == FROM_VECTOR) {
            if constexpr (HALVES) return D2MHE_ERR_RANGE;       // the caller encodes first (EngineOps::halves)
            else
                launch_encrypt<ENG, FROM_VECTOR>(ctx, jobs, njobs, ct_base, n_values, C,
                                                 ctx->rc.coeff_packing ? SAMPLES : SAMPLES + ENCODING, whole, st);
        } else {
            choose<HALVES && ENG::A::KIND == 0>(encrypt_in_halves(ctx, (uint64_t)C * njobs), [&](auto shape) {
                typedef typename decltype(shape)::type E;
                if (from == FROM_WORDS32) launch_encrypt<E, FROM_WORDS32>(ctx, jobs, njobs, ct_base, n_values, C, SAMPLES, whole, st);
                else launch_encrypt<E, FROM_WORDS64>(ctx, jobs, njobs, ct_base, n_values, C, SAMPLES, whole, st);
            });
        }
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status share(d2mhe_ctx *ctx, const RoundJobs &jobs, uint32_t njobs, uint32_t ct_base, uint32_t C,
                              bool whole, hipStream_t st)
    {
        choose<HALVES>(share_in_halves(ctx, (uint64_t)C * njobs), [&](auto shape) {
            typedef typename decltype(shape)::type E;
            const LimbSplit sp = split<E>(ctx, (uint64_t)C * njobs, SAMPLES, whole);
            hipLaunchKernelGGL(k_share<E>, dim3(C << E::LOGP, njobs, sp.parts), dim3(E::T), 0, st, jobs, ct_base, sp.word, ctx->d_tabs,
                               ctx->rc);
        });
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    // Up to how many members a combine reads 8 bytes a lane: with 16 coefficients per thread the registers that pairs take are missed
    // elsewhere, and pay for many members only.  N = 2^14, times of pairs by those of 8 bytes (geometric mean, some 300 shapes): 36 and 44 bits two
    // members 1.03, three 1.01, five 0.99, seven 0.98, twelve 0.95; 30 bits 1.04, 1.02, 1.01, 1.00, 0.98.  Shoup and
    // split multiplicands spill either way (ArithS two members 1.00, three 1.01, five 0.97, twelve 0.92; the others 0.92 to 0.98).
    static constexpr bool FEW = ENG::E > 8 && (ENG::A::KIND == 0 || ENG::A::KIND == 3);
    static constexpr uint32_t FEW_MEMBERS = 3;

    static d2mhe_status combine(d2mhe_ctx *ctx, const uint64_t *ct, const PtrList &shares, uint32_t K, uint32_t C,
                                uint64_t *pt, hipStream_t st)
    {
        if (FEW && K <= FEW_MEMBERS)
            hipLaunchKernelGGL((k_combine<ENG, FEW>), dim3(C), dim3(ENG::T), 0, st, ct, shares, K, pt, ctx->d_tabs, ctx->rc);
        else
            hipLaunchKernelGGL((k_combine<ENG, false>), dim3(C), dim3(ENG::T), 0, st, ct, shares, K, pt, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status combine_decode(d2mhe_ctx *ctx, const GroupJobs &jobs, uint32_t njobs, size_t stride,
                                       uint32_t C, uint64_t n_values, hipStream_t st)
    {
        uint32_t most = 0;
        for (uint32_t j = 0; j < njobs; ++j) most = jobs.K[j] > most ? jobs.K[j] : most;
        if (FEW && most <= FEW_MEMBERS)
            hipLaunchKernelGGL((k_combine_decode<ENG, FEW>), dim3(C, njobs), dim3(ENG::T), 0, st, jobs, stride, n_values, ctx->d_tabs,
                               ctx->rc);
        else
            hipLaunchKernelGGL((k_combine_decode<ENG, false>), dim3(C, njobs), dim3(ENG::T), 0, st, jobs, stride, n_values, ctx->d_tabs,
                               ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status finish(d2mhe_ctx *ctx, const FinishJobs &jobs, uint32_t ngroups, const uint64_t *cts,
                               uint64_t *agg, uint64_t *shares, uint32_t ct_base, uint32_t C, uint64_t n_values,
                               hipStream_t st)
    {
        hipLaunchKernelGGL((k_finish<HALF, HALF::LOGP == 0>), dim3(C << HALF::LOGP, ngroups), dim3(HALF::T), 0, st, jobs, cts,
                           agg, shares, (size_t)C * 2 * ctx->L * HALF::N, ct_base, n_values, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }
    static constexpr auto finish_or_null()
    {
        if constexpr (HALF::E == 8) return &finish;
        else return nullptr;
    }

    static d2mhe_status receiver_keygen(d2mhe_ctx *ctx, uint32_t party, uint64_t *sk, uint64_t *pk, hipStream_t st)
    {
        hipLaunchKernelGGL(k_receiver_keygen<ENG>, dim3(ctx->L), dim3(ENG::T), 0, st, party, sk, pk, ctx->d_tabs,
                           ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status convert_share(d2mhe_ctx *ctx, const ConvJobs &jobs, uint32_t njobs, uint32_t ct_base,
                                      uint32_t C, bool whole, hipStream_t st)
    {
        choose<HALVES && ENG::A::KIND == 0>(encrypt_in_halves(ctx, (uint64_t)C * njobs), [&](auto shape) {
            typedef typename decltype(shape)::type E;
            const LimbSplit sp = split<E>(ctx, (uint64_t)C * njobs, SAMPLES, whole);
            hipLaunchKernelGGL(k_convert_share<E>, dim3(C << E::LOGP, njobs, sp.parts), dim3(E::T), 0, st, jobs, ct_base, sp.word, ctx->d_tabs,
                               ctx->rc);
        });
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status decrypt(d2mhe_ctx *ctx, const uint64_t *ct, const uint64_t *sk, uint32_t C, uint64_t *pt, hipStream_t st)
    {
        hipLaunchKernelGGL(k_decrypt<ENG>, dim3(C), dim3(ENG::T), 0, st, ct, sk, pt, ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status convert_combine_decode(d2mhe_ctx *ctx, const RecvJobs &jobs, uint32_t njobs, size_t stride,
                                               uint32_t C, uint64_t n_values, hipStream_t st)
    {
        // N = 2^14, rounds with 16-byte loads of pairs (they spill) and 8-byte loads, us: 54 bits, 10 workgroups of 8 limbs 563.5 / 569.8, 16 of 4 415.6 /
        // 428.2, 36 of 6 907 / 930, 64 of 3 583 / 592, 120 of 3 941 / 940;  60 bits 586 / 593, 433 / 442, 960 / 981, 621 / 626, 1,003 / 999;  Shoup
        // quotients, 54 bits 679 / 712, 510 / 534, 1,065 / 1,105, 706 / 724, 1,194 / 1,213;  60 bits 761 / 768, 578 / 587, 1,234 / 1,257, 839 / 844, 1,435 /
        // 1,444;  30 bits 551 / 547, 424 / 425, 878 / 885, 571 / 577, 970 / 968;  36 bits 596 / 585, 432 / 433, 916 / 920, 585 / 581, 912 / 900.
        constexpr bool FEW = ENG::E > 8, PAIRS = FEW && ENG::A::KIND != 0 && ENG::A::KIND != 3;
        if (PAIRS && (uint64_t)C * njobs <= 64)
            hipLaunchKernelGGL((k_convert_combine_decode<ENG, FEW && !PAIRS>), dim3(C, njobs), dim3(ENG::T), 0, st, jobs, stride,
                               n_values, ctx->d_tabs, ctx->rc);
        else
            hipLaunchKernelGGL((k_convert_combine_decode<ENG, FEW>), dim3(C, njobs), dim3(ENG::T), 0, st, jobs, stride, n_values, ctx->d_tabs,
                               ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status bootstrap_alpha(d2mhe_ctx *ctx, uint32_t group, uint32_t ct_base, uint32_t C, uint64_t *alpha,
                                        hipStream_t st)
    {
        hipLaunchKernelGGL(k_bootstrap_alpha<ENG>, dim3(C, ctx->L), dim3(ENG::T), 0, st, alpha, group, ct_base,
                           ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    static d2mhe_status bootstrap_share(d2mhe_ctx *ctx, const ConvJobs &jobs, uint32_t njobs, uint32_t ct_base,
                                        uint32_t C, bool whole, hipStream_t st)
    {
        choose<HALVES>(refresh_in_halves((uint64_t)C * njobs), [&](auto shape) {
            typedef typename decltype(shape)::type E;
            const LimbSplit sp = split<E>(ctx, (uint64_t)C * njobs, MASKS, whole);
            hipLaunchKernelGGL(k_bootstrap_share<E>, dim3(C << E::LOGP, njobs, sp.parts), dim3(E::T), 0, st, jobs, ct_base, sp.word, ctx->d_tabs,
                               ctx->rc);
        });
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    // Up to how many indices the limbs of refreshed ciphertexts go in a launch of their own.  Measured, us in one launch / in two,
    // 32, 64, 128 and 200 indices by seven members:
    //   N = 8192, 54 bits, four limbs 119 / 92, 145 / 114, 158 / 146, 186 / 203;  two 62 / 57, 64 / 63, 87 / 86, 102 / 114;  one 33 / 39
    //   N = 4096, 36 bits, three limbs 45 / 37, 46 / 42, 51 / 57, 79 / 84;  eight 116 / 86, 147 / 110, 161 / 145, 192 / 196
    //   N = 2048, 54 bits, six limbs 66 / 46, 67 / 54, 69 / 64, 84 / 83;  N = 1024, 30 bits, two limbs 15 / 15, 15 / 15, 16 / 16, 21 / 21
    //   N = 2^14, 36 bits, two limbs 140 / 113, 145 / 120, 158 / 144, 186 / 203
    static uint32_t refresh_apart(const d2mhe_ctx *ctx)
    {
        const uint32_t L = ctx->L;
        return L >= 4 || (L > 1 && ENG::LOGN == 14) ? 128 : L == 3 ? 85 : L == 2 && ENG::LOGN > 10 ? 32 : 0;
    }
    static d2mhe_status bootstrap_combine(d2mhe_ctx *ctx, const uint64_t *ct, const PtrList &shares, uint32_t K,
                                          const uint64_t *alpha, uint32_t C, uint64_t *ct_out, bool whole, hipStream_t st)
    {
        if (!whole && C <= refresh_apart(ctx)) {
            hipLaunchKernelGGL(k_bootstrap_round<ENG>, dim3(C), dim3(ENG::T), 0, st, ct, shares, K, ct_out, ctx->d_tabs, ctx->rc);
            D2_LAUNCHED(ctx);
            hipLaunchKernelGGL(k_bootstrap_refresh<ENG>, dim3(C, ctx->L), dim3(ENG::T), 0, st, shares, K, alpha, ct_out, ctx->d_tabs,
                               ctx->rc);
            D2_LAUNCHED(ctx);
            return D2MHE_OK;
        }
        hipLaunchKernelGGL(k_bootstrap_combine<ENG>, dim3(C), dim3(ENG::T), 0, st, ct, shares, K, alpha, ct_out,
                           ctx->d_tabs, ctx->rc);
        D2_LAUNCHED(ctx);
        return D2MHE_OK;
    }

    // full set (ring degrees a single workgroup can hold)
    static EngineOps full()
    {
        return EngineOps{ENG::ELOG, ENG::LOGB, HALVES, &ntt, &keygen, &encode, &decode, &encode_parties, &encrypt, &share,
                         &combine, &combine_decode, finish_or_null(), &receiver_keygen, &convert_share, &decrypt,
                         &convert_combine_decode, &bootstrap_alpha, &bootstrap_share, &bootstrap_combine};
    }
    // transforms only (longer rings)
    static EngineOps transforms_only()
    {
        return EngineOps{ENG::ELOG, ENG::LOGB, false, &ntt, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                         nullptr,   nullptr,   nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    }
};

}  // namespace d2
