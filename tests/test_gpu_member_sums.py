"""Sums over members inside the combining kernels (16-byte loads, their words brought back to their owners; two or three members
under way; kept in the caches or streamed): shares of K members against one share that is their sum modulo q, which takes
no loop; with words at the ends of their range, whose sums are multiples of q."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import DEV, dzeros, make_ctx
from test_pm_policies import primes_away_from_powers_of_two


# C = 129 or 200: streamed; 64 members: as many as there can be
@pytest.mark.parametrize("bits,log2n,L,C,Ks", [
    ("30", 10, 2, 3, (2, 3, 64)), ("36", 11, 2, 2, (2, 3, 4, 5, 63, 64)), ("44", 12, 1, 200, (6, 64)), ("36", 14, 2, 2, (3, 4, 64)), ("30", 14, 2, 2, (2, 3, 4, 5)), ("54a", 14, 1, 2, (3, 4)),
    ("54", 12, 2, 129, (3, 8)), ("54", 13, 2, 3, (2, 7, 64)), ("60", 13, 2, 2, (5, 64)), ("54a", 13, 1, 2, (4, 64)),
    ("60a", 11, 2, 2, (3, 64)), ("54", 14, 2, 1, (2, 3, 64)), ("60a", 14, 1, 130, (5,)),
])
def test_members_equal_their_sum(bits, log2n, L, C, Ks):
    N, t = 1 << log2n, 12289 if log2n <= 11 else 65537
    q = primes_away_from_powers_of_two(int(bits[:-1]), log2n, L) if bits.endswith("a") else O.find_primes(int(bits), log2n, L)
    ctx = make_ctx(log2n, q, t, f=3, max_group=64, seed=12)
    qs = torch.tensor(q, dtype=torch.int64, device=DEV).view(1, 1, L, 1)
    gen = torch.Generator(device=DEV).manual_seed(log2n)

    def words(polys):
        w = torch.randint(0, 1 << 62, (C, polys, L, N), generator=gen, dtype=torch.int64, device=DEV) % qs
        end = torch.randint(0, 4, (C, polys, 1, N), generator=gen, device=DEV)           # half of the words at an end
        return torch.where(end == 0, qs - 1, torch.where(end == 1, torch.zeros_like(qs), w)).contiguous()

    ct, alpha = words(2), words(1)
    for K in Ks:
        shares, pairs = [words(1) for _ in range(K)], [words(2) for _ in range(K)]

        def total(parts):
            s = parts[0]
            for p in parts[1:]:
                s = s + p - torch.where(s >= qs - p, qs, torch.zeros_like(qs))
            return s.contiguous()

        if K == 64:     # c0 and the shares add up to 64 q
            shares = [(qs - 1).expand(C, 1, L, N).contiguous() for _ in range(K)]
            ct[:, 0] = 64
        got, want = dzeros(C * N), dzeros(C * N)
        ctx.combine(ct, shares, C, got)
        ctx.combine(ct, [total(shares)], C, want)
        assert torch.equal(got, want), f"combine of {K}"
        got, want = dzeros(C * 2 * L * N), dzeros(C * 2 * L * N)
        ctx.bootstrap_combine(ct, alpha, pairs, C, got)
        ctx.bootstrap_combine(ct, alpha, [total(pairs)], C, want)
        assert torch.equal(got, want), f"refresh by {K}"
    torch.cuda.synchronize()
    ctx.close()


# C indices refreshed in one launch against runs of `part` of them (rounding and limbs in a launch each)
@pytest.mark.parametrize("bits,log2n,L,C,part", [("30", 11, 2, 64, 32), ("54", 12, 3, 170, 85), ("36", 13, 4, 150, 40), ("60a", 14, 2, 129, 43),
                                                 ("54", 10, 6, 140, 128)])
def test_refresh_in_parts(bits, log2n, L, C, part):
    LN, t, K = L << log2n, 12289 if log2n <= 11 else 65537, 3
    q = primes_away_from_powers_of_two(int(bits[:-1]), log2n, L) if bits.endswith("a") else O.find_primes(int(bits), log2n, L)
    ctx = make_ctx(log2n, q, t, f=3, max_group=K, seed=14)
    words = dzeros((3 + 2 * K) * C * LN)
    ctx.bench_polys(words, (3 + 2 * K) * C)
    ct, alpha = words[:2 * C * LN], words[2 * C * LN:3 * C * LN]
    shares = [words[(3 + 2 * k) * C * LN:(5 + 2 * k) * C * LN] for k in range(K)]
    whole, parts = dzeros(2 * C * LN), dzeros(2 * C * LN)
    ctx.bootstrap_combine(ct, alpha, shares, C, whole)
    for c in range(0, C, part):
        at = slice(2 * c * LN, None)
        ctx.bootstrap_combine(ct[at], alpha[c * LN:], [s[at] for s in shares], min(part, C - c), parts[at])
    assert torch.equal(whole, parts)
    torch.cuda.synchronize()
    ctx.close()


# the sums of both halves of conversion shares inside a round (K members, one after another or in pairs) against the same shares
# added up by d2mhe_convert_combine and decrypted
@pytest.mark.parametrize("bits,log2n,L,C,Ks", [
    ("30", 10, 2, 2, (1, 2, 5, 64)), ("36", 11, 3, 2, (1, 3, 64)), ("44", 13, 2, 2, (1, 2, 4, 5, 64)), ("54", 13, 2, 2, (1, 2, 3, 64)),
    ("60", 13, 1, 2, (1, 2, 5)), ("54a", 12, 2, 2, (1, 4)), ("60a", 13, 2, 2, (3, 64)), ("36", 14, 2, 2, (1, 2, 5, 64)), ("54", 14, 1, 2, (1, 4)),
    ("60a", 14, 1, 2, (1, 3)), ("30", 14, 2, 2, (2, 3)),
    ("54", 14, 2, 64, (3, 5)), ("60", 14, 1, 2, (1, 2, 64)), ("54", 14, 1, 65, (1, 3)), ("60", 14, 2, 65, (4,)), ("54a", 14, 1, 3, (1, 2, 64)),
    ("60a", 14, 1, 65, (3,)),      # N = 2^14: loads in pairs up to C = 64
])
def test_conversion_shares_in_a_round(bits, log2n, L, C, Ks):
    N, t, receiver = 1 << log2n, 12289 if log2n <= 11 else 65537, 0
    q = primes_away_from_powers_of_two(int(bits[:-1]), log2n, L) if bits.endswith("a") else O.find_primes(int(bits), log2n, L)
    ctx = make_ctx(log2n, q, t, f=3, max_group=64, seed=15)
    LN, n = L * N, C * N - 3
    sks, pk0 = [dzeros(2 * LN) for _ in range(max(Ks))], [dzeros(LN) for _ in range(max(Ks))]
    for k in range(max(Ks)):
        ctx.keygen_share(k, sks[k], pk0[k])
    rsk, rpk = dzeros(2 * LN), dzeros(4 * LN)
    ctx.receiver_keygen(receiver, rsk, rpk)
    gen = torch.Generator(device=DEV).manual_seed(L)
    grads = [torch.randn(C * N, generator=gen, dtype=torch.float32, device=DEV) for _ in range(max(Ks))]
    for K in Ks:
        pk = dzeros(4 * LN)
        ctx.aggregate_pk(pk0[:K], pk)
        got, want = dzeros(C * N, dtype=torch.float32), dzeros(C * N, dtype=torch.float32)
        desc = ctx.make_round([list(range(K))], [pk], sks[:K], grads[:K], [None], n)
        conv = ctx.make_convert(desc, [[receiver]], {receiver: rpk}, {receiver: rsk}, [got])
        size = ctx.round_convert_scratch_bytes(K, 1, K, n)
        scratch = dzeros(size // 8 + 2)
        ctx.round_convert(desc, conv, scratch, size)
        agg, first = scratch[K * C * 2 * LN:], (K + 1) * C * 2 * LN
        ct, pt = dzeros(C * 2 * LN), dzeros(C * N)
        ctx.convert_combine(agg, [scratch[first + k * C * 2 * LN:] for k in range(K)], C, ct)
        ctx.decrypt(rsk, ct, C, pt)
        ctx.decode(pt, C, n, want)
        assert torch.equal(got, want), f"{K} members"
    torch.cuda.synchronize()
    ctx.close()
