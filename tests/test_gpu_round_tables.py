"""Rounds whose job tables do not fit one launch (880 jobs, 112 parties, 112 groups), rounds of as many jobs as a table
lists in rows (112, 64 conversion shares) and one more, and rounds whose parties are in
many groups, so that their vectors are encoded once ahead of the encryption: every message against the per-call entry
points, which the other tests hold to the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import DEV, dzeros, make_ctx, to_dev


def ring(parties, reach):
    return [sorted((i + d) % parties for d in range(-reach, reach + 1)) for i in range(parties)]


def pairs(n):
    return [[g, g + 1] for g in range(n)]


def shuffled(groups, seed):
    rng = np.random.default_rng(seed)
    return [[int(k) for k in rng.permutation(g)] for g in groups]


# (prime bits, log2 N, limbs, groups, ciphertexts, packing, one event between the phases)
@pytest.mark.parametrize("bits,log2n,L,groups,C,packing,split", [
    (54, 10, 1, ring(200, 4), 1, 0, True),                      # 1,800 jobs, more parties and groups than a table lists
    (36, 10, 2, shuffled(ring(41, 10), 1), 2, 0, True),         # 861 jobs: one launch; members in any order
    (30, 10, 1, shuffled(ring(42, 10), 2), 2, 0, True),         # 882: two
    (54, 11, 1, ring(125, 3), 2, 0, False),                     # 875 jobs, parties beyond the table before the jobs are
    (60, 13, 1, ring(39, 19), 1, 0, False),                     # 39 groups of the same 39 members: 1,521 jobs
    (54, 14, 1, ring(23, 5), 5, 0, False),                      # encryption in halves of polynomials
    (30, 14, 1, ring(23, 5), 5, 0, False),                      # whole ones, 16 coefficients per thread
    (54, 10, 1, pairs(56), 2, 0, True),                         # 112 jobs: rows of the table
    (36, 11, 1, pairs(57), 2, 0, True),                         # 114: parties and groups listed once
    (60, 10, 1, [[65535, 7, 40000], [7, 9], [40000, 65528]], 2, 0, True),       # ids far apart, two pairs of which collide
    (30, 10, 1, [[(40503 * k) % 65521 for k in range(g, g + 5)] for g in range(30)], 1, 0, True),
    (44, 11, 1, ring(130, 3), 2, 1, True),                      # coefficient packing: never encoded ahead
    (54, 10, 1, [[0, 1, 2], [3, 4]], 300, 0, True),             # nobody in two groups
])
def test_round_equals_per_call(bits, log2n, L, groups, C, packing, split):
    N = 1 << log2n
    groups = [list(dict.fromkeys(g)) for g in groups]
    K = max(len(g) for g in groups)
    q, t = O.find_primes(bits, log2n, L), 12289 if log2n <= 11 else 65537
    ids, J, G = sorted({k for g in groups for k in g}), sum(len(g) for g in groups), len(groups)
    n, LN = C * N - 5, L * N
    ctx = make_ctx(log2n, q, t, f=3, max_group=K, seed=5)
    sk, pk0 = {k: dzeros(2 * LN) for k in ids}, {k: dzeros(LN) for k in ids}
    for k in ids:
        ctx.keygen_share(k, sk[k], pk0[k])
    pks = [dzeros(4 * LN) for _ in groups]
    for g, pk in zip(groups, pks):
        ctx.aggregate_pk([pk0[k] for k in g], pk)
    vec = to_dev(np.random.default_rng(bits).normal(0, 2.0, n + 4 * len(ids)).astype(np.float32))
    grads = {k: vec[4 * i:4 * i + n] for i, k in enumerate(ids)}
    outs = [torch.zeros((n + 3) // 4 * 4, dtype=torch.float32, device=DEV) for _ in groups]
    nbytes = ctx.round_scratch_bytes(J, G, n)
    scratch = dzeros(nbytes // 8)
    gids = [3 + 2 * g for g in range(G)]
    desc = ctx.make_round(groups, pks, sk, grads, outs, n, group_ids=gids, ct_base=7, packing=packing)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
    for e in events:
        e.record()
    ctx.round(desc, scratch, nbytes, [e.cuda_event for e in events] if split else None)
    cts = scratch[:J * C * 2 * LN].view(J, C * 2 * LN)
    agg = scratch[J * C * 2 * LN:(J + G) * C * 2 * LN].view(G, C * 2 * LN)
    shares = scratch[(J + G) * C * 2 * LN:].view(J, C * LN)
    pts = {k: dzeros(C * N) for k in ids}
    for k in ids:
        (ctx.encode_coefficients if packing else ctx.encode)(grads[k], n, pts[k], C)
    ct, share, j = dzeros(C * 2 * LN), dzeros(C * LN), 0
    for g, members in enumerate(groups):
        total = None
        for k in members:
            ctx.encrypt(pks[g], pts[k], C, k, gids[g], 7, ct)
            assert torch.equal(ct, cts[j]), f"ciphertext of party {k} in group {g}"
            if total is None:
                total = ct.clone()
            else:
                ctx.add(total, ct, C)
            ctx.partial_decrypt(sk[k], agg[g], C, k, gids[g], 7, share)
            assert torch.equal(share, shares[j]), f"share of party {k} in group {g}"
            j += 1
        assert torch.equal(total, agg[g]), f"aggregate of group {g}"
    torch.cuda.synchronize()
    ctx.close()


# conversion shares: 320 jobs, 104 members, 104 receivers, 64 groups to a launch; rows up to 64 jobs
@pytest.mark.parametrize("bits,log2n,L,parties,reach,C", [
    (54, 10, 1, 130, 1, 1),          # 390 jobs; more members, receivers and groups than a table lists
    (36, 10, 2, 64, 2, 1),           # exactly 320, 64 groups
    (54, 11, 1, 65, 2, 2),           # 325
    (30, 10, 1, 12, 5, 2),           # 11 members each, 132
    (54, 14, 1, 7, 1, 2),            # halves of polynomials
    (44, 14, 1, 7, 1, 7),            # 147 polynomials of one limb: whole
    (60, 10, 1, 21, 1, 2),           # 63: rows of the table
    (54, 10, 1, 13, 2, 2),           # 65
])
def test_round_convert_equals_per_call(bits, log2n, L, parties, reach, C):
    N, LN, groups = 1 << log2n, L << log2n, ring(parties, reach)
    K, P = len(groups[0]), parties
    q, t = O.find_primes(bits, log2n, L), 12289 if log2n <= 11 else 65537
    n = C * N - 3
    ctx = make_ctx(log2n, q, t, f=3, max_group=K, seed=9)
    sk, pk0 = [dzeros(2 * LN) for _ in range(P)], [dzeros(LN) for _ in range(P)]
    rsk, rpk = [dzeros(2 * LN) for _ in range(P)], [dzeros(4 * LN) for _ in range(P)]
    for k in range(P):
        ctx.keygen_share(k, sk[k], pk0[k])
        ctx.receiver_keygen(k, rsk[k], rpk[k])
    pks = [dzeros(4 * LN) for _ in groups]
    for g, pk in zip(groups, pks):
        ctx.aggregate_pk([pk0[k] for k in g], pk)
    vec = to_dev(np.random.default_rng(bits).normal(0, 2.0, n + 4 * P).astype(np.float32))
    grads = [vec[4 * k:4 * k + n] for k in range(P)]
    outs = [torch.zeros((n + 3) // 4 * 4, dtype=torch.float32, device=DEV) for _ in groups]
    ids, receivers = [3 + 2 * g for g in range(P)], [[g] for g in range(P)]
    desc = ctx.make_round(groups, pks, sk, grads, outs, n, group_ids=ids, ct_base=7)
    conv = ctx.make_convert(desc, receivers, rpk, rsk, outs)
    nbytes = ctx.round_convert_scratch_bytes(K * P, P, conv.num_shares, n)
    scratch = dzeros(nbytes // 8)
    ctx.round_convert(desc, conv, scratch, nbytes)
    agg = scratch[K * P * C * 2 * LN:(K + 1) * P * C * 2 * LN].view(P, C * 2 * LN)
    shares = scratch[(K + 1) * P * C * 2 * LN:].view(K * P, C * 2 * LN)
    share = dzeros(C * 2 * LN)
    for g, members in enumerate(groups):
        for i, k in enumerate(members):
            ctx.convert_share(sk[k], rpk[g], agg[g], C, k, g, ids[g], 7, share)
            assert torch.equal(share, shares[g * K + i]), f"share of party {k} in group {g}"
    torch.cuda.synchronize()
    ctx.close()


# N = 2^14 where a launch may take whole polynomials or halves of them: 130 (two turns of the chip in halves, one in whole
# polynomials) against 65 and 65 (halves); with four limbs also shares of 520 (five turns in halves, three in whole
# polynomials: halves) against four times 130 (whole)
@pytest.mark.parametrize("bits,L,C,part", [(44, 1, 130, 65), (36, 2, 130, 65), (54, 1, 130, 65), (60, 1, 130, 65),
                                           (36, 4, 520, 130)])
def test_whole_polynomials_equal_halves(bits, L, C, part):
    log2n, LN = 14, L << 14
    ctx = make_ctx(log2n, O.find_primes(bits, log2n, L), 65537, f=3, max_group=2, seed=21)
    sk, pk0, pk, rsk, rpk = (dzeros(n * LN) for n in (2, 1, 4, 2, 4))
    ctx.keygen_share(1, sk, pk0)
    ctx.aggregate_pk([pk0], pk)
    ctx.receiver_keygen(2, rsk, rpk)
    pt = to_dev(np.random.default_rng(bits).integers(0, 65537, C << log2n, dtype=np.uint64))
    ct, alpha = dzeros(C * 2 * LN), dzeros(C * LN)
    ctx.encrypt(pk, pt, C, 1, 5, 3, ct)
    ctx.bootstrap_alpha(5, 3, C, alpha)
    calls = {
        "ciphertexts": (2, lambda c, n, out: ctx.encrypt(pk, pt[c << log2n:], n, 1, 5, 3 + c, out)),
        "shares": (1, lambda c, n, out: ctx.partial_decrypt(sk, ct[c * 2 * LN:], n, 1, 5, 3 + c, out)),
        "conversion shares": (2, lambda c, n, out: ctx.convert_share(sk, rpk, ct[c * 2 * LN:], n, 1, 2, 5, 3 + c, out)),
        "refresh shares": (2, lambda c, n, out: ctx.bootstrap_share(sk, ct[c * 2 * LN:], alpha[c * LN:], n, 1, 5, 3 + c, out)),
    }
    for name, (polys, call) in calls.items():
        whole, parts = dzeros(C * polys * LN), dzeros(C * polys * LN)
        call(0, C, whole)
        for c in range(0, C, part):
            call(c, part, parts[c * polys * LN:])
        assert torch.equal(whole, parts), name
    torch.cuda.synchronize()
    ctx.close()
