"""The launch that sums, makes the shares, combines and decodes (taken by d2mhe_round where it fills the chip and no
event between those phases is asked for) against the separate launches, which the other tests hold to the oracle:
every word of the scratch and every decoded value."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import DEV, dzeros, make_ctx, to_dev


def ring(parties, reach):
    return [sorted((i + d) % parties for d in range(-reach, reach + 1)) for i in range(parties)]


# (prime bits, log2 N, limbs, groups, ciphertexts, packing): groups of one member, and around the 32 terms after which
# a lazy sum is reduced; more parties, more members and more groups than one launch's table holds (128, 1400, 64); the
# chip exactly filled (256 workgroups, 1024 for N = 1024) on every kind of arithmetic
@pytest.mark.parametrize("bits,log2n,L,groups,C,packing", [
    (54, 11, 2, [list(range(k)) for k in (1, 2, 32, 33, 64)], 52, 0),
    (44, 11, 2, [list(range(k)) for k in (31, 33, 64)], 86, 0),
    (60, 11, 1, [list(range(k)) for k in (1, 33, 64)], 86, 0),
    (54, 11, 1, ring(200, 4), 12, 1),
    (36, 11, 1, ring(100, 15), 16, 0),
    (30, 10, 2, ring(32, 1), 32, 0),
    (54, 12, 3, ring(16, 2), 16, 0),
    (36, 13, 2, ring(8, 1), 32, 0),
    (54, 14, 2, ring(8, 1), 32, 0),            # halves of polynomials: sum and shares, then the combine
    (44, 14, 1, [list(range(k)) for k in (1, 2, 5)], 86, 0),
    (60, 14, 2, ring(9, 2), 29, 1),
])
def test_one_launch_equals_three(bits, log2n, L, groups, C, packing):
    N, K = 1 << log2n, max(len(g) for g in groups)
    q, t = O.find_primes(bits, log2n, L), 12289 if log2n <= 11 else 65537
    P, J, G = 1 + max(max(g) for g in groups), sum(len(g) for g in groups), len(groups)
    n = C * N - 13
    ctx = make_ctx(log2n, q, t, f=3, max_group=K, seed=11)
    sk, pk0 = [dzeros(2 * L * N) for _ in range(P)], [dzeros(L * N) for _ in range(P)]
    for k in range(P):
        ctx.keygen_share(k, sk[k], pk0[k])
    pks = []
    for g in groups:
        pks.append(dzeros(4 * L * N))
        ctx.aggregate_pk([pk0[k] for k in g], pks[-1])
    rng = np.random.default_rng(bits + log2n)
    vec = to_dev(rng.normal(0, 2.0, n + 4 * P).astype(np.float32))
    outs = [torch.zeros((n + 3) // 4 * 4, dtype=torch.float32, device=DEV) for _ in groups]
    nbytes = ctx.round_scratch_bytes(J, G, n)
    scratch = dzeros(nbytes // 8)
    desc = ctx.make_round(groups, pks, sk, [vec[4 * k:4 * k + n] for k in range(P)], outs, n,
                          group_ids=[3 + 2 * g for g in range(G)], ct_base=7, packing=packing)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
    for e in events:
        e.record()
    ctx.round(desc, scratch, nbytes, [e.cuda_event for e in events])
    want, sums = scratch.clone(), [o.clone() for o in outs]
    scratch.fill_(-1)
    for o in outs:
        o.zero_()
    ctx.round(desc, scratch, nbytes)
    torch.cuda.synchronize()
    assert torch.equal(scratch, want)
    for g, (a, b) in enumerate(zip(outs, sums)):
        assert torch.equal(a, b), f"group {g}"
    ctx.close()
