"""The launch that sums, makes the shares, combines and decodes (taken by d2mhe_round where it leaves no part of the
chip idle and no event between those phases is asked for) against the separate launches, which the other tests hold to
the oracle: every word of the scratch and every decoded value; and which of the two a round takes, from the nodes of
the graph that a capture of it makes."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import DEV, dzeros, make_ctx, to_dev
from test_pm_policies import primes_away_from_powers_of_two


def ring(parties, reach):
    return [sorted((i + d) % parties for d in range(-reach, reach + 1)) for i in range(parties)]


def sizes(*ks):
    return [list(range(k)) for k in ks]


def launches(call):
    """Nodes of the graph that `call` makes under capture: its kernel launches."""
    graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            call(side.cuda_stream)
    n = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# (prime bits, a: far from a power of two; log2 N, limbs, groups, ciphertexts, packing, taken): every kind of arithmetic;
# groups of one member, and around the 32 terms after which a lazy sum is reduced; more parties, more members and more
# groups than one launch's table holds (128, 1400, 64); the chip exactly filled, and the edges of the rule
@pytest.mark.parametrize("bits,log2n,L,groups,C,packing,taken", [
    ("54", 11, 2, sizes(1, 32, 33, 64), 128, 0, True),
    ("54a", 11, 2, sizes(1, 32, 33, 64), 128, 0, True),
    ("60a", 11, 1, sizes(1, 32, 33, 64), 128, 0, True),
    ("44", 11, 2, sizes(31, 33, 64), 171, 0, False),       # 513 workgroups: a third turn of the chip for one of them
    ("44", 11, 2, sizes(31, 33, 64), 209, 0, True),        # 627 of 768
    ("60", 11, 1, sizes(1, 33, 64, 2), 128, 0, True),
    ("54", 11, 1, ring(200, 4), 24, 1, True),              # four launches of 50 groups: 1,200 of 1,280 workgroups each
    ("54", 11, 1, ring(200, 4), 13, 1, False),             # 650 of 768
    ("44", 11, 2, ring(12, 1), 31, 1, True),               # three members each: 372 of 512
    ("36", 11, 1, ring(100, 15), 36, 0, True),             # 34, 34 and 32 groups
    ("30", 12, 1, ring(100, 1), 10, 0, False),             # two launches of 500
    ("36", 11, 1, ring(32, 1), 8, 0, True),                # three members each: 256 are enough
    ("36", 11, 1, ring(32, 2), 8, 0, False),
    ("30", 10, 2, ring(32, 1), 32, 0, True),
    ("30", 10, 1, ring(32, 2), 32, 0, False),
    ("54a", 10, 2, ring(32, 1), 32, 0, True),
    ("60a", 10, 1, ring(32, 2), 56, 0, True),
    ("54", 12, 3, ring(16, 2), 16, 0, True),
    ("54", 12, 2, ring(16, 2), 20, 0, False),              # 320 of 512
    ("36", 12, 3, ring(16, 2), 25, 0, True),               # 400
    ("36", 12, 1, ring(16, 2), 36, 0, False),              # 576 of 768
    ("30", 13, 2, ring(16, 2), 24, 0, True),               # 384 of 512
    ("60a", 12, 1, sizes(1, 2, 33, 64), 64, 0, True),
    ("54a", 12, 2, ring(16, 2), 16, 0, True),
    ("36", 13, 2, ring(8, 1), 32, 0, True),
    ("54a", 13, 2, ring(8, 1), 32, 0, True),
    ("60a", 13, 1, ring(8, 1), 32, 1, True),
    ("54", 14, 4, ring(8, 1), 32, 0, True),                # halves of polynomials: sum and shares, then the combine
    ("54", 14, 2, ring(8, 1), 64, 0, False),
    ("44", 14, 3, sizes(1, 2, 5), 192, 0, True),
    ("60", 14, 8, ring(5, 1), 51, 1, True),
    ("54a", 14, 3, ring(8, 1), 64, 0, False),              # whole polynomials: no such kernel
])
def test_one_launch_equals_three(bits, log2n, L, groups, C, packing, taken):
    find = primes_away_from_powers_of_two if bits.endswith("a") else O.find_primes
    bits = int(bits.rstrip("a"))
    N, K = 1 << log2n, max(len(g) for g in groups)
    q, t = find(bits, log2n, L), 12289 if log2n <= 11 else 65537
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
    split = launches(lambda stream: ctx.round(desc, scratch, nbytes, [e.cuda_event for e in events], stream))
    fused = launches(lambda stream: ctx.round(desc, scratch, nbytes, None, stream))
    assert fused < split if taken else fused == split, (fused, split)
    ctx.close()
