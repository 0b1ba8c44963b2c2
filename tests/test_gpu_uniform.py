"""Uniform residues from 128 random bits, modulo the primes of a context and modulo plaintext primes up to the largest it takes:
the common polynomial and a refresh share against the oracle, which reduces the same blocks with 128-bit integers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import dzeros, make_ctx, to_dev, to_eval, to_host


def largest_plaintext_prime(log2n):
    step = 2 << log2n
    t = ((1 << 30) - 1) // step * step + 1
    while t >= 1 << 30 or any(t % d == 0 for d in range(3, 32769, 2)):
        t -= step
    return t


@pytest.mark.parametrize("bits,log2n,t", [(60, 10, 0), (36, 11, 0), (44, 10, 12289), (54, 12, 65537), (60, 13, 0)])
def test_alpha_and_refresh_share(bits, log2n, t):
    L, N, C, q = 2, 1 << log2n, 2, O.find_primes(bits, log2n, 2)
    t = t or largest_plaintext_prime(log2n)
    o, ctx = O.Oracle(log2n, q, t, 21, 3, 2, 77), make_ctx(log2n, q, t, f=3, max_group=2, seed=77)
    perm = ctx.index_map()
    osk = o.keygen_share(1)[0]
    sk, pk0 = dzeros(2 * L * N), dzeros(L * N)
    ctx.keygen_share(1, sk, pk0)
    rng = np.random.default_rng(bits)
    oagg = np.stack([rng.integers(0, m, (C, 2, N), dtype=np.uint64) for m in q], axis=2)
    alpha, share = dzeros(C * L * N), dzeros(C * 2 * L * N)
    ctx.bootstrap_alpha(9, 4, C, alpha)
    oalpha = np.stack([o.bootstrap_alpha(9, 4 + c) for c in range(C)])
    assert np.array_equal(to_host(alpha, oalpha.shape), to_eval(o, perm, oalpha)), "alpha"
    ctx.bootstrap_share(sk, to_dev(to_eval(o, perm, oagg)), alpha, C, 1, 9, 4, share)
    oshare = o.bootstrap_share(osk, oagg, 1, 9, 4)
    assert np.array_equal(to_host(share, oshare.shape), to_eval(o, perm, oshare)), "refresh share"
    ctx.close()
