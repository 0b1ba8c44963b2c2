"""Batches of transforms: how many polynomials a workgroup walks through depends on the batch (in the transforms of two kernels
one member where the chip has room, up to sixteen; N = 8192 and 2^14 more than one beyond 256 polynomials, unless that takes a
turn of the chip more), so every batch is compared with its members transformed one by one."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O

from gpu_util import dzeros, make_ctx
from test_pm_policies import primes_away_from_powers_of_two


# members to a workgroup: 1, 2 (remainder), 3, 4, 6, 8 (remainder), 12, 16
@pytest.mark.parametrize("bits,log2n,L,B", [(54, 15, 2, 31), (60, 15, 3, 37), (36, 15, 8, 24), (30, 16, 1, 97), (54, 16, 2, 90),
                                            (60, 16, 1, 251), (36, 15, 7, 96), (44, 16, 16, 32),
                                            (54, 13, 1, 257), (60, 13, 7, 75), (36, 14, 3, 171), (30, 14, 16, 17),
                                            # Shoup quotients; one by one (two turns instead of three); a turn more than one by one
                                            ("54a", 13, 7, 40), ("60a", 13, 1, 300), ("60a", 13, 6, 85), (54, 13, 7, 73), (60, 13, 13, 39),
                                            (54, 13, 13, 136), ("54a", 13, 7, 292), (36, 14, 13, 78), (30, 14, 7, 109), (36, 14, 10, 102)])
def test_batch_equals_members(bits, log2n, L, B):
    away = str(bits).endswith("a")
    q = primes_away_from_powers_of_two(int(bits[:-1]), log2n, L) if away else O.find_primes(bits, log2n, L)
    ctx = make_ctx(log2n, q, 0, seed=3)
    words = L << log2n
    batch = dzeros(B * words)
    ctx.bench_polys(batch, B)
    single, first = batch.clone(), batch.clone()
    ctx.ntt_forward(batch, B)
    for b in range(B):
        ctx.ntt_forward(single[b * words:], 1)
    assert torch.equal(batch, single), "forward"
    ctx.ntt_inverse(batch, B)
    for b in range(B):
        ctx.ntt_inverse(single[b * words:], 1)
    assert torch.equal(batch, single), "inverse"
    assert torch.equal(batch, first), "there and back"
    torch.cuda.synchronize()
    ctx.close()
