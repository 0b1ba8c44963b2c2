"""Launches that share the limbs of a polynomial among several workgroups."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_limb_in_one_part(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    exe = str(tmp_path / "check")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-o", exe, os.path.join(ROOT, "tests", "limb_split_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    counts, us = out.stdout.split()[:3], float(out.stdout.split()[3])
    assert min(int(v) for v in counts) > 20, out.stdout
    assert us < 15, "a launch takes 2.5 us by itself, and a caller that waits for each pays for this in front of it"


# C indices at once (whole polynomials, or other parts) against runs of `part` of them (one limb, two, or all but one or two to a
# workgroup; either component of a ciphertext by itself): every word
@pytest.mark.gpu
@pytest.mark.parametrize("bits,log2n,L,C,part", [
    (30, 10, 3, 2050, 205), (54, 10, 6, 2050, 41), (36, 11, 5, 1024, 128), (60, 11, 2, 1024, 64), (44, 12, 3, 512, 150),
    (54, 12, 2, 512, 100), (36, 13, 8, 256, 33), (54, 13, 4, 256, 153), (60, 13, 3, 256, 1), (54, 14, 8, 128, 50),
    (36, 14, 3, 128, 16), (54, 12, 1, 512, 128), (30, 10, 1, 300, 128), (60, 13, 2, 256, 64), (54, 14, 1, 128, 64),
])
def test_parts_equal_whole_polynomials(bits, log2n, L, C, part):
    from oracle import oracle as O
    import torch
    from gpu_util import dzeros, make_ctx, to_dev
    LN, t = L << log2n, 12289 if log2n <= 11 else 65537
    ctx = make_ctx(log2n, O.find_primes(bits, log2n, L), t, f=3, max_group=2, seed=33)
    sk, pk0, pk, rsk, rpk = (dzeros(n * LN) for n in (2, 1, 4, 2, 4))
    ctx.keygen_share(1, sk, pk0)
    ctx.aggregate_pk([pk0], pk)
    ctx.receiver_keygen(2, rsk, rpk)
    pt = to_dev(np.random.default_rng(bits).integers(0, t, C << log2n, dtype=np.uint64))
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
            call(c, min(part, C - c), parts[c * polys * LN:])
        assert torch.equal(whole, parts), name
    torch.cuda.synchronize()
    ctx.close()


# One ciphertext whose result lies where an input is read: as if it lay elsewhere, though its limbs and components could go to several workgroups
@pytest.mark.gpu
@pytest.mark.parametrize("bits,log2n,L", [(30, 10, 1), (54, 10, 6), (36, 11, 5), (60, 12, 2), (54, 13, 4), (60, 13, 1)])
def test_one_ciphertext_in_place(bits, log2n, L):
    from oracle import oracle as O
    import torch
    from gpu_util import dzeros, make_ctx, to_dev
    N, LN, t = 1 << log2n, L << log2n, 12289 if log2n <= 11 else 65537
    ctx = make_ctx(log2n, O.find_primes(bits, log2n, L), t, f=3, max_group=2, seed=34)
    sk, pk0, pk, rsk, rpk = (dzeros(n * LN) for n in (2, 1, 4, 2, 4))
    ctx.keygen_share(1, sk, pk0)
    ctx.aggregate_pk([pk0], pk)
    ctx.receiver_keygen(2, rsk, rpk)
    pt = to_dev(np.random.default_rng(bits).integers(0, t, N, dtype=np.uint64))
    ct, alpha = dzeros(2 * LN), dzeros(LN)
    ctx.encrypt(pk, pt, 1, 1, 5, 3, ct)
    ctx.bootstrap_alpha(5, 3, 1, alpha)
    shares = [dzeros(2 * LN) for _ in range(2)]
    for k in range(2):
        ctx.bootstrap_share(sk, ct, alpha, 1, 1 + k, 5, 3, shares[k])
    room = dzeros(6 * LN)

    def check(what, call, data, words, offsets):
        """call(data, out): out `offset` words from where data begins"""
        want = dzeros(words)
        call(data, want)
        for offset in offsets:
            room.zero_()
            at = room[2 * LN:2 * LN + data.numel()]
            at.copy_(data)
            out = room[2 * LN + offset:]
            call(at, out)
            assert torch.equal(out[:words], want), (what, offset)

    check("ciphertext", lambda d, out: ctx.encrypt(pk, d, 1, 1, 5, 3, out), pt, 2 * LN, (0, -LN, N - 2 * LN, -N // 2))
    check("share", lambda d, out: ctx.partial_decrypt(sk, d, 1, 1, 5, 3, out), ct, LN, (0, LN, LN - N))
    check("conversion share", lambda d, out: ctx.convert_share(sk, rpk, d, 1, 1, 2, 5, 3, out), ct, 2 * LN, (0, -N))
    check("refresh share", lambda d, out: ctx.bootstrap_share(sk, d, alpha, 1, 1, 5, 3, out), ct, 2 * LN, (0, -N))
    check("refreshed", lambda d, out: ctx.bootstrap_combine(ct, alpha, [d, shares[1]], 1, out), shares[0], 2 * LN, (0, LN))
    torch.cuda.synchronize()
    ctx.close()
