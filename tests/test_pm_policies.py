"""The arithmetic for moduli just below a power of two (ArithP, ArithQ): contracts on the host, and the
moduli that do not have this form, which keep the quotient-based back-ends, on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("bits", [34, 45, 50, 54, 55, 56, 59, 60, 61])
def test_contracts_of_moduli_just_below_a_power_of_two(tmp_path, bits):
    """tests/arith_pm_check.cpp on 2^bits - c for the smallest c, ones as the prime search gives them, and c up to
    what 2c < 2^32 and the range of the policies let through (55 bits: the end of ArithP, 60: of ArithQ)."""
    cxx = shutil.which("g++") or shutil.which("clang++")
    exe = str(tmp_path / "check")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-w", "-o", exe, os.path.join(ROOT, "tests", "arith_pm_check.cpp")])
    cs = [1, 3, (1 << 15) - 1, 262143, 5275647, 36044799, (1 << 26) - 1, (1 << 31) - 1]
    out = subprocess.run([exe] + [str((1 << bits) - c) for c in cs], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    narrow, wide = (int(out.stdout.split()[i]) for i in (2, 5))
    assert (narrow >= 5) == (45 <= bits <= 55) and (wide >= 5) == (45 <= bits <= 60), out.stdout


def primes_away_from_powers_of_two(bits, log2n, count):
    """Primes = 1 (mod 2N) around 1.37 * 2^(bits - 1)."""
    from oracle import oracle as O
    step, found = 2 << log2n, []
    q = int(1.37 * 2 ** (bits - 1)) // step * step + 1
    while len(found) < count:
        if O.is_prime(q):
            found.append(q)
        q += step
    return found


@pytest.mark.gpu
@pytest.mark.parametrize("log2n,bits", [(10, 45), (13, 55), (14, 54), (16, 50), (12, 56), (14, 61), (16, 60)])
def test_moduli_of_any_other_form(log2n, bits):
    """Moduli far from a power of two: transforms of random and extreme polynomials and, where the scheme covers the
    ring, every object of a round."""
    from oracle import oracle as O
    from paper_2207_04604_amd.synth import toy_config
    from gpu_util import Keys, make_ctx, make_pair, to_dev, to_eval, to_host
    from test_gpu_parity import run_calls_and_compare
    N, q = 1 << log2n, primes_away_from_powers_of_two(bits, log2n, 2)
    o = O.Oracle(log2n, q, 0, 21, 0, 1, 77)
    ctx = make_ctx(log2n, q, 0, seed=77)
    polys = o.bench_polys(3)
    polys[1] = np.array(q, dtype=np.uint64)[:, None] - 1
    d = to_dev(polys.reshape(-1))
    ctx.ntt_forward(d, 3)
    assert np.array_equal(to_host(d, polys.shape), to_eval(o, ctx.index_map(), polys)), "forward transform"
    ctx.ntt_inverse(d, 3)
    assert np.array_equal(to_host(d, polys.shape), polys), "inverse transform"
    ctx.close()
    if log2n <= 14:
        cfg = toy_config(log2n, q, 12289 if log2n <= 11 else 65537, parties=2, n_values=N + 37, frac_bits=5)
        o, ctx, perm = make_pair(cfg, max_group=2)
        rng = np.random.default_rng(log2n)
        grads = {k: rng.normal(0, 6.0, cfg.n_values).astype(np.float32) for k in range(2)}
        run_calls_and_compare(cfg, o, ctx, perm, Keys(o, ctx, perm, range(2)), [0, 1], 4, grads, ct_base=9)
        ctx.close()
