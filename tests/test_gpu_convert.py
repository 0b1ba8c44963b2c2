"""GPU parity of MBFV.Convert (Sec. 4.2 item 3, Eq. (1)-(2)) through the C ABI: receiver keys,
conversion shares, the converted ciphertext, its single-key decryption and the fused round, every
integer bit-exact against the oracle and every decoded float equal to the fixed-point sum."""
import numpy as np
import pytest
import torch

from paper_2207_04604_amd import binding as B
from oracle import oracle as O
from paper_2207_04604_amd.synth import CONFIGS, toy_config

from gpu_util import DEV, Keys, dzeros, make_pair, to_dev, to_eval, to_host
from test_gpu_parity import fixed_point_sum
from test_pm_policies import primes_away_from_powers_of_two

pytestmark = pytest.mark.gpu


class RecvKeys:
    """Single-key pairs of the receivers on both sides (checked against the oracle)."""

    def __init__(self, o, ctx, perm, parties):
        L, N = o.L, o.N
        self.osk, self.opk, self.sk, self.pk = {}, {}, {}, {}
        for r in parties:
            osk, opk, _, _ = o.receiver_keygen(r)
            dsk, dpk = dzeros(2 * L * N), dzeros(4 * L * N)
            ctx.receiver_keygen(r, dsk, dpk)
            hsk, hpk = to_host(dsk, (2, L, N)), to_host(dpk, (2, 2, L, N))
            assert np.array_equal(hsk[0], to_eval(o, perm, osk)), f"secret key of receiver {r}"
            assert np.array_equal(hpk[0, 0], to_eval(o, perm, opk[0])), f"p0 of receiver {r}"
            assert np.array_equal(hpk[1, 0], to_eval(o, perm, opk[1])), f"p1 of receiver {r}"
            for i in range(L):           # Shoup quotients, spot-checked with Python integers
                for j in range(0, N, 263):
                    for vals, quots in ((hsk[0], hsk[1]), (hpk[0, 0], hpk[0, 1]), (hpk[1, 0], hpk[1, 1])):
                        assert int(quots[i, j]) == (int(vals[i, j]) << 64) // o.q[i]
            self.osk[r], self.opk[r], self.sk[r], self.pk[r] = osk, opk, dsk, dpk


def convert_calls_and_compare(cfg, o, ctx, perm, keys, rkeys, members, receiver, group, grads, ct_base=0):
    """Per-call path for one (group, receiver): every object is compared with the oracle's."""
    L, N = o.L, o.N
    n_values = grads[members[0]].size
    C_ = (n_values + N - 1) // N
    opk, dpk = keys.group_pk(members, perm, check=False)
    dagg, oagg = None, None
    for k in members:
        dpt = dzeros(C_ * N)
        ctx.encode(to_dev(grads[k]), n_values, dpt, C_)
        dct = dzeros(C_ * 2 * L * N)
        ctx.encrypt(dpk, dpt, C_, k, group, ct_base, dct)
        oct_ = o.encrypt(opk, o.encode(grads[k]), k, group, ct_base)
        if dagg is None:
            dagg, oagg = dct, oct_
        else:
            ctx.add(dagg, dct, C_)
            oagg = o.add(oagg, oct_)
    dshares, oshares = [], []
    for k in members:
        dsh = dzeros(C_ * 2 * L * N)
        ctx.convert_share(keys.sk[k], rkeys.pk[receiver], dagg, C_, k, receiver, group, ct_base, dsh)
        osh = o.convert_share(keys.osk[k], rkeys.opk[receiver], oagg, k, receiver, group, ct_base)
        assert np.array_equal(to_host(dsh, osh.shape), to_eval(o, perm, osh)), f"conversion share of party {k}"
        dshares.append(dsh)
        oshares.append(osh)
    dnew = dzeros(C_ * 2 * L * N)
    ctx.convert_combine(dagg, dshares, C_, dnew)
    onew = o.convert_combine(oagg, oshares)
    assert np.array_equal(to_host(dnew, onew.shape), to_eval(o, perm, onew)), "converted ciphertext"
    dout = dzeros(C_ * N)
    ctx.decrypt(rkeys.sk[receiver], dnew, C_, dout)
    oout = o.decrypt_with_secret(rkeys.osk[receiver], onew)
    assert np.array_equal(to_host(dout, (C_, N)), oout), "single-key decryption"
    dres = torch.zeros(n_values, dtype=torch.float32, device=DEV)
    ctx.decode(dout, C_, n_values, dres)
    expect = fixed_point_sum([grads[k] for k in members], cfg.frac_bits, o.encode_clamp())
    assert np.array_equal(dres.cpu().numpy(), expect), "decoded sum"
    assert np.array_equal(o.decode(oout, n_values), expect)
    return dpk, opk


def test_convert_C1_every_coefficient_every_receiver():
    """C1 is a complete graph: one group, and each of its four nodes is a receiver."""
    cfg = CONFIGS["C1"]
    o, ctx, perm = make_pair(cfg)
    grads = cfg.gradients()
    keys = Keys(o, ctx, perm, range(cfg.parties), check=False)
    rkeys = RecvKeys(o, ctx, perm, range(cfg.parties))
    members = cfg.groups()[0]
    for r in members:
        convert_calls_and_compare(cfg, o, ctx, perm, keys, rkeys, members, r, 0, grads)
    ctx.close()


def test_convert_C2_two_groups_every_coefficient():
    cfg = CONFIGS["C2"]
    o, ctx, perm = make_pair(cfg)
    grads = cfg.gradients()
    keys = Keys(o, ctx, perm, range(cfg.parties), check=False)
    groups = cfg.groups()
    rkeys = RecvKeys(o, ctx, perm, [3, 12])
    for g in (3, 12):            # group g is the closed neighbourhood of node g
        assert g in groups[g]
        convert_calls_and_compare(cfg, o, ctx, perm, keys, rkeys, groups[g], g, g, grads)
    ctx.close()


def test_convert_wide_primes_ragged_tail_and_extreme_ids():
    """54- and 60-bit primes (just below a power of two: ArithP and ArithQ), doubles, a ragged last ciphertext, ids at their limits,
    a receiver that is not a member, and the plain single-key path (encrypt under a receiver key)."""
    from oracle import oracle as O
    from paper_2207_04604_amd.synth import toy_config
    for bits, log2n, L in ((54, 11, 2), (60, 10, 2), (36, 13, 2), (54, 14, 2), (60, 14, 1), (44, 14, 1)):
        cfg = toy_config(log2n, O.find_primes(bits, log2n, L), 65537, 3, (1 << log2n) + 77, frac_bits=6)
        o, ctx, perm = make_pair(cfg)
        rng = np.random.default_rng(bits)
        members = [1, 40000, 65535]
        grads = {k: rng.normal(0, 3.0, cfg.n_values).astype(np.float32) for k in members}
        keys = Keys(o, ctx, perm, members, check=False)
        rkeys = RecvKeys(o, ctx, perm, [65535, 7])
        for r in (65535, 7):
            convert_calls_and_compare(cfg, o, ctx, perm, keys, rkeys, members, r, 65535, grads, ct_base=2**32 - 4)
        # BFV.Encrypt under a receiver's own key, BFV.Decrypt with its secret (Sec. 3.2 items 3, 5)
        L_, N = o.L, o.N
        m = rng.integers(0, cfg.t, (2, N), dtype=np.uint64)
        dct = dzeros(2 * 2 * L_ * N)
        ctx.encrypt(rkeys.pk[7], to_dev(m), 2, 7, 0, 0, dct)
        oct_ = o.encrypt(rkeys.opk[7], m, 7, 0, 0)
        assert np.array_equal(to_host(dct, oct_.shape), to_eval(o, perm, oct_))
        dout = dzeros(2 * N)
        ctx.decrypt(rkeys.sk[7], dct, 2, dout)
        assert np.array_equal(to_host(dout, (2, N)), m)
        ctx.close()


# the shapes that the primes above, all just below a power of two, do not reach: quotients (54, 60 bits) with 8 and with 16
# coefficients per thread, 32-bit words with 16
@pytest.mark.parametrize("bits,log2n,L", [(54, 10, 1), (60, 10, 2), (54, 11, 2), (60, 11, 1), (60, 12, 1), (54, 13, 1), (54, 14, 1),
                                          (60, 14, 1), (30, 14, 2), (30, 13, 2), (36, 10, 2)])
def test_convert_other_shapes(bits, log2n, L):
    q = primes_away_from_powers_of_two(bits, log2n, L) if bits > 44 else O.find_primes(bits, log2n, L)
    cfg = toy_config(log2n, q, 12289 if log2n <= 11 else 65537, 3, (1 << log2n) + 77, frac_bits=6)
    o, ctx, perm = make_pair(cfg)
    rng = np.random.default_rng(bits + log2n)
    members = [1, 40000, 65535]
    grads = {k: rng.normal(0, 3.0, cfg.n_values).astype(np.float32) for k in members}
    keys, rkeys = Keys(o, ctx, perm, members, check=False), RecvKeys(o, ctx, perm, [7])
    convert_calls_and_compare(cfg, o, ctx, perm, keys, rkeys, members, 7, 65535, grads, ct_base=2**32 - 4)
    ctx.close()


@pytest.mark.parametrize("name,share_sample,ct_sample", [("C1", [(0, 0, 0), (0, 3, 2)], (0, 3)),
                                                        ("C2", [(0, 0, 0), (7, 0, 2), (15, 0, 4)], (0, 13, 24)),
                                                        ("C3", [(0, 0, 0), (19, 0, 3), (31, 0, 6)], (0, 152))])
def test_convert_round_in_the_benchmark_launch_shape(name, share_sample, ct_sample):
    """All groups in one d2mhe_round_convert call (what bench.py --convert times): every node
    receives the sum over its closed neighbourhood; sampled conversion shares are recomputed by
    the oracle.  share_sample: (group, receiver index, member index)."""
    cfg = CONFIGS[name]
    o, ctx, perm = make_pair(cfg)
    grads = cfg.gradients()
    keys = Keys(o, ctx, perm, range(cfg.parties), check=False)
    groups = cfg.groups()
    receivers = cfg.receivers()
    assert sorted(r for rs in receivers for r in rs) == list(range(cfg.parties))     # every node receives once
    rkeys = RecvKeys(o, ctx, perm, range(cfg.parties))
    pks = [keys.group_pk(g, perm, check=False) for g in groups]
    J = sum(len(g) for g in groups)
    dgr = [to_dev(g) for g in grads]
    unused = [torch.zeros(1, dtype=torch.float32, device=DEV) for _ in groups]
    desc = ctx.make_round(groups, [p[1] for p in pks], [keys.sk[k] for k in range(cfg.parties)], dgr, unused,
                          cfg.n_values)
    outs = [torch.zeros(cfg.n_values, dtype=torch.float32, device=DEV) for rs in receivers for _ in rs]
    conv = ctx.make_convert(desc, receivers, [rkeys.pk[k] for k in range(cfg.parties)],
                            [rkeys.sk[k] for k in range(cfg.parties)], outs)
    S = conv.num_shares
    assert S == sum(len(g) * len(r) for g, r in zip(groups, receivers))
    nbytes = ctx.round_convert_scratch_bytes(J, len(groups), S, cfg.n_values)
    scratch = dzeros(nbytes // 8)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
    for e in evs:                # torch creates the underlying event at the first record
        e.record()
    for rep in range(2):
        ctx.round_convert(desc, conv, scratch, nbytes, [e.cuda_event for e in evs],
                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert all(evs[i].elapsed_time(evs[i + 1]) > 0 for i in range(4))
    clamp = o.encode_clamp()
    i = 0
    for gi, g in enumerate(groups):
        expect = fixed_point_sum([grads[k] for k in g], cfg.frac_bits, clamp)
        for r in receivers[gi]:
            assert np.array_equal(outs[i].cpu().numpy(), expect), f"group {gi} receiver {r}"
            i += 1
    L, N, C_, G = cfg.L, cfg.N, cfg.C, len(groups)
    LN = L * N
    shares = scratch[(J + G) * C_ * 2 * LN:(J + G + S) * C_ * 2 * LN].view(S, C_, 2 * LN)
    first = np.cumsum([0] + [len(g) * len(r) for g, r in zip(groups, receivers)])
    for (gi, ri, mi) in share_sample:
        g, opk = groups[gi], pks[gi][0]
        r = receivers[gi][ri]
        for c in ct_sample:
            lo, hi = c * N, min((c + 1) * N, cfg.n_values)
            oagg = None
            for k in g:
                oct_ = o.encrypt(opk, o.encode(grads[k][lo:hi]), k, gi, c)
                oagg = oct_ if oagg is None else o.add(oagg, oct_)
            osh = o.convert_share(keys.osk[g[mi]], rkeys.opk[r], oagg, g[mi], r, gi, c)
            pos = first[gi] + ri * len(g) + mi
            assert np.array_equal(to_host(shares[pos, c], (1, 2, L, N)), to_eval(o, perm, osh)), (gi, ri, mi, c)
    ctx.close()


def test_convert_argument_checks():
    cfg = CONFIGS["C1"]
    o, ctx, perm = make_pair(cfg)
    L, N = o.L, o.N
    buf = dzeros(4 * L * N)
    with pytest.raises(B.D2mheError) as ei:
        ctx.receiver_keygen(70000, buf, buf)
    assert ei.value.status == B.ERR_RANGE
    with pytest.raises(B.D2mheError) as ei:
        ctx.convert_share(buf, buf, buf, 1, 1, 70000, 0, 0, buf)
    assert ei.value.status == B.ERR_RANGE
    with pytest.raises(B.D2mheError) as ei:
        ctx.convert_combine(buf, [], 1, buf)
    assert ei.value.status == B.ERR_RANGE
    with pytest.raises(B.D2mheError) as ei:
        ctx.decrypt(None, buf, 1, buf)
    assert ei.value.status == B.ERR_NULL
    ctx.convert_share(buf, buf, buf, 0, 1, 2, 0, 0, buf)        # C = 0: nothing to do
    ctx.close()


def test_rounds_with_more_groups_than_one_launch_takes():
    """130 two-member groups over 131 parties: more parties and groups than one launch's table holds (112 and 112 of a
    round, 104 and 64 of conversion shares, 80 receivers), so every phase of both rounds is split over several launches.
    Every group's result against the fixed-point sum, sampled objects against the oracle."""
    P, G = 131, 130
    cfg = toy_config(10, O.find_primes(36, 10, 2), 12289, P, 1024 + 11, frac_bits=4)
    o, ctx, perm = make_pair(cfg, max_group=2)
    L, N, C_, n = o.L, o.N, cfg.C, cfg.n_values
    rng = np.random.default_rng(130)
    grads = [rng.normal(0, 20.0, n).astype(np.float32) for _ in range(P)]
    groups = [[g, g + 1] for g in range(G)]
    receivers = [[g + (g % 2)] for g in range(G)]                 # one of the two members
    keys = Keys(o, ctx, perm, range(P), check=False)
    rkeys = RecvKeys(o, ctx, perm, sorted({r[0] for r in receivers}))
    pks = [keys.group_pk(g, perm, check=False) for g in groups]
    dgr = [to_dev(g) for g in grads]
    outs = [torch.zeros(n, dtype=torch.float32, device=DEV) for _ in groups]
    desc = ctx.make_round(groups, [p[1] for p in pks], [keys.sk[k] for k in range(P)], dgr, outs, n, ct_base=5)
    J = 2 * G
    nbytes = ctx.round_scratch_bytes(J, G, n)
    scratch = dzeros(nbytes // 8)
    ctx.round(desc, scratch, nbytes)
    torch.cuda.synchronize()
    clamp = o.encode_clamp()
    expects = [fixed_point_sum([grads[k] for k in g], cfg.frac_bits, clamp) for g in groups]
    for gi in range(G):
        assert np.array_equal(outs[gi].cpu().numpy(), expects[gi]), f"group {gi}"
    LN = L * N
    cts = scratch[:J * C_ * 2 * LN].view(J, C_, 2 * LN)
    agg = scratch[J * C_ * 2 * LN:(J + G) * C_ * 2 * LN].view(G, C_, 2 * LN)
    shares = scratch[(J + G) * C_ * 2 * LN:(J + G) * C_ * 2 * LN + J * C_ * LN].view(J, C_, LN)
    for gi in (0, 55, 56, 111, 112, 129):                          # around the launch boundaries
        opk = pks[gi][0]
        octs = [o.encrypt(opk, o.encode(grads[k]), k, gi, ct_base=5) for k in groups[gi]]
        oagg = o.add(octs[0], octs[1])
        for m in range(2):
            assert np.array_equal(to_host(cts[2 * gi + m], octs[m].shape), to_eval(o, perm, octs[m])), (gi, m)
            osh = o.partial_decrypt(keys.osk[groups[gi][m]], oagg, groups[gi][m], gi, ct_base=5)
            assert np.array_equal(to_host(shares[2 * gi + m], osh.shape), to_eval(o, perm, osh)), (gi, m)
        assert np.array_equal(to_host(agg[gi], oagg.shape), to_eval(o, perm, oagg)), gi
    del scratch
    routs = [torch.zeros(n, dtype=torch.float32, device=DEV) for _ in range(G)]
    conv = ctx.make_convert(desc, receivers, rkeys.pk, rkeys.sk, routs)
    assert conv.num_shares == 2 * G
    nbytes = ctx.round_convert_scratch_bytes(J, G, conv.num_shares, n)
    scratch = dzeros(nbytes // 8)
    ctx.round_convert(desc, conv, scratch, nbytes)
    torch.cuda.synchronize()
    for gi in range(G):
        assert np.array_equal(routs[gi].cpu().numpy(), expects[gi]), f"receiver of group {gi}"
    cshares = scratch[(J + G) * C_ * 2 * LN:(J + G + 2 * G) * C_ * 2 * LN].view(2 * G, C_, 2 * LN)
    for gi in (39, 40, 79, 80, 129):
        opk = pks[gi][0]
        octs = [o.encrypt(opk, o.encode(grads[k]), k, gi, ct_base=5) for k in groups[gi]]
        oagg = o.add(octs[0], octs[1])
        r = receivers[gi][0]
        for m in range(2):
            osh = o.convert_share(keys.osk[groups[gi][m]], rkeys.opk[r], oagg, groups[gi][m], r, gi, ct_base=5)
            assert np.array_equal(to_host(cshares[2 * gi + m], osh.shape), to_eval(o, perm, osh)), (gi, m)
    ctx.close()
