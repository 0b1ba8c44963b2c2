"""The work that a program built on this library has it do, through the public entry points of
``paper_2207_04604_amd.binding``, as cases that can be timed.

Five kinds of pass:

``round``      one exchange round of all neighbourhoods (encode + encrypt, sum, decryption shares,
               combine + decode), on one device; with ``convert`` the paper's own decryption path (key
               switching to every receiver); with ``update`` also the float step of a training iteration
``node``       what one node of a deployment does for its own messages of a round: encode and encrypt its
               vector, make its decryption share of the neighbourhood's aggregate
``receiver``   what the node that collects the shares does: combine, decode, update its weights
``bootstrap``  collective refresh of aggregated ciphertexts
``ntt``        the batched negacyclic transform by itself, either direction

Parameter sets follow ``paper_2207_04604_amd.synth``: primes 2^b - k 2N + 1, 30 to 60 bits, rings of degree
2^10 to 2^16, neighbourhoods of rings, complete graphs and random graphs of a given connection rate.
"""
import math
import random

import torch

from paper_2207_04604_amd import binding
from paper_2207_04604_amd.synth import CBD_ETA, closed_neighbourhood_groups

DEV = "cuda:0"


# ---- parameter sets ---------------------------------------------------------------------------------------

def _is_prime(n):
    odd, twos = n - 1, 0
    while odd % 2 == 0:
        odd, twos = odd // 2, twos + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if n % a == 0:
            return n == a
        y = pow(a, odd, n)
        if y in (1, n - 1):
            continue
        for _ in range(twos - 1):
            y = y * y % n
            if y == n - 1:
                break
        else:
            return False
    return True


_primes = {}


def primes(bits, log2n, count):
    """The largest `count` primes 2^bits - k 2N + 1 (the rule of synth.py)."""
    found = _primes.setdefault((bits, log2n), [])
    k = ((1 << bits) - found[-1]) // (2 << log2n) + 2 if found else 1
    while len(found) < count:
        q = (1 << bits) - k * (2 << log2n) + 1
        if _is_prime(q):
            found.append(q)
        k += 1
    return found[:count]


def adjacency(case):
    P, graph = case["parties"], case["graph"]
    if graph == "complete":
        return [[j for j in range(P) if j != i] for i in range(P)]
    if graph == "ring":                                     # circulant: `reach` neighbours on either side
        return [sorted({(i + d) % P for d in range(-case["reach"], case["reach"] + 1)} - {i}) for i in range(P)]
    rng = random.Random(P * 1000 + int(case["rate"] * 100))  # "random": every pair is connected at `rate`
    adj = [set() for _ in range(P)]
    for i in range(P):
        for j in range(i):
            if rng.random() < case["rate"]:
                adj[i].add(j)
                adj[j].add(i)
    for i in range(P):
        if not adj[i]:
            adj[i].add((i + 1) % P)
            adj[(i + 1) % P].add(i)
    return [sorted(a)[:31] for a in adj]                    # at most 32 members in a closed neighbourhood


def plaintext_modulus(case):
    return 12289 if case["log2n"] <= 11 else 65537


def listed():
    return [
        # the smallest round of the repository's configurations: four nodes, four ciphertexts each, 30-bit prime
        {"name": "round_small", "kind": "round", "log2n": 10, "bits": 30, "limbs": 1, "graph": "complete", "parties": 4,
         "values": 4096, "frac": 8, "packing": 0, "convert": False, "update": False},
        # an MNIST-sized model on a ring of 16 nodes
        {"name": "round_ring16", "kind": "round", "log2n": 12, "bits": 36, "limbs": 3, "graph": "ring", "reach": 2,
         "parties": 16, "values": 101770, "frac": 10, "packing": 0, "convert": False, "update": False},
        # a CIFAR-sized model, 32 nodes with six neighbours each: the headline round of the benchmark
        {"name": "round_graph32", "kind": "round", "log2n": 13, "bits": 54, "limbs": 4, "graph": "ring", "reach": 3,
         "parties": 32, "values": 1250000, "frac": 12, "packing": 0, "convert": False, "update": False},
        # the largest vector: an 11-million-parameter model, eight nodes that all know each other, eight limbs
        {"name": "round_complete8", "kind": "round", "log2n": 14, "bits": 54, "limbs": 8, "graph": "complete",
         "parties": 8, "values": 11200000, "frac": 14, "packing": 0, "convert": False, "update": False},
        # the paper's population: 100 users at connection rate 0.2, so neighbourhoods of many different sizes; a
        # short ragged vector
        {"name": "round_users100", "kind": "round", "log2n": 12, "bits": 54, "limbs": 2, "graph": "random", "rate": 0.2,
         "parties": 100, "values": 19371, "frac": 8, "packing": 0, "convert": False, "update": False},
        # training iteration with coefficient packing on 12 nodes, 44-bit primes, ragged vector
        {"name": "train_packed12", "kind": "round", "log2n": 11, "bits": 44, "limbs": 2, "graph": "ring", "reach": 1,
         "parties": 12, "values": 61706, "frac": 6, "packing": 1, "convert": False, "update": True},
        # the paper's decryption path on the 32-node graph
        {"name": "convert_graph32", "kind": "round", "log2n": 13, "bits": 54, "limbs": 4, "graph": "ring", "reach": 3,
         "parties": 32, "values": 300001, "frac": 12, "packing": 0, "convert": True, "update": False},
        # one node's own work for its neighbourhood, message by message
        {"name": "node_1250000", "kind": "node", "log2n": 13, "bits": 54, "limbs": 4, "members": 7, "values": 1250000,
         "frac": 12},
        # the collecting node's work, a small model
        {"name": "receiver_101770", "kind": "receiver", "log2n": 12, "bits": 36, "limbs": 3, "members": 5,
         "values": 101770, "frac": 10},
        # seven members refresh the aggregates of a 1.25-million-value vector
        {"name": "bootstrap_153", "kind": "bootstrap", "log2n": 13, "bits": 54, "limbs": 4, "members": 7, "batch": 153,
         "frac": 12},
        # the long transform of the benchmark, each direction
        {"name": "ntt_forward_65536", "kind": "ntt", "log2n": 16, "bits": 60, "limbs": 16, "batch": 64, "inverse": False},
        {"name": "ntt_inverse_65536", "kind": "ntt", "log2n": 16, "bits": 60, "limbs": 16, "batch": 64, "inverse": True},
    ]


def _spread(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "node", "receiver", "bootstrap", "ntt", "ntt"])
    if kind == "ntt":
        case = {"kind": kind, "log2n": rng.randint(10, 16), "bits": rng.choice([30, 36, 44, 50, 54, 60]),
                "limbs": rng.randint(1, 16), "inverse": rng.random() < 0.5}
        most = (1 << 26) // (case["limbs"] << case["log2n"])        # no more coefficients than the listed batches
        case["batch"] = _spread(rng, 1, max(2, most))
        return case
    log2n = rng.randint(10, 14)
    case = {"kind": kind, "log2n": log2n, "bits": rng.choice([36, 44, 50, 54, 60] if log2n > 10 else [30, 36, 44, 54]),
            "frac": rng.randint(6, 12)}
    case["limbs"] = rng.randint(1, 2) if case["bits"] == 30 else rng.randint(1 if case["bits"] > 44 else 2, 8)
    n = 1 << log2n
    if kind != "round":
        case["members"] = rng.randint(2, 16)
        # largest: some 40 million limb coefficients in all messages of a member
        most = max(2, 40_000_000 // (case["limbs"] * n))
        batch = _spread(rng, 1, min(800, most))
        if kind == "bootstrap":
            case["batch"] = batch
        else:
            case["values"] = max(1, batch * n - rng.randrange(n))
        return case
    case["graph"] = rng.choice(["ring", "ring", "complete", "random"])
    case["parties"] = _spread(rng, 3, 100) if case["graph"] != "complete" else rng.randint(2, 12)
    if case["graph"] == "ring":
        case["reach"] = rng.randint(1, max(1, min(5, (case["parties"] - 1) // 2)))
    if case["graph"] == "random":
        case["rate"] = rng.choice([0.1, 0.2, 0.3])
    case["packing"] = int(rng.random() < 0.2)
    case["convert"] = rng.random() < 0.25
    case["update"] = rng.random() < 0.3
    groups, owner = closed_neighbourhood_groups(adjacency(case))
    jobs = sum(len(g) for g in groups) * 2
    if case["convert"]:
        jobs += sum(len(groups[g]) for g in owner)
    # largest: about a tenth of the coefficients of the listed large rounds, so that odd shapes stay quick
    most = max(1, 100_000_000 // (jobs * case["limbs"] * n))
    case["values"] = max(1, _spread(rng, 1, max(2, most)) * n - rng.randrange(n))
    return case


# ---- what a program holds before the pass ------------------------------------------------------------------

def _words(n):
    return torch.empty(n, dtype=torch.int64, device=DEV)


def _floats(rows, n):
    """`rows` float vectors of n values, each 16-byte aligned; the padding is zero."""
    return torch.zeros((rows, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)


def _gradients(case, seed, rows):
    """Laplace-distributed model updates (sharply peaked, as gradients are)."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n = case["values"]
    out = _floats(rows, n)
    for r in range(rows):
        u = torch.rand(n, generator=gen, device=DEV) - 0.5
        out[r, :n] = -0.005 * torch.sign(u) * torch.log1p(-2 * u.abs().clamp(max=0.4999999))
    return out


def _context(case, seed, max_group, scheme=True):
    q = primes(case["bits"], case["log2n"], case["limbs"])
    return binding.Context(case["log2n"], q, plaintext_modulus(case) if scheme else 0, CBD_ETA, case.get("frac", 0),
                           max_group, (0x0123456789ABCDEF + 0x9E3779B97F4A7C15 * seed) % (1 << 64),
                           alloc=lambda nbytes: torch.zeros(nbytes // 8 + 2, dtype=torch.int64, device=DEV))


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _key_shares(ctx, parties):
    LN = ctx.L * ctx.N
    sks, pk0 = [_words(2 * LN) for _ in range(parties)], [_words(LN) for _ in range(parties)]
    for k in range(parties):
        ctx.keygen_share(k, sks[k], pk0[k], _stream())
    return sks, pk0


def _public_key(ctx, pk0):
    pk = _words(4 * ctx.L * ctx.N)
    ctx.aggregate_pk(pk0, pk, _stream())
    return pk


def _prepare_round(case, seed):
    groups, owner = closed_neighbourhood_groups(adjacency(case))
    n, P = case["values"], case["parties"]
    ctx = _context(case, seed, max(len(g) for g in groups))
    sks, pk0 = _key_shares(ctx, P)
    pks = [_public_key(ctx, [pk0[k] for k in g]) for g in groups]
    jobs = sum(len(g) for g in groups)
    LN = ctx.L * ctx.N
    s = {"ctx": ctx, "grads": _gradients(case, seed, P), "keys": (sks, pks), "groups": groups, "owner": owner, "P": P, "n": n}
    s["sums"] = _floats(len(groups), n)
    s["desc"] = ctx.make_round(groups, pks, sks, list(s["grads"]), list(s["sums"]), n, ct_base=3, packing=case["packing"])
    if case["convert"]:
        receivers = [[i for i, g in enumerate(owner) if g == gi] for gi in range(len(groups))]
        rsk, rpk = [_words(2 * LN) for _ in range(P)], [_words(4 * LN) for _ in range(P)]
        for k in range(P):
            ctx.receiver_keygen(k, rsk[k], rpk[k], _stream())
        s["recv_keys"] = (rsk, rpk)
        s["sums"] = _floats(P, n)                            # one result per receiver
        s["row"] = [0] * P                                   # the row of a node's own result
        at = 0
        for rs in receivers:
            for i in rs:
                s["row"][i] = at
                at += 1
        s["conv"] = ctx.make_convert(s["desc"], receivers, rpk, rsk, list(s["sums"]))
        s["bytes"] = ctx.round_convert_scratch_bytes(jobs, len(groups), s["conv"].num_shares, n)
    else:
        s["row"] = owner
        s["conv"] = None
        s["bytes"] = ctx.round_scratch_bytes(jobs, len(groups), n)
    s["scratch"] = _words(s["bytes"] // 8)
    s["weights"] = _floats(P, n) if case["update"] else None
    return s


def _run_round(s):
    ctx, st = s["ctx"], _stream()
    if s["conv"] is None:
        ctx.round(s["desc"], s["scratch"], s["bytes"], None, st)
    else:
        ctx.round_convert(s["desc"], s["conv"], s["scratch"], s["bytes"], None, st)
    if s["weights"] is None:
        return {"sums": s["sums"], "messages": s["scratch"]}
    for i in range(s["P"]):
        binding.average_update(s["sums"][s["row"][i]], len(s["groups"][s["owner"][i]]), s["grads"][i], 0.01, s["n"],
                               s["weights"][i], st)
    return {"sums": s["sums"], "messages": s["scratch"], "weights": s["weights"]}


def _prepare_group(case, seed):
    """A neighbourhood's keys, its members' vectors and the aggregate of their ciphertexts."""
    K, n = case["members"], case.get("values") or case["batch"] << case["log2n"]
    ctx = _context(case, seed, K)
    C, LN = (n + ctx.N - 1) // ctx.N, ctx.L * ctx.N
    sks, pk0 = _key_shares(ctx, K)
    pk = _public_key(ctx, pk0)
    grads = _gradients(dict(case, values=n), seed, K)
    pt, ct, agg = _words(C * ctx.N), _words(C * 2 * LN), _words(C * 2 * LN)
    for k in range(K):
        ctx.encode(grads[k], n, pt, C, _stream())
        ctx.encrypt(pk, pt, C, k, 5, 0, ct if k else agg, _stream())
        if k:
            ctx.add(agg, ct, C, _stream())
    return {"ctx": ctx, "K": K, "n": n, "C": C, "LN": LN, "sks": sks, "pk": pk, "grads": grads, "agg": agg, "pt": pt, "ct": ct}


def _prepare_node(case, seed):
    s = _prepare_group(case, seed)
    s["share"] = _words(s["C"] * s["LN"])
    return s


def _run_node(s):
    ctx, st = s["ctx"], _stream()
    ctx.encode(s["grads"][0], s["n"], s["pt"], s["C"], st)
    ctx.encrypt(s["pk"], s["pt"], s["C"], 0, 5, 0, s["ct"], st)
    ctx.partial_decrypt(s["sks"][0], s["agg"], s["C"], 0, 5, 0, s["share"], st)
    return {"ciphertexts": s["ct"], "share": s["share"]}


def _prepare_receiver(case, seed):
    s = _prepare_group(case, seed)
    s["shares"] = [_words(s["C"] * s["LN"]) for _ in range(s["K"])]
    for k in range(s["K"]):
        s["ctx"].partial_decrypt(s["sks"][k], s["agg"], s["C"], k, 5, 0, s["shares"][k], _stream())
    s["out"], s["weights"] = _floats(1, s["n"])[0], _floats(1, s["n"])[0]
    return s


def _run_receiver(s):
    ctx, st = s["ctx"], _stream()
    ctx.combine(s["agg"], s["shares"], s["C"], s["pt"], st)
    ctx.decode(s["pt"], s["C"], s["n"], s["out"], st)
    binding.average_update(s["out"], s["K"], s["grads"][0], 0.01, s["n"], s["weights"], st)
    return {"plaintexts": s["pt"], "sum": s["out"], "weights": s["weights"]}


def _prepare_bootstrap(case, seed):
    s = _prepare_group(case, seed)
    s["alpha"] = _words(s["C"] * s["LN"])
    s["shares"] = [_words(s["C"] * 2 * s["LN"]) for _ in range(s["K"])]
    return s


def _run_bootstrap(s):
    ctx, st = s["ctx"], _stream()
    ctx.bootstrap_alpha(5, 0, s["C"], s["alpha"], st)
    for k in range(s["K"]):
        ctx.bootstrap_share(s["sks"][k], s["agg"], s["alpha"], s["C"], k, 5, 0, s["shares"][k], st)
    ctx.bootstrap_combine(s["agg"], s["alpha"], s["shares"], s["C"], s["ct"], st)
    return {"ciphertexts": s["ct"], "shares": s["shares"]}


def _prepare_ntt(case, seed):
    ctx = _context(case, seed, 1, scheme=False)
    polys = _words(case["batch"] * ctx.L * ctx.N)
    ctx.bench_polys(polys, case["batch"], _stream())         # uniform residues
    return {"ctx": ctx, "polys": polys, "batch": case["batch"],
            "call": ctx.ntt_inverse if case["inverse"] else ctx.ntt_forward}


def _run_ntt(s):
    s["call"](s["polys"], s["batch"], _stream())             # in place; the result is a batch of residues again
    return {"polynomials": s["polys"]}


KINDS = {"round": (_prepare_round, _run_round), "node": (_prepare_node, _run_node),
         "receiver": (_prepare_receiver, _run_receiver), "bootstrap": (_prepare_bootstrap, _run_bootstrap),
         "ntt": (_prepare_ntt, _run_ntt)}


def prepare(case, seed):
    s = KINDS[case["kind"]][0](case, seed)
    s["run"] = KINDS[case["kind"]][1]
    return s


def run(state):
    return state["run"](state)


# ---- what the pass cannot do without -----------------------------------------------------------------------

def work(case):
    """Bytes: every input (vectors, keys, ciphertexts a call is given) read once, every output (ciphertexts,
    shares, sums) written once.  Operations: three modular ones (a product, a sum, a difference) per butterfly of the
    transforms, two per product with a key, one per addition of a residue."""
    N, L = 1 << case["log2n"], case["limbs"]
    poly, ntt, LN = 8 * N * L, 3 * L * (N // 2) * case["log2n"], L * N
    plain = 3 * (N // 2) * case["log2n"]                     # one transform modulo t
    if case["kind"] == "ntt":
        return {"bytes": 2 * case["batch"] * poly, "flops": case["batch"] * ntt}
    n = case.get("values") or case["batch"] * N
    C = (n + N - 1) // N
    encrypt, share, combine = 3 * ntt + plain + 5 * LN, ntt + 2 * LN, ntt + plain + 2 * LN
    if case["kind"] == "node":
        return {"bytes": C * 4 * poly + 4 * n + 6 * poly, "flops": C * (encrypt + share)}
    if case["kind"] == "receiver":
        K = case["members"]
        return {"bytes": C * (K + 1) * poly + 8 * C * N + 12 * n, "flops": C * (combine + K * LN)}
    if case["kind"] == "bootstrap":
        K = case["members"]
        return {"bytes": C * (2 + 1 + 2 * K + 2) * poly + 2 * K * poly,
                "flops": C * (ntt + K * (2 * ntt + 5 * LN) + 2 * ntt + (2 * K + 2) * LN)}
    groups, owner = closed_neighbourhood_groups(adjacency(case))
    J, G, P = sum(len(g) for g in groups), len(groups), case["parties"]
    nbytes = 4 * n * P + C * poly * (2 * J + 2 * G)          # vectors in, fresh ciphertexts and aggregates out
    nbytes += P * 2 * poly + G * 4 * poly                    # keys
    flops = C * (J * (encrypt if not case["packing"] else encrypt - plain) + 2 * J * LN)
    if case["convert"]:
        S = sum(len(groups[g]) for g in owner)
        nbytes += C * S * 2 * poly + 4 * n * P + P * 6 * poly
        flops += C * (S * (3 * ntt + 6 * LN + 2 * LN) + P * (combine + 2 * LN))
    else:
        nbytes += C * J * poly + 4 * n * G
        flops += C * (J * (share + LN) + G * combine)
    if case["update"]:
        nbytes += 4 * n * P * 2
        flops += 3 * n * P
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Residues are whole numbers, and a decoded sum or a float step is defined operation by operation: bit for bit."""
    return "exact"
