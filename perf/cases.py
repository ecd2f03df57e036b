"""What users of this framework have it do, as cases to be timed: single
homomorphic operations at the parameter sets of the repository's workloads,
raw transforms, client-side encryption, an op list, and whole inferences.

listed() gives the named cases, draw(rng) more of the same ranges, prepare()
what a program holds before the call, run() one pass through the public entry
points, work() what a pass cannot do without, exact() the same outputs by
plain integer arithmetic where that is cheap.

Ciphertexts are made as uniform residues: an RLWE ciphertext is
indistinguishable from that.  Documents and client messages go through the
encoder and ENC.  A server keeps its context, keys and model for many inputs,
so these are kept per parameter set; everything that comes with a request is
made from the seed.
"""

import json
import os

import numpy as np
import torch

import paper_1908_06972_amd
from paper_1908_06972_amd import ckks
from paper_1908_06972_amd.inference import BowModel, encrypted_inference, split_counts
from paper_1908_06972_amd.training import EncryptedBowModel, bsgs_plan, predict_encrypted, rotation_steps

# log2 N, ciphertext primes, bits of q_0 and of the others, special primes,
# their bits, digits, log2 of the scale
SETS = {
    "n12": (12, 2, 40, 40, 1, 50, 2, 30),    # single operations
    "n13": (13, 5, 40, 40, 1, 60, 5, 40),    # the paper's inference ring
    "n14": (14, 8, 60, 40, 2, 60, 4, 40),    # batched primitives
    "n15": (15, 16, 60, 40, 4, 60, 4, 40),   # bag of words
    "n16": (16, 24, 60, 50, 6, 60, 4, 50),   # large ring
}
KEY_SEED = 7
DIM, CLASSES, N_IN = 64, 8, 2  # the bag-of-words model: 32768 words, 64 dimensions, 8 classes
PREDICT_LEVEL = 6              # encrypted weights: five levels are consumed


def listed():
    return [
        # the smallest call: one product of two ciphertexts and its rescale; launches and latency
        {"name": "hmult_n12_b1", "op": "hmult", "set": "n12", "level": 2, "batch": 1, "rescale": True},
        # plaintext affine map on one ciphertext at an odd level: mul_plain, add, rescale
        {"name": "affine_n14_l5_b1", "op": "affine", "set": "n14", "level": 5, "batch": 1},
        # 64 pairs of mixed levels through the op-list executor
        {"name": "oplist_n14_p64", "op": "oplist", "set": "n14", "pairs": 64, "mix": 202},
        # both directions of the raw transform over the whole chain
        {"name": "ntt_n16_l24_p8", "op": "ntt", "set": "n16", "level": 24, "polys": 8},
        # a client's side: encrypt a message from host memory, decrypt the answer to it
        {"name": "encdec_n15_l16", "op": "encdec", "set": "n15", "level": 16},
        # HMULT with relinearisation at the top of the large ring: one ciphertext, and a full batch
        {"name": "hmult_n16_l24_b1", "op": "hmult", "set": "n16", "level": 24, "batch": 1, "rescale": False},
        {"name": "hmult_n16_l24_b16", "op": "hmult", "set": "n16", "level": 24, "batch": 16, "rescale": False},
        # rotation of a few ciphertexts with a ragged last digit
        {"name": "rotate_n16_l17_b5", "op": "rotate", "set": "n16", "level": 17, "batch": 5, "log_step": 9},
        # depth-8 product chain then rotate-and-sum over all slots
        {"name": "chain_n16_b16", "op": "chain", "set": "n16", "level": 24, "batch": 16, "depth": 8, "log_slots": 15},
        # encrypted bag-of-words inference: one document's latency, and a batch's throughput
        {"name": "bow_n15_d1", "op": "bow", "set": "n15", "docs": 1},
        {"name": "bow_n15_d32", "op": "bow", "set": "n15", "docs": 32},
        # the predict step with encrypted weights on a few documents
        {"name": "predict_n15_d6", "op": "predict", "set": "n15", "docs": 6},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(["hmult", "hmult", "rotate", "rotate", "affine", "ntt", "encdec", "chain", "oplist", "bow",
                     "predict"])
    s = {"oplist": "n14", "bow": "n15", "predict": "n15"}.get(op) or rng.choice(sorted(SETS))
    levels = SETS[s][1]
    case = {"op": op, "set": s}
    if op in ("hmult", "rotate", "affine", "chain"):
        case["level"] = rng.randint(2, levels)
        case["batch"] = _log_int(rng, 1, 24)
    if op == "hmult":
        case["rescale"] = rng.random() < 0.5
    elif op == "rotate":
        case["log_step"] = rng.randint(0, SETS[s][0] - 2)
    elif op == "ntt":
        case["level"] = rng.randint(1, levels)
        case["polys"] = _log_int(rng, 1, 40)
    elif op == "encdec":
        case["level"] = rng.randint(1, levels)
    elif op == "chain":
        case["batch"] = min(case["batch"], 16)
        case["depth"] = rng.randint(1, min(8, case["level"] - 1))
        case["log_slots"] = rng.randint(1, SETS[s][0] - 1)
    elif op == "oplist":
        case["pairs"] = rng.randint(3, 64)
        case["mix"] = rng.randint(0, 999)
    elif op == "bow":
        case["docs"] = _log_int(rng, 1, 31)
    elif op == "predict":
        case["docs"] = rng.randint(1, 16)
    return case


# ---- what a server keeps: parameters, context, keys, models

_worlds = {}


class _World:
    def __init__(self, name):
        log_n, n_q, q0, qb, n_p, pb, dnum, log_scale = SETS[name]
        self.params = ckks.Params(log_n, n_q, q0, qb, n_p, pb, dnum, 2.0 ** log_scale)
        self.ctx = ckks.Context(self.params, 0)
        steps = {1 << k for k in range(log_n - 1)}
        if name == "n15":
            t = self.params.n // 2
            steps.update(rotation_steps(DIM, t, N_IN), rotation_steps(DIM, t), rotation_steps(CLASSES, DIM))
        if name == "n14":
            self.list_steps = [int(x) for x in np.random.default_rng(203).integers(1, self.params.n // 2, size=16)]
            steps.update(self.list_steps)
        if name == "n16":
            # the schedule table that ships for this ring
            path = os.path.join(os.path.dirname(paper_1908_06972_amd.__file__), "tuning", "large_ring_n16_l24.json")
            with open(path) as fh:
                self.ctx.ntt_tuning_import([(e[0], e[1], (tuple(e[2]), int(e[3]))) for e in json.load(fh)])
        self.ctx.keygen(KEY_SEED, sorted(steps))
        self.models = {}

    def bow_model(self):
        if "bow" not in self.models:
            g = np.random.default_rng(404)
            H, O = g.normal(0.0, 0.1, (32768, DIM)), g.normal(0.0, 0.1, (DIM, CLASSES))
            self.models["bow"] = BowModel(self.ctx, H, O, self.params.L)
        return self.models["bow"]

    def encrypted_model(self):
        if "enc" not in self.models:
            p, lv = self.params, PREDICT_LEVEL
            gen = torch.Generator(device="cuda").manual_seed(62)

            def diagonals(n_o, n_in, level):
                b, G = bsgs_plan(n_o, n_in)
                return [_cipher(p, gen, level, float(p.q[level - 1])) for _ in range(n_in * b * G)]

            self.models["enc"] = EncryptedBowModel(diagonals(DIM, N_IN, lv), diagonals(CLASSES, 1, lv - 2), DIM,
                                                   CLASSES, N_IN, p.n // 2)
        return self.models["enc"]


def _world(name):
    if name not in _worlds:
        _worlds[name] = _World(name)
    return _worlds[name]


def _residues(q, n, polys, gen, out=None):
    """[polys][len(q)][n] uniform residues on the GPU."""
    t = torch.empty((polys, len(q), n), dtype=torch.int64, device="cuda") if out is None else out
    for i, m in enumerate(q):
        t[:, i] = torch.randint(0, m, (polys, n), generator=gen, dtype=torch.int64, device="cuda")
    return t


def _cipher(p, gen, level, scale, out=None):
    return ckks.Ciphertext(_residues(p.q[:level], p.n, 2, gen, out), level, scale)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)


def _zipf_documents(seed, n_docs, vocab):
    g = np.random.default_rng(int(seed))
    perm = np.random.default_rng(7).permutation(vocab)
    cdf = np.cumsum(1.0 / np.arange(1, vocab + 1))
    cdf /= cdf[-1]
    counts = np.zeros((n_docs, vocab))
    words = g.integers(50, 501, size=n_docs)
    for d in range(n_docs):
        ranks = np.searchsorted(cdf, g.random(int(words[d])), side="right")
        np.add.at(counts[d], perm[np.minimum(ranks, vocab - 1)], 1.0)
    return counts, [int(w) for w in words]


# ---- prepare and run

def prepare(case, seed):
    w = _world(case["set"])
    p, ctx, op = w.params, w.ctx, case["op"]
    gen = _generator(seed)
    s = {"op": op, "ctx": ctx, "case": case}
    if op == "hmult":
        for k in ("a", "b"):
            s[k] = [_cipher(p, gen, case["level"], p.scale) for _ in range(case["batch"])]
    elif op in ("rotate", "chain"):
        s["a"] = [_cipher(p, gen, case["level"], p.scale) for _ in range(case["batch"])]
    elif op == "affine":
        lv = case["level"]
        s["a"] = [_cipher(p, gen, lv, p.scale) for _ in range(case["batch"])]
        s["b"] = [_cipher(p, gen, lv, p.scale * p.scale) for _ in range(case["batch"])]
        s["p"] = ckks.Plaintext(_residues(p.q[:lv], p.n, 1, gen)[0].contiguous(), lv, p.scale)
    elif op == "ntt":
        s["x"] = _residues(p.q[:case["level"]], p.n, case["polys"], gen)
        s["y"] = _residues(p.q[:case["level"]], p.n, case["polys"], gen)
        s["fx"], s["iy"] = torch.empty_like(s["x"]), torch.empty_like(s["y"])
    elif op == "encdec":
        z = np.random.default_rng(int(seed)).uniform(-1.0, 1.0, p.n // 2)
        s["m"] = p.encode(z)
        s["level"], s["scale"], s["seed"] = case["level"], p.scale, int(seed) + 11
        s["answer"] = _cipher(p, gen, case["level"], p.scale)
    elif op == "oplist":
        _op_list(s, w, gen, case["pairs"], case["mix"])
    elif op == "bow":
        s["model"] = w.bow_model()
        counts, s["words"] = _zipf_documents(seed, case["docs"], 32768)
        s["docs"] = [[ctx.encrypt_seeded(p.encode(v), p.L, p.scale, int(seed) * 64 + 2 * d + c)
                      for c, v in enumerate(split_counts(counts[d], N_IN, p.n // 2))] for d in range(case["docs"])]
    elif op == "predict":
        s["model"] = w.encrypted_model()
        s["words"] = [int(x) for x in np.random.default_rng(int(seed)).integers(50, 501, size=case["docs"])]
        s["docs"] = [[_cipher(p, gen, PREDICT_LEVEL, p.scale) for _ in range(N_IN)] for _ in range(case["docs"])]
    return s


def _op_list(s, w, gen, pairs, mix):
    """Per pair (a, b) at a level of 3..8 (the list's mix draws them):
    m = HMult+relin(a, b), r = RESCALE(m), t = ROTATE(r), s = t + r; every
    fourth pair also takes a copy of a through NTT and INTT.  Every result
    lives in one buffer."""
    p = w.params
    levels = np.random.default_rng(mix).integers(3, p.L + 1, size=pairs)
    cts, ops, outs, copies = [], [], [], []
    for i, lv in enumerate(int(x) for x in levels):
        cts += [_cipher(p, gen, lv, p.scale) for _ in range(2)]
        outs += [lv, lv - 1, lv - 1, lv - 1] + ([lv] if i % 4 == 0 else [])
    arena = torch.zeros(sum(2 * lv * p.n for lv in outs), dtype=torch.int64, device="cuda")
    at = 0
    for lv in outs:
        size = 2 * lv * p.n
        cts.append(ckks.Ciphertext(arena[at:at + size].view(2, lv, p.n), lv, p.scale))
        at += size
    k = 2 * pairs
    for i in range(pairs):
        ops += [("mul_relin", 2 * i, 2 * i + 1, k, 0, 0), ("rescale", k, 0, k + 1, 0, 0),
                ("rotate", k + 1, 0, k + 2, w.list_steps[i % len(w.list_steps)], 0), ("add", k + 2, k + 1, k + 3, 0, 0)]
        k += 4
        if i % 4 == 0:
            copies.append((k, 2 * i))
            ops += [("ntt", k, 0, 0, 0, 0), ("intt", k, 0, 0, 0, 0)]
            k += 1
    s.update(cts=cts, ops=ops, copies=copies, arena=arena)


def run(s):
    ctx, op, case = s["ctx"], s["op"], s["case"]
    if op == "hmult":
        out = ctx.mul_relin_batch(s["a"], s["b"])
        if case["rescale"]:
            out = ctx.rescale_batch(out)
    elif op == "rotate":
        out = ctx.rotate_batch(s["a"], 1 << case["log_step"])
    elif op == "chain":
        out = s["a"]
        for _ in range(case["depth"]):
            out = ctx.rescale_batch(ctx.mul_relin_batch(out, out))
        out = ctx.total_sum_batch(out, 1 << case["log_slots"])
    elif op == "affine":
        out = [ctx.rescale(ctx.add(ctx.mul_plain(a, s["p"]), b)) for a, b in zip(s["a"], s["b"])]
    elif op == "ntt":
        s["fx"].copy_(s["x"])
        ctx.ntt_forward(s["fx"], case["level"])
        s["iy"].copy_(s["y"])
        ctx.ntt_inverse(s["iy"], case["level"])
        return {"forward": s["fx"], "inverse": s["iy"]}
    elif op == "encdec":
        ct = ctx.encrypt_seeded(s["m"], s["level"], s["scale"], s["seed"])
        return {"ct": ct.data, "message": ctx.decrypt(s["answer"]).view(np.int64)}
    elif op == "oplist":
        for dst, src in s["copies"]:
            s["cts"][dst].data.copy_(s["cts"][src].data)
        ctx.exec_batch(s["cts"], s["ops"])
        return s["arena"]
    elif op == "bow":
        out = encrypted_inference(ctx, s["model"], s["docs"], s["words"])
    elif op == "predict":
        out = predict_encrypted(ctx, s["model"], s["docs"], s["words"])
    return [c.data for c in out]


# ---- the least work of a pass: operands read once, results written once,
# keys and weights once; operations: two per modular product

def _switch_products(log_n, level, alpha, K):
    """Modular products of one key switch: the transforms, the base
    conversions and the products with the key."""
    n, beta = 1 << log_n, -(-level // alpha)
    butterflies = n // 2 * log_n
    ext = sum(level + K - min(alpha, level - j * alpha) for j in range(beta))
    transforms = (level + ext + 2 * K + 2 * level) * butterflies
    conversions = n * (sum((level + K) * min(alpha, level - j * alpha) for j in range(beta)) + 2 * K * level)
    return transforms + conversions + 2 * n * beta * (level + K)


def _key_bytes(log_n, level, alpha, K):
    return 8.0 * (1 << log_n) * 2 * -(-level // alpha) * (level + K)


def work(case):
    log_n, L, _, _, K, _, dnum, _ = SETS[case["set"]]
    n, alpha, op = 1 << log_n, -(-L // dnum), case["op"]
    ct = lambda level: 16.0 * level * n  # noqa: E731
    key = lambda level: _key_bytes(log_n, level, alpha, K)  # noqa: E731
    switch = lambda level: 2.0 * _switch_products(log_n, level, alpha, K)  # noqa: E731
    rescale = lambda level: 2.0 * (2 * level * (n // 2 * log_n) + 2 * level * n)  # noqa: E731
    lv, b = case.get("level", 0), case.get("batch", 1)
    if op == "hmult":
        out = lv - 1 if case["rescale"] else lv
        return {"bytes": b * (2 * ct(lv) + ct(out)) + key(lv),
                "flops": b * (switch(lv) + 8.0 * lv * n + (rescale(lv) if case["rescale"] else 0.0))}
    if op == "rotate":
        return {"bytes": b * 2 * ct(lv) + key(lv), "flops": b * switch(lv)}
    if op == "affine":
        return {"bytes": b * (2 * ct(lv) + ct(lv - 1)) + ct(lv) / 2, "flops": b * (rescale(lv) + 4.0 * lv * n)}
    if op == "ntt":
        limbs = 2.0 * case["polys"] * lv
        return {"bytes": 16.0 * limbs * n, "flops": limbs * n * log_n}
    if op == "encdec":  # message and keys in, ciphertext out; ciphertext and secret in, message out
        return {"bytes": 8.0 * n + 2 * ct(lv) + ct(lv) + 1.5 * ct(lv), "flops": 5.0 * lv * n * log_n}
    if op == "chain":
        levels = [lv - d for d in range(case["depth"])]
        end, rots = lv - case["depth"], case["log_slots"]
        return {"bytes": b * (ct(lv) + ct(end)) + sum(key(x) for x in levels) + rots * key(end),
                "flops": b * (sum(switch(x) + 8.0 * x * n + rescale(x) for x in levels) + rots * switch(end))}
    if op == "oplist":  # levels 3..8 in equal shares
        mid = range(3, 9)
        per = sum(2 * ct(x) + ct(x) + 3 * ct(x - 1) for x in mid) / 6 + sum(ct(x) for x in mid) / 6 / 4 * 2
        ops = sum(switch(x) + switch(x - 1) + rescale(x) + 8.0 * x * n for x in mid) / 6
        return {"bytes": case["pairs"] * per + 17 * key(7), "flops": case["pairs"] * ops}
    d, t = case["docs"], n // 2
    if op == "bow":
        total, keys, terms = 0.0, 0.0, 0.0
        for n_o, n_i, n_in, x in ((DIM, t, N_IN, L), (CLASSES, DIM, 1, L - 2)):
            bb, G = bsgs_plan(n_o, n_in)
            steps = rotation_steps(n_o, n_i, n_in)
            rots = len(steps) + (bb - 1) * (n_in - 1)
            total += d * rots * switch(x) + d * 4.0 * n_in * bb * G * x * n
            keys += len(steps) * key(x) + 8.0 * n_in * bb * G * x * n
            terms += d * rescale(x)
        return {"bytes": d * (N_IN * ct(L) + ct(L - 3)) + keys, "flops": total + terms + d * rescale(L - 1)}
    total, keys = 0.0, 0.0
    for n_o, n_i, n_in, x in ((DIM, t, N_IN, PREDICT_LEVEL), (CLASSES, DIM, 1, PREDICT_LEVEL - 2)):
        bb, G = bsgs_plan(n_o, n_in)
        steps = rotation_steps(n_o, n_i, n_in)
        total += d * (len(steps) + (bb - 1) * (n_in - 1) + G) * switch(x) + d * 8.0 * n_in * bb * G * x * n
        keys += (len(steps) + 1) * key(x) + n_in * bb * G * ct(x)
    total += d * (switch(PREDICT_LEVEL - 3) + sum(rescale(x) for x in range(2, PREDICT_LEVEL + 1)))
    return {"bytes": d * (N_IN * ct(PREDICT_LEVEL) + ct(PREDICT_LEVEL - 5)) + keys, "flops": total}


# ---- the same outputs by plain 64-bit integer arithmetic

def _is_prime(m):
    if m % 2 == 0:
        return m == 2
    d, r = m - 1, 0
    while d % 2 == 0:
        d, r = d // 2, r + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if a % m == 0:
            continue
        x = pow(a, d, m)
        if x in (1, m - 1):
            continue
        for _ in range(r - 1):
            x = x * x % m
            if x == m - 1:
                break
        else:
            return False
    return True


def _chain(name):
    """The ciphertext primes: the largest of their bit length that are 1
    modulo 2N, descending."""
    log_n, n_q, q0_bits, q_bits = SETS[name][:4]
    out = []
    for bits, count in ((q0_bits, 1), (q_bits, n_q - 1)):
        c = ((1 << bits) - 2 >> log_n + 1 << log_n + 1) + 1
        while count:
            if c not in out and _is_prime(c):
                out.append(c)
                count -= 1
            c -= 2 << log_n
    return out


def _mod_small(x, b, q):
    """x b mod q for 0 <= x < q < 2^60 and 0 <= b < 2^30 (tensors or numbers):
    the quotient is below 2^30 and comes from doubles, off by at most one."""
    k = (x.double() * (b.double() if torch.is_tensor(b) else float(b)) / float(q)).long()
    r = x * b - k * q  # modulo 2^64, the true value is within 2q
    r = torch.where(r < 0, r + q, r)
    r = torch.where(r < 0, r + q, r)
    return torch.where(r >= q, r - q, r)


def _mul(x, y, q):
    hi, lo = y >> 30, y & (1 << 30) - 1
    s = _mod_small(_mod_small(x, hi, q), 1 << 30, q) + _mod_small(x, lo, q)
    return torch.where(s >= q, s - q, s)


def _powers(root, q, n):
    """root^brv(k) for k < n."""
    bits, out, cur = n.bit_length() - 1, [1], 1
    for j in range(bits):
        f = pow(root, n >> j + 1, q)
        out += [v * f % q for v in out]
    return out


def _transform(x, q, n, inverse, tables):
    """Negacyclic transform of rows x [.., n] modulo q, bit-reversed order:
    entry k is the evaluation at psi^(2 brv(k) + 1)."""
    key = (q, inverse)
    if key not in tables:
        g = 2
        while pow(g, (q - 1) // 2, q) != q - 1:
            g += 1
        psi = pow(g, (q - 1) // (2 * n), q)
        tables[key] = torch.tensor(_powers(pow(psi, -1, q) if inverse else psi, q, n), dtype=torch.int64,
                                   device=x.device)
    tw, shape = tables[key], x.shape
    x = x.reshape(-1, n)
    stages = range(n.bit_length() - 1)
    for s in reversed(stages) if inverse else stages:
        m = 1 << s
        v = x.view(-1, m, 2, n // (2 * m))
        w = tw[m:2 * m].view(1, m, 1)
        a, b = v[:, :, 0], v[:, :, 1]
        if inverse:
            u, d = a + b, a - b
            u = torch.where(u >= q, u - q, u)
            t = _mul(torch.where(d < 0, d + q, d), w.expand_as(d), q)
        else:
            b = _mul(b, w.expand_as(b), q)
            u, t = a + b, a - b
            u, t = torch.where(u >= q, u - q, u), torch.where(t < 0, t + q, t)
        x = torch.stack((u, t), 2).reshape(-1, n)
    if inverse:
        x = _mul(x, torch.full_like(x, pow(n, -1, q)), q)
    return x.reshape(shape)


def exact(case, seed):
    if case["op"] not in ("affine", "ntt"):
        return None  # key switches and draws: outputs are whole numbers, compared as such
    q, n, lv = _chain(case["set"])[:case["level"]], 1 << SETS[case["set"]][0], case["level"]
    gen, tables = _generator(seed), {}
    if case["op"] == "ntt":
        out = {}
        for name in ("forward", "inverse"):
            x = _residues(q, n, case["polys"], gen)
            for i, m in enumerate(q):
                x[:, i] = _transform(x[:, i].contiguous(), m, n, name == "inverse", tables)
            out[name] = x
        return out
    a = [_residues(q, n, 2, gen) for _ in range(case["batch"])]
    b = [_residues(q, n, 2, gen) for _ in range(case["batch"])]
    p = _residues(q, n, 1, gen)[0]
    last, h, out = q[-1], (q[-1] - 1) // 2, []
    for x, y in zip(a, b):
        for i, m in enumerate(q):
            t = _mul(x[:, i], p[i].expand_as(x[:, i]), m) + y[:, i]
            x[:, i] = torch.where(t >= m, t - m, t)
        c = _transform(x[:, lv - 1].contiguous(), last, n, True, tables) + h
        c = torch.where(c >= last, c - last, c) - h  # the centred remainder of the last limb
        r = torch.empty((2, lv - 1, n), dtype=torch.int64, device="cuda")
        for i, m in enumerate(q[:-1]):
            d = x[:, i] - _transform(torch.where(c < 0, c + m, c), m, n, False, tables)
            d = torch.where(d < 0, d + m, d)
            r[:, i] = _mul(d, torch.full_like(d, pow(last, -1, m)), m)
        out.append(r)
    return out
