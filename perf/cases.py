"""The calls whose time matters to a program that uses this library, each through the binding's own functions.

A server evaluates projections (ckks_ctpt_matmul), rotation banks, ciphertext products and rescales; a model is
loaded by encoding its diagonals and expanding them to residues; the key holder encodes and decodes.  The rings are
the two of the repository's own workloads (N = 2^16 with 24 + 8 primes, the toy ring at 2^12) and the ones between
them, with as many 50-bit and 60-bit primes as 128-bit security leaves a ring of that degree (log2 PQ of about 218,
438 and 881 at 2^13, 2^14 and 2^15), three digits each.

Keys and ciphertexts are uniform residues: that is what valid ones look like to the server, and no kernel's work
depends on the message.  Weights, slots and coefficients have the distributions of the model and of its encoding.
"""
import functools

import numpy as np
import torch

from paper_2604_09975_amd import binding as B
from paper_2604_09975_amd import plan

DNUM = 3
# log2 N -> bit sizes of the ciphertext and special primes, log2 of the encoding scale
CHAINS = {
    12: ((40, 30, 30), (40,), 30),
    13: ((50,) * 3, (60,), 40),
    14: ((50,) * 6, (60,) * 2, 40),
    15: ((50,) * 12, (60,) * 4, 40),
    16: ((50,) * 24, (60,) * 8, 40),
}


@functools.lru_cache(maxsize=None)
def ring(logN):
    """The parameter set a program creates once when it starts."""
    q_bits, p_bits, _ = CHAINS[logN]
    hits = {b: B.ckks_find_primes(b, logN, (q_bits + p_bits).count(b)) for b in set(q_bits + p_bits)}
    p = [hits[b].pop(0) for b in p_bits]
    q = [hits[b].pop(0) for b in q_bits]
    return B.ckks_params_create(logN, q, p, DNUM)


def listed():
    return [
        # BERT-base QKV projection, the headline workload: real packing, merged giant step, rescale in the call
        {"name": "proj_qkv_16", "kind": "proj", "logN": 16, "level": 24, "m": 128, "C": 256, "d_in": 768,
         "d_out": 2304, "N1": 32, "packing": "real", "merged": True},
        # a layer of a smaller model with complex-pair compression, ragged widths, below the top level
        {"name": "proj_pair_15", "kind": "proj", "logN": 15, "level": 11, "m": 128, "C": 128, "d_in": 700,
         "d_out": 384, "N1": 16, "packing": "pair", "merged": True},
        # the toy projection of the tests: a short call that launches dominate; every giant rotation a complete switch
        {"name": "proj_toy_12", "kind": "proj", "logN": 12, "level": 3, "m": 16, "C": 64, "d_in": 64, "d_out": 64,
         "N1": 8, "packing": "real", "merged": False},
        # the bank of 27 rotations of one ciphertext
        {"name": "bank_27_16", "kind": "rotate", "logN": 16, "level": 24, "steps": 27},
        # one rotation in the middle of a circuit (level 17: digits of 8, 8 and 1 limbs): latency of a lone switch
        {"name": "rot_1_16", "kind": "rotate", "logN": 16, "level": 17, "steps": 1},
        # intra-segment shifts of the attention kernels on a small ring
        {"name": "shift_bank_14", "kind": "shift", "logN": 14, "level": 5, "count": 12, "m": 64},
        # ciphertext product, relinearised and rescaled
        {"name": "ctmul_rescale_15", "kind": "ctmul", "logN": 15, "level": 12},
        # the transform benchmark of the repository, forward
        {"name": "ntt_64x24_16", "kind": "ntt", "logN": 16, "limbs": 24, "batch": 64, "inverse": False},
        # a few polynomials of a small ring, inverse (special limb included)
        {"name": "intt_3x4_13", "kind": "ntt", "logN": 13, "limbs": 4, "batch": 3, "inverse": True},
        # the diagonals of one (output block, giant step) pair of the QKV layer, encoded when a model is loaded
        {"name": "encode_96_16", "kind": "encode", "logN": 16, "count": 96, "real": True},
        # a batch of decrypted results
        {"name": "decode_5_15", "kind": "decode", "logN": 15, "count": 5},
        # masks and weights expanded to evaluation form
        {"name": "expand_32_15", "kind": "expand", "logN": 15, "level": 9, "count": 32},
    ]


def _log_spread(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["proj", "proj", "rotate", "rotate", "shift", "ctmul", "ntt", "ntt", "encode", "decode", "expand"])
    logN = rng.choice(sorted(CHAINS))
    L, n = len(CHAINS[logN][0]), 1 << (logN - 1)
    c = {"kind": kind, "logN": logN}
    if kind == "proj":
        c["level"] = rng.randint(max(2, L // 2), L)
        c["m"] = rng.choice([16, 32, 64, 128])
        c["C"] = min(256, n // c["m"]) >> rng.randint(0, 1)
        c["d_in"] = rng.randint(1, 3 * c["C"])
        c["d_out"] = rng.randint(1, 4 * c["C"])
        c["packing"] = rng.choice(["real", "real", "pair"])
        G, B_out = _groups(c)
        c["N1"] = plan.choose_n1(G, B_out, c["C"])
        c["merged"] = rng.random() < 0.7
    elif kind == "rotate":
        c["level"], c["steps"] = rng.randint(1, L), _log_spread(rng, 1, 40)
    elif kind == "shift":
        c["level"], c["count"], c["m"] = rng.randint(2, L), _log_spread(rng, 1, 24), rng.choice([16, 32, 64, 128])
    elif kind == "ctmul":
        c["level"] = rng.randint(2, L)
    elif kind == "ntt":
        c["limbs"], c["batch"] = rng.randint(1, L), _log_spread(rng, 1, 64)
        c["inverse"] = rng.random() < 0.5
    elif kind == "encode":
        c["count"], c["real"] = _log_spread(rng, 1, 130), rng.random() < 0.6
    elif kind == "decode":
        c["count"] = _log_spread(rng, 1, 70)
    else:
        c["level"], c["count"] = rng.randint(1, L), _log_spread(rng, 1, 64)
    return c


def _groups(case):
    """Input ciphertexts and output blocks of a projection."""
    G = -(-case["d_in"] // case["C"])
    return (G + 1) // 2 if case["packing"] == "pair" else G, -(-case["d_out"] // case["C"])


def _uniform(g, moduli, lead, N):
    q = torch.tensor(moduli, dtype=torch.int64, device="cuda").view(-1, 1)
    return torch.randint(0, 1 << 62, tuple(lead) + (len(moduli), N), dtype=torch.int64, device="cuda", generator=g) % q


def _keys(P, g, steps):
    """Galois keys of the steps that are no full turn, handed to the library without a copy."""
    elts = [B.ckks_galois_elt(P, s) for s in steps]
    return [B.ckks_galois_key_adopt(P, e, _uniform(g, P.q + P.p, (P.dnum, 2), P.N)) if e != 1 else None for e in elts]


def _relin_key(P, g):
    return B.ckks_relin_key_load(P, _uniform(g, P.q + P.p, (P.dnum, 2), P.N))


def _diagonals(Wm, c, nseg, b, p):
    """Slot values, one per segment, of the plaintexts of output block b and giant step p: [G][N1][nseg]."""
    C, N1 = c["C"], c["N1"]
    seg = torch.arange(nseg, device="cuda") % C
    col = b * C + (seg - p * N1) % C
    row = torch.arange(Wm.shape[0] // C, device="cuda").view(-1, 1, 1) * C + (seg + torch.arange(N1, device="cuda").view(-1, 1)) % C
    return Wm[row, col]


def _steps(count, n, seed):
    """The first steps of a rotation bank: 1, 2, ..., powers of two and the conjugation among them."""
    r = np.random.default_rng(seed)
    first = list(range(1, 17)) + [s for s in (1 << k for k in range(5, 16)) if s < n] + ["conj"]
    if count == 1:
        return [int(r.integers(1, n))]
    more = [int(s) for s in r.integers(1, n, max(0, count - len(first)))]
    return (first[-1:] + first[:-1] + more)[:count]


def _projection(case, P, g):
    N, n, level, C, N1, m = P.N, P.N // 2, case["level"], case["C"], case["N1"], case["m"]
    (G, B_out), N2, scale = _groups(case), case["C"] // case["N1"], 2.0 ** CHAINS[case["logN"]][2]
    pair = case["packing"] == "pair"
    Gr = 2 * G if pair else G
    Wm = torch.zeros((Gr * C, B_out * C), dtype=torch.float64, device="cuda")
    Wm[:case["d_in"], :case["d_out"]] = 0.02 * torch.randn((case["d_in"], case["d_out"]), dtype=torch.float64, device="cuda", generator=g)
    w = B.ckks_weights_create(P, level, m, C, G, B_out, N1)
    for b in range(B_out):
        for p in range(N2):
            z = _diagonals(Wm, case, n // m, b, p).to(torch.complex128)
            if pair:
                z = 0.5 * (z[0::2] - 1j * z[1::2])
            slots = z.repeat_interleave(m, dim=-1).reshape(-1, n).contiguous()
            B.ckks_weights_set_diagonals(w, (b * N2 + p) * G * N1, B.ckks_encode(P, slots, scale, 0 if pair else B.ENCODE_REAL))
    bias = (0.02 * torch.randn((B_out, n // m, 1), dtype=torch.float64, device="cuda", generator=g)).expand(-1, -1, m)
    B.ckks_weights_set_bias(w, B.ckks_encode(P, bias.reshape(B_out, n).to(torch.complex128).contiguous(), scale, B.ENCODE_REAL), int(scale))
    return {"w": w, "x": _uniform(g, P.q[:level], (G, 2), N), "baby": _keys(P, g, [q * m for q in range(1, N1)]),
            "giant": _keys(P, g, [p * N1 * m for p in range(1, N2)]), "conj": _keys(P, g, ["conj"])[0] if pair else None,
            "B_out": B_out}


def prepare(case, seed):
    P = ring(case["logN"])
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    N, n, kind = P.N, P.N // 2, case["kind"]
    scale = 2.0 ** CHAINS[case["logN"]][2]
    s = {"case": case, "P": P}
    if kind == "proj":
        s.update(_projection(case, P, g))
    elif kind == "rotate":
        s["steps"] = _steps(case["steps"], n, seed)
        s["x"], s["keys"] = _uniform(g, P.q[:case["level"]], (2,), N), _keys(P, g, s["steps"])
    elif kind == "shift":
        level, m = case["level"], case["m"]
        ts = [1 + t % (m - 1) for t in range(case["count"])]
        s["steps"] = [x for t in ts for x in (t, (t - m) % n)]
        r = torch.arange(n, device="cuda") % m
        masks = torch.stack([v for t in ts for v in (r < m - t, r >= m - t)]).to(torch.complex128)
        s["masks"] = B.ckks_plain_expand(P, level, B.ckks_encode(P, masks, scale, B.ENCODE_REAL))
        s["x"], s["keys"] = _uniform(g, P.q[:level], (2,), N), _keys(P, g, s["steps"])
    elif kind == "ctmul":
        q = P.q[:case["level"]]
        s["a"], s["b"], s["key"] = _uniform(g, q, (2,), N), _uniform(g, q, (2,), N), _relin_key(P, g)
    elif kind == "ntt":
        # an inverse transform that is not of the ciphertext primes alone: the special limb last
        s["ids"] = list(range(case["limbs"])) if not case["inverse"] else list(range(case["limbs"] - 1)) + [P.L]
        s["x"] = _uniform(g, [(P.q + P.p)[i] for i in s["ids"]], (case["batch"],), N)
    elif kind == "encode":
        s["z"], s["scale"] = _slots(case, seed, n), scale
    elif kind == "decode":
        # two-limb residues of a product at twice the scale after one rescale: coefficients of a few times 2^30
        c = (2.0 ** 32 * torch.randn((case["count"], 1, N), dtype=torch.float64, device="cuda", generator=g)).to(torch.int64)
        s["r"], s["scale"] = c % torch.tensor(P.q[:2], dtype=torch.int64, device="cuda").view(1, 2, 1), scale
    else:
        s["c"] = B.ckks_encode(P, _slots({"count": case["count"], "real": True}, seed, n), scale, B.ENCODE_REAL)
    return s


def _slots(case, seed, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    re = 0.02 * torch.randn((case["count"], n), dtype=torch.float64, device="cuda", generator=g)
    im = torch.zeros_like(re) if case["real"] else 0.02 * torch.randn((case["count"], n), dtype=torch.float64, device="cuda", generator=g)
    return torch.complex(re, im)


def run(s):
    case, P = s["case"], s["P"]
    kind = case["kind"]
    if kind == "proj":
        if case["merged"]:
            return B.ckks_ctpt_matmul(P, s["w"], s["x"], s["baby"], s["giant"], conj_key=s["conj"],
                                      flags=B.MATMUL_MERGED_GIANT | B.MATMUL_RESCALE)[0]
        y, _ = B.ckks_ctpt_matmul(P, s["w"], s["x"], s["baby"], s["giant"], conj_key=s["conj"])
        return B.ckks_rescale(P, y, case["level"], s["B_out"])
    if kind == "rotate":
        return B.ckks_rotate_hoisted(P, s["x"], case["level"], s["steps"], s["keys"])
    if kind == "shift":
        y = B.ckks_shift_bank(P, s["x"], case["level"], s["steps"], s["keys"], s["masks"])
        return B.ckks_rescale(P, y, case["level"], case["count"])
    if kind == "ctmul":
        return B.ckks_rescale(P, B.ckks_ctmul(P, s["a"], s["b"], case["level"], s["key"]), case["level"], 1)
    if kind == "ntt":
        return (B.ckks_intt if case["inverse"] else B.ckks_ntt)(P, s["x"], s["ids"], case["batch"])
    if kind == "encode":
        return B.ckks_encode(P, s["z"], s["scale"], B.ENCODE_REAL if case["real"] else 0)
    if kind == "decode":
        return B.ckks_decode(P, s["r"], 2, s["scale"])
    return B.ckks_plain_expand(P, case["level"], s["c"])


def _switch_work(N, logN, level, L, K, switches, sources):
    """Modular operations of `switches` key switches whose digits come from `sources` decompositions."""
    alpha = L // DNUM
    beta, W = -(-level // alpha), level + K
    fly = 1.5 * logN * N                        # N/2 butterflies a stage: one product, two sums
    up = level * fly + beta * (W - min(alpha, level)) * (fly + 2 * alpha * N)
    down = 2 * (2 * beta * W * N + (K + level) * fly + 2 * K * level * N + 2 * level * N)
    return sources * up + switches * down


def work(case):
    q_bits, p_bits, _ = CHAINS[case["logN"]]
    logN, N, L, K = case["logN"], 1 << case["logN"], len(q_bits), len(p_bits)
    kind, level = case["kind"], case.get("level", 0)
    alpha = L // DNUM
    key = -(-level // alpha) * 2 * (level + K) * N * 8
    limb, fly = N * 8, 1.5 * logN * N
    if kind == "proj":
        (G, B_out), N1, N2 = _groups(case), case["N1"], case["C"] // case["N1"]
        diag = G * N1 * B_out * N2
        pair = case["packing"] == "pair"
        turns = G * (N1 - 1) + B_out * (N2 - 1) + (B_out if pair else 0)
        # residues of a weight limb are log2 q bits each; those of a real diagonal are a palindrome
        wbytes = diag * sum(q_bits[:level]) / 8 * N / (1 if pair else 2)
        flops = diag * level * N * 4 + _switch_work(N, logN, level, L, K, turns, G + turns - G * (N1 - 1))
        return {"bytes": wbytes + (N1 - 1 + N2 - 1 + pair) * key + G * 2 * level * limb + B_out * (2 * level - 1) * limb + B_out * level * limb,
                "flops": flops + B_out * 2 * level * fly}
    if kind == "rotate":
        c = case["steps"]
        return {"bytes": c * key + (1 + c) * 2 * level * limb, "flops": _switch_work(N, logN, level, L, K, c, 1)}
    if kind == "shift":
        c = case["count"]
        return {"bytes": 2 * c * key + 2 * level * limb + c * 2 * level * limb + c * 2 * (level - 1) * limb,
                "flops": _switch_work(N, logN, level, L, K, 2 * c, 1) + c * level * (8 * N + 2 * fly)}
    if kind == "ctmul":
        return {"bytes": key + 4 * level * limb + 2 * (level - 1) * limb,
                "flops": _switch_work(N, logN, level, L, K, 1, 1) + level * (8 * N + 2 * fly)}
    if kind == "ntt":
        rows = case["batch"] * case["limbs"]
        return {"bytes": 2 * rows * limb, "flops": rows * fly}
    fft = 5.0 * N * logN
    if kind == "encode":
        return {"bytes": case["count"] * 2 * limb, "flops": case["count"] * fft}
    if kind == "decode":
        return {"bytes": case["count"] * 3 * limb, "flops": case["count"] * fft}
    return {"bytes": case["count"] * (level + 1) * limb, "flops": case["count"] * level * fly}


def tolerance(case):
    if case["kind"] == "encode":
        return {"rel": 1e-9, "differ": 4e-5}     # a coefficient next to a tie, and its mirror, of one short vector
    if case["kind"] == "decode":
        return {"rel": 2e-15, "max": 2e-14}      # one fp64 transform of 2^12 .. 2^16 points: 4e-16 measured
    return "exact"                               # residues


@functools.lru_cache(maxsize=None)
def _bins(n):
    e, out = 1, np.empty(n, dtype=np.int64)
    for j in range(n):
        out[j] = (e - 1) >> 1
        e = e * 5 % (4 * n)
    return out


def exact(case, seed):
    """encode and decode by numpy's transform in 64 bits; the residues of the other cases are whole numbers, compared
    as they are."""
    N = 1 << case["logN"]
    n, scale = N // 2, 2.0 ** CHAINS[case["logN"]][2]
    zeta = np.exp(1j * np.pi * np.arange(N) / N)
    if case["kind"] == "encode":
        z = _slots(case, seed, n).cpu().numpy()
        v = np.zeros((case["count"], N), dtype=np.complex128)
        v[:, _bins(n)] = z
        v[:, N - 1 - _bins(n)] = z.conj()
        return np.rint(scale / N * (np.fft.fft(v, axis=1) * zeta.conj()).real).astype(np.int64)
    if case["kind"] == "decode":
        P = ring(case["logN"])
        r = prepare(case, seed)["r"][:, 0].cpu().numpy()
        c = np.where(r > P.q[0] // 2, r - P.q[0], r).astype(np.float64)
        return np.fft.ifft(c * zeta, axis=1)[:, _bins(n)] * (N / scale)
    return None
