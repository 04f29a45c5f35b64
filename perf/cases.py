"""Performance cases of the library: the calls a program built on it makes, at the sizes it makes them.

A case is a dict of plain values with a "kind":
  lookup     one table lookup per ciphertext: slz_pbs_batch, then slz_keyswitch_batch_prepared (the step bench.py times)
  ks_first   the same in keyswitch-first order: slz_ks_pbs_batch on ciphertexts under the big key
  keyswitch  slz_keyswitch_batch with the standard key
  lincomb    slz_lwe_lincomb_batch, the leveled sums of the matrix product
  loss       slz_int_ce_loss_deriv, five dependent rounds of lookups on a batch of logits
Keys and ciphertexts are uniform 64-bit words, as TFHE material is; tables are random maps of the message space.  Every
output is an array of 64-bit words that is a function of the input bytes, so the tolerance is "exact".
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2504_17785_amd as slz

# Parameter sets by polynomial size (k = 1): those of the repository's configurations 1, 2 / 4 / 5 and 3, and the shapes in
# between that the fused kernels take (N = 1024 and 4096: 2- and 5-bit messages).
SETS = {
    512: dict(n=128, k=1, N=512, pbs_base_log=8, pbs_level=2, ks_base_log=4, ks_level=3, msg_bits=3),
    1024: dict(n=630, k=1, N=1024, pbs_base_log=23, pbs_level=1, ks_base_log=3, ks_level=5, msg_bits=2),
    2048: dict(n=742, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=3, ks_level=5, msg_bits=4),
    4096: dict(n=800, k=1, N=4096, pbs_base_log=22, pbs_level=1, ks_base_log=3, ks_level=5, msg_bits=5),
    32768: dict(n=1024, k=1, N=32768, pbs_base_log=15, pbs_level=2, ks_base_log=4, ks_level=5, msg_bits=8),
}
# ciphertexts that make a drawn lookup cost no more than the largest listed ones
MAX_BATCH = {512: 16384, 1024: 16384, 2048: 16384, 4096: 4096, 32768: 256}


def listed():
    def lookup(name, N, batch, n_luts, kind="lookup"):
        return dict(name=name, kind=kind, batch=batch, n_luts=n_luts, **SETS[N])

    return [
        # the tiny set with a handful of ciphertexts: launches and the latency of 128 dependent steps
        lookup("lookup_n512_b8", 512, 8, 1),
        # one value looked up alone: the latency of 742 dependent steps
        lookup("lookup_n2048_b1", 2048, 1, 1),
        # an update of a few hundred weights (28 x 8 + 8 x 2, and the biases of a few more units): a ragged, half-full chip
        lookup("lookup_n2048_b301", 2048, 301, 1),
        # one round over a mini-batch's activations
        lookup("lookup_n2048_b1024", 2048, 1024, 3),
        # the largest batch of one GPU, many tables (the headline of bench.py)
        lookup("lookup_n2048_b16384", 2048, 16384, 64),
        # low-precision messages, ciphertexts kept under the big key between lookups, an odd batch
        lookup("ks_first_n1024_b777", 1024, 777, 3, kind="ks_first"),
        # 5-bit messages
        lookup("lookup_n4096_b100", 4096, 100, 4),
        # 8-bit messages, the paper's mini-batch of 8
        lookup("lookup_n32768_b8", 32768, 8, 1),
        # 8-bit messages, a full round
        lookup("lookup_n32768_b256", 32768, 256, 16),
        # the keyswitch alone, with the key as it was generated (the form the gadgets take)
        dict(name="keyswitch_n2048_b1024", kind="keyswitch", batch=1024, **SETS[2048]),
        # leveled sums of a 32 x 784 by 784 x 128 layer modulo one residue
        dict(name="lincomb_g32_784x128", kind="lincomb", groups=32, inputs=784, outputs=128, n=742),
        # the loss gradient of 8 samples with 3 classes
        dict(name="loss_n32768_8x3", kind="loss", samples=8, classes=3, big_gamma=7, kappa=2, **SETS[32768]),
    ]


def _between(rng, lo, hi):
    """An integer of [lo, hi], uniform over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "lookup", "ks_first", "keyswitch", "lincomb", "loss"])
    if kind == "lincomb":
        return dict(kind=kind, groups=_between(rng, 1, 32), inputs=_between(rng, 15, 784), outputs=_between(rng, 8, 128),
                    n=rng.choice([630, 742, 1024]))
    if kind == "loss":
        return dict(kind=kind, samples=_between(rng, 1, 8), classes=rng.randint(2, 3), big_gamma=rng.randint(4, 8), kappa=2, **SETS[32768])
    if kind == "keyswitch":
        N = rng.choice([1024, 2048, 2048, 32768])
        return dict(kind=kind, batch=_between(rng, 1, 256 if N == 32768 else 16384), **SETS[N])
    N = rng.choice([512, 1024, 2048, 2048, 2048, 4096, 32768])
    p = dict(SETS[N])
    p["n"] = rng.randint(p["n"] * 9 // 10, p["n"])
    return dict(kind=kind, batch=_between(rng, 1, MAX_BATCH[N]), n_luts=rng.choice([1, 3, 16, 64]), **p)


# ---- inputs ---------------------------------------------------------------------------------------------------------------
def _params(case):
    return SimpleNamespace(n=case["n"], k=case.get("k", 1), N=case.get("N", 2048), pbs_base_log=case.get("pbs_base_log", 23),
                           pbs_level=case.get("pbs_level", 1), ks_base_log=case.get("ks_base_log", 3),
                           ks_level=case.get("ks_level", 5), msg_bits=case.get("msg_bits", 4))


def _words(gen, *shape):
    return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda", generator=gen)


def _raw(case, seed):
    """Everything that is random: keys in standard form, ciphertexts, tables, indices, weights."""
    p = _params(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    host = np.random.RandomState(seed % (1 << 32))
    r = SimpleNamespace(p=p)
    kind = case["kind"]
    if kind == "lincomb":
        r.cts = _words(gen, case["groups"], case["inputs"], p.n + 1)
        r.w = torch.randint(0, 13, (case["inputs"], case["outputs"]), dtype=torch.int32, device="cuda", generator=gen)
        return r
    r.ksk = _words(gen, p.k * p.N, p.ks_level, p.n + 1)
    if kind == "keyswitch":
        r.cts = _words(gen, case["batch"], p.k * p.N + 1)
        return r
    r.bsk = _words(gen, p.n, p.k + 1, p.pbs_level, p.k + 1, p.N)
    if kind == "loss":
        r.logits = _words(gen, case["samples"], case["classes"], p.n + 1)
        r.labels = _words(gen, case["samples"], case["classes"], p.n + 1)
        r.luts = slz.loss_luts(p, case["classes"], case["big_gamma"], case["kappa"])
        return r
    r.cts = _words(gen, case["batch"], (p.k * p.N if kind == "ks_first" else p.n) + 1)
    r.luts = slz.lut_encode(p, host.randint(0, 1 << p.msg_bits, (case["n_luts"], 1 << p.msg_bits)).astype(np.uint64))
    r.idx = torch.from_numpy(host.randint(0, case["n_luts"], case["batch"]).astype(np.int32)).cuda()
    return r


def prepare(case, seed):
    r = _raw(case, seed)
    s = SimpleNamespace(case=case, p=r.p, kind=case["kind"])
    if s.kind == "lincomb":
        s.ctx = slz.Context(r.p, 1)
        s.cts, s.w = r.cts, r.w
        return s
    s.ctx = slz.Context(r.p, 256 if s.kind == "loss" else case["batch"])
    if s.kind == "keyswitch":
        s.cts, s.ksk = r.cts, r.ksk
        return s
    s.luts = slz.to_device_u64(r.luts)
    s.bskp = s.ctx.bsk_prepare(r.bsk)
    if s.kind == "loss":
        s.logits, s.labels, s.ksk = r.logits, r.labels, r.ksk
        return s
    s.cts, s.idx = r.cts, r.idx
    if s.kind == "ks_first":
        s.ksk = r.ksk
    else:
        s.kskp = s.ctx.ksk_prepare(r.ksk)
    return s


def run(s):
    if s.kind == "lookup":
        big = s.ctx.pbs_batch(s.cts, s.luts, s.idx, s.bskp)
        return big, s.ctx.keyswitch_batch_prepared(big, s.kskp)
    if s.kind == "ks_first":
        return s.ctx.ks_pbs_batch(s.cts, s.ksk, s.luts, s.idx, s.bskp)
    if s.kind == "keyswitch":
        return s.ctx.keyswitch_batch(s.cts, s.ksk)
    if s.kind == "lincomb":
        return s.ctx.lwe_lincomb_batch(s.cts, s.w)
    return s.ctx.int_ce_loss_deriv(s.logits, s.labels, s.case["big_gamma"], s.case["kappa"], s.luts, s.bskp, s.ksk)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------
def work(case):
    """Bytes: keys in standard form, ciphertexts and tables once.  Operations: one double-precision transform of N / 2 complex
    points per polynomial and step and the products between them (the least that any transform method needs, whatever it does
    for exactness), and the multiply-adds of the contractions."""
    p = _params(case)
    small, big = 8 * (p.n + 1), 8 * (p.k * p.N + 1)
    if case["kind"] == "lincomb":
        G, J, O = case["groups"], case["inputs"], case["outputs"]
        return {"bytes": G * (J + O) * small + 4 * J * O, "flops": 2 * G * J * O * (p.n + 1)}
    ksk = p.k * p.N * p.ks_level * small
    ks_flops = 2 * p.k * p.N * p.ks_level * (p.n + 1)
    if case["kind"] == "keyswitch":
        return {"bytes": ksk + case["batch"] * (small + big), "flops": case["batch"] * ks_flops}
    R, C, M = (p.k + 1) * p.pbs_level, p.k + 1, p.N // 2
    bsk = 8 * p.n * R * C * p.N
    pbs_flops = p.n * ((R + C) * 5 * M * math.log2(M) + 8 * R * C * M)
    if case["kind"] == "loss":
        count = case["samples"] * case["classes"]
        return {"bytes": bsk + ksk + 3 * count * small + 5 * 8 * p.N, "flops": 5 * count * (pbs_flops + ks_flops)}
    b = case["batch"]
    return {"bytes": bsk + ksk + b * (small + 2 * big if case["kind"] == "ks_first" else 2 * small + big) + 8 * p.N * case["n_luts"],
            "flops": b * (pbs_flops + ks_flops)}


def tolerance(case):
    return "exact"


# ---- the same results in plain torch --------------------------------------------------------------------------------------
def _limbs(w):
    """int64 words as four signed 16-bit limbs in float64: w = sum_i limb_i 2^(16 i) mod 2^64."""
    out = []
    for _ in range(4):
        low = ((w + (1 << 15)) & 0xFFFF) - (1 << 15)
        out.append(low.double())
        w = (w - low) >> 16
    return out


def _wide(products):
    """sum_i products_i 2^(16 i) mod 2^64 for four exact float64 arrays."""
    total = torch.zeros_like(products[0], dtype=torch.int64)
    for i, x in enumerate(products):
        total += x.to(torch.int64) << (16 * i)
    return total


def _digits(w, beta, level):
    """The signed digits of the gadget decomposition, most significant level first: list of `level` int64 arrays."""
    v = ((w >> (63 - beta * level)) + 1 >> 1) & ((1 << (beta * level)) - 1)      # rounded to the top beta * level bits
    out = []
    for _ in range(level):
        d = v & ((1 << beta) - 1)
        v = v >> beta
        up = d >= (1 << (beta - 1))
        out.append(torch.where(up, d - (1 << beta), d))
        v = v + up
    return out[::-1]


def _modswitch(w, logN2):
    return ((w >> (63 - logN2)) + 1 >> 1) & ((1 << logN2) - 1)


def _rotated(poly, amount):
    """X^amount * poly for polynomials [batch][N] and amounts [batch] in [0, 2N)."""
    N = poly.shape[-1]
    src = (torch.arange(N, device=poly.device)[None, :] - amount[:, None]) % (2 * N)
    v = torch.gather(poly, 1, src % N)
    return torch.where(src >= N, -v, v)


def _exact_keyswitch(p, cts, ksk):
    a, body = cts[:, :-1], cts[:, -1]
    dig = torch.stack(_digits(a, p.ks_base_log, p.ks_level), dim=2).reshape(cts.shape[0], -1).double()
    key = ksk.reshape(-1, p.n + 1)
    out = -_wide([dig @ limb for limb in _limbs(key)])
    out[:, -1] += body
    return out


def _exact_pbs(p, cts, luts, idx, bsk):
    N, logN2 = p.N, p.N.bit_length()
    amounts = _modswitch(cts, logN2)
    acc = [torch.zeros((cts.shape[0], N), dtype=torch.int64, device=cts.device) for _ in range(p.k)]
    acc.append(_rotated(luts[idx.long()], (2 * N - amounts[:, p.n]) % (2 * N)))
    for i in range(p.n):
        rows = []
        for c in range(p.k + 1):
            rows += _digits(_rotated(acc[c], amounts[:, i]) - acc[c], p.pbs_base_log, p.pbs_level)
        rows = [d.flip(1).double() for d in rows]                     # row N - 1 - j of the matrices below
        key = bsk[i].reshape(len(rows), p.k + 1, N)
        for c in range(p.k + 1):
            sums = [0.0] * 4
            for r, d in enumerate(rows):
                for q, limb in enumerate(_limbs(key[r, c])):
                    ext = torch.cat([-limb, limb])                    # negacyclic matrix: entry (j, x) = ext[N + x - j]
                    sums[q] = sums[q] + d @ ext[1:].as_strided((N, N), (1, 1)).contiguous()
            acc[c] = acc[c] + _wide(sums)
    mask = [torch.cat([a[:, :1], -a[:, 1:].flip(1)], dim=1) for a in acc[:-1]]
    return torch.cat(mask + [acc[-1][:, :1]], dim=1)


def exact(case, seed):
    kind, p = case["kind"], _params(case)
    if kind in ("lookup", "ks_first"):
        products = p.n * (p.k + 1) ** 2 * p.pbs_level * 4
        if p.N > 8192 or products * (p.N * p.N * (2.0 * case["batch"] / 3e13 + 3e-11) + 3e-4) > 15.0:
            return None
    elif kind == "loss" or (kind == "keyswitch" and case["batch"] * p.k * p.N > 1 << 26):
        return None
    r = _raw(case, seed)
    if kind == "lincomb":
        w = r.w.double().t().contiguous()
        return torch.stack([_wide([w @ limb for limb in _limbs(g)]) for g in r.cts])
    if kind == "keyswitch":
        return _exact_keyswitch(p, r.cts, r.ksk)
    luts = slz.to_device_u64(r.luts)
    if kind == "ks_first":
        return _exact_pbs(p, _exact_keyswitch(p, r.cts, r.ksk), luts, r.idx, r.bsk)
    big = _exact_pbs(p, r.cts, luts, r.idx, r.bsk)
    return big, _exact_keyswitch(p, big, r.ksk)
