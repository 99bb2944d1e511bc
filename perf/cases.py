"""Performance cases: the work a user of this library has it do.

Each case is one call (or one planned batch of calls) through the public entry
points, with the inputs, keys and contexts a program would already hold on the
GPU.  The cases cover the public and the private operation (encryption with
e = 65537, CRT decryption), exponentiation with shared and per-element
exponents, single products, a batch over keys of mixed sizes and the two
primality steps of key generation, from one message to full batches, with
batch sizes that do and do not divide the kernels' tiles.

Keys come from a pool of fixed primes (the first prime after a SHAKE-256
expansion), a pair picked by the seed; messages, exponents and candidates are
drawn from the seed.
"""
from __future__ import annotations

import hashlib
import math
import random
from functools import lru_cache

import numpy as np
import torch

import paper_1305_3699_amd as rns

E = 65537
SMALL_PRIMES = 10000

# distance from the expansion to the first prime p with p - 1 coprime to E
_OFFSETS = {
    512: (272, 118, 50, 202, 288, 78),
    1024: (250, 78, 250, 560, 634, 34),
    1536: (370, 1394, 2968, 704, 2602, 230),
    2048: (3268, 218, 346, 2270, 442, 1506),
}

# channels per base for moduli up to the given length, and so the number of
# residue products in the two base extensions of one product
_CHANNELS = ((512, 17), (1024, 33), (1536, 49), (2048, 65), (3072, 97), (4096, 129), (8192, 257), (16384, 513))


def listed():
    return [
        # one small public operation: 64 messages, the latency of 19 products
        dict(name="encrypt_1024_64", kind="encrypt", bits=1024, batch=64),
        # signature checks / bulk encryption with the common key size, ragged
        dict(name="encrypt_2048_10007", kind="encrypt", bits=2048, batch=10007),
        # the public operation of a very large modulus (constants beyond LDS)
        dict(name="encrypt_8192_1000", kind="encrypt", bits=8192, batch=1000),
        # a single private operation, as a lone TLS handshake asks for it
        dict(name="decrypt_2048_1", kind="decrypt", bits=2048, batch=1),
        # the headline workload: a full batch of private operations
        dict(name="decrypt_2048_16384", kind="decrypt", bits=2048, batch=16384),
        # private operations with the largest common key
        dict(name="decrypt_4096_4096", kind="decrypt", bits=4096, batch=4096),
        # a long exponent shared by 1,024 bases
        dict(name="modexp_2048_e8192_1024", kind="modexp", bits=2048, exp_bits=8192, batch=1024, per_element=False),
        # every base with an exponent of its own, odd modulus length and batch
        dict(name="modexp_1000_each_3001", kind="modexp", bits=1000, exp_bits=1000, batch=3001, per_element=True),
        # independent products of residue vectors
        dict(name="montmul_3072_65536", kind="montmul", bits=3072, batch=65536),
        # operations on 16 keys of four sizes planned as one batch
        dict(name="mixed_16keys", kind="mixed", keys=16, median=128),
        # candidates of a prime search sieved by the first 10,000 primes
        dict(name="trial_1024_20000", kind="trial", bits=1024, batch=20000),
        # the survivors' strong tests
        dict(name="rabin_1024_500", kind="rabin", bits=1024, batch=500, rounds=5),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["encrypt", "decrypt", "decrypt", "modexp", "modexp", "montmul", "mixed", "trial", "rabin"])
    if kind == "encrypt":
        bits = rng.choice([1024, 1536, 2048, 3072, 4096, 8192])
        return dict(kind=kind, bits=bits, batch=_log_uniform(rng, 1, 40000 if bits < 8192 else 4000))
    if kind == "decrypt":
        bits = rng.choice([1024, 2048, 2048, 3072, 4096])
        return dict(kind=kind, bits=bits, batch=_log_uniform(rng, 1, {1024: 30000, 2048: 16384, 3072: 8000, 4096: 4096}[bits]))
    if kind == "modexp":
        bits = _log_uniform(rng, 128, 3072)
        per_element = rng.random() < 0.5
        exp_bits = _log_uniform(rng, 2, bits if per_element else 2 * bits)
        return dict(kind=kind, bits=bits, exp_bits=exp_bits, batch=_log_uniform(rng, 1, 3000), per_element=per_element)
    if kind == "montmul":
        return dict(kind=kind, bits=rng.choice([512, 1024, 2048, 3072, 4096]), batch=_log_uniform(rng, 1, 65536))
    if kind == "mixed":
        return dict(kind=kind, keys=rng.randint(2, 16), median=_log_uniform(rng, 4, 128))
    if kind == "trial":
        bits = 32 * rng.randint(8, 64)
        return dict(kind=kind, bits=bits, batch=_log_uniform(rng, 64, 20000 * 32 * 32 // bits))
    bits = rng.choice([512, 1024, 1024, 1536])
    return dict(kind="rabin", bits=bits, batch=_log_uniform(rng, 32, 1000 if bits <= 1024 else 300),
                rounds=rng.randint(1, 8))


# ---- inputs ---------------------------------------------------------------

@lru_cache(maxsize=None)
def _prime(bits, i):
    x = int.from_bytes(hashlib.shake_256(b"rsa prime %d %d" % (bits, i)).digest(bits // 8), "big")
    return (x | (3 << (bits - 2)) | 1) + _OFFSETS[bits][i]


def _key(bits, rng):
    """(n, d, p, q) of an RSA key: two primes of the pool."""
    i, j = rng.sample(range(len(_OFFSETS[bits // 2])), 2)
    p, q = _prime(bits // 2, i), _prime(bits // 2, j)
    return p * q, pow(E, -1, (p - 1) * (q - 1)), p, q


def _odd(bits, rng):
    return rng.getrandbits(bits) | (1 << (bits - 1)) | 1


def _limbs(x, n):
    return np.frombuffer(int(x).to_bytes(4 * n, "little"), dtype="<u4").copy()


def _ints(rows):
    w = 4 * rows.shape[1]
    raw = np.ascontiguousarray(rows, dtype="<u4").tobytes()
    return [int.from_bytes(raw[i:i + w], "little") for i in range(0, len(raw), w)]


def _rows(values, n):
    raw = b"".join(int(v).to_bytes(4 * n, "little") for v in values)
    return np.frombuffer(raw, dtype="<i4").reshape(len(values), n).copy()


def _below(n, batch, limbs, gen):
    """Rows of values below n (uniform words; the top one below n's)."""
    x = gen.integers(0, 1 << 32, size=(batch, limbs), dtype=np.uint32)
    top = (n.bit_length() - 1) // 32
    x[:, top + 1:] = 0
    x[:, top] = gen.integers(0, n >> (32 * top), size=batch, dtype=np.uint32)
    return x


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()


def _words(bits):
    return (bits + 31) // 32


def _draws(case, seed):
    """The numbers of a case, before they go to the GPU."""
    rng, gen = random.Random(seed), np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "encrypt":
        n = _odd(case["bits"], rng)
        return dict(n=n, x=_below(n, case["batch"], _words(case["bits"]), gen))
    if kind == "decrypt":
        n, d, p, q = _key(case["bits"], rng)
        return dict(n=n, d=d, p=p, q=q, x=_below(n, case["batch"], _words(case["bits"]), gen))
    if kind == "modexp":
        n, ew = _odd(case["bits"], rng), _words(case["exp_bits"])
        e = gen.integers(0, 1 << 32, size=(case["batch"] if case["per_element"] else 1, ew), dtype=np.uint32)
        top = (case["exp_bits"] - 1) % 32
        e[:, -1] &= np.uint32((1 << (top + 1)) - 1)
        e[:, -1] |= np.uint32(1 << top)
        return dict(n=n, e=e, x=_below(n, case["batch"], _words(case["bits"]), gen))
    if kind == "montmul":
        n, L = _odd(case["bits"], rng), _words(case["bits"])
        return dict(n=n, x=_below(n, case["batch"], L, gen), y=_below(n, case["batch"], L, gen))
    if kind == "mixed":
        # the trace (messages per key and kind) belongs to the case
        ops, trace = [], random.Random(case["keys"] * 10007 + case["median"])
        for j in range(case["keys"]):
            bits = (1024, 2048, 3072, 4096)[j % 4]
            key = _key(bits, rng)
            count = min(1024, max(1, round(case["median"] * math.exp(trace.gauss(0.0, 0.5)))))
            dec = sum(trace.random() < 0.5 for _ in range(count))
            parts = [(what, _below(key[0], c, bits // 32, gen)) for what, c in (("encrypt", count - dec), ("decrypt", dec)) if c]
            ops.append((bits, key, parts))
        return dict(ops=ops)
    L = _words(case["bits"])
    cand = gen.integers(0, 1 << 32, size=(case["batch"], L), dtype=np.uint32)
    cand[:, 0] |= 1
    cand[:, -1] |= np.uint32(3 << 30)
    if kind == "trial":
        return dict(cand=cand)
    # about every 8th candidate a prime of the pool, as among a sieve's survivors
    for i in range(case["batch"]):
        if rng.random() < 0.125:
            cand[i] = _limbs(_prime(case["bits"], rng.randrange(6)), L)
    bases = gen.integers(0, 1 << 32, size=(case["batch"], case["rounds"], L), dtype=np.uint32)
    bases[:, :, -1] &= np.uint32(0x7FFFFFFF)
    bases[:, :, 0] |= 2
    return dict(cand=cand, bases=bases)


def _load(key):
    n, d, p, q = key
    return rns.RsaKey(n, E, d, p, q, d % (p - 1), d % (q - 1), pow(q, -1, p))


def _residues(x, moduli):
    """[len(moduli) + 1, batch] residues of the rows of x, 2^32 last."""
    limbs = torch.from_numpy(x.astype(np.int64)).cuda()
    m = torch.tensor(moduli, dtype=torch.int64, device="cuda")[:, None]
    r = torch.zeros((len(moduli), x.shape[0]), dtype=torch.int64, device="cuda")
    for col in reversed(range(x.shape[1])):
        for half in (limbs[:, col] >> 16, limbs[:, col] & 0xFFFF):
            r = ((r << 16) + half) % m
    r = torch.cat([r, limbs[:, 0][None]])
    return torch.where(r >= 1 << 31, r - (1 << 32), r).to(torch.int32).contiguous()


def prepare(case, seed):
    v = _draws(case, seed)
    kind = case["kind"]
    if kind == "encrypt":
        return dict(kind=kind, key=rns.RsaKey(v["n"], E), x=_gpu(v["x"]))
    if kind == "decrypt":
        return dict(kind=kind, key=_load((v["n"], v["d"], v["p"], v["q"])), x=_gpu(v["x"]))
    if kind == "modexp":
        e = _gpu(v["e"])
        return dict(kind=kind, ctx=rns.RnsContext(v["n"]), x=_gpu(v["x"]), e=e if case["per_element"] else e[0])
    if kind == "montmul":
        ctx = rns.RnsContext(v["n"])
        return dict(kind=kind, ctx=ctx, x=_residues(v["x"], ctx.primes), y=_residues(v["y"], ctx.primes))
    if kind == "mixed":
        ops = []
        for _, key, parts in v["ops"]:
            handle = _load(key)
            for what, rows in parts:
                x = _gpu(rows)
                ops.append((handle, rns.OP_ENCRYPT if what == "encrypt" else rns.OP_DECRYPT, x, torch.zeros_like(x)))
        return dict(kind=kind, batch=rns.RsaBatch(ops), outs=[op[3] for op in ops])
    if kind == "trial":
        return dict(kind=kind, cand=_gpu(v["cand"]))
    return dict(kind=kind, cand=v["cand"], bases=v["bases"])


# ---- one pass -------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "encrypt":
        return state["key"].encrypt(state["x"])
    if kind == "decrypt":
        return state["key"].decrypt(state["x"])
    if kind == "modexp":
        return state["ctx"].modexp(state["x"], state["e"])
    if kind == "montmul":
        return state["ctx"].mont_mul(state["x"], state["y"])
    if kind == "mixed":
        state["batch"].run()
        return state["outs"]
    if kind == "trial":
        return rns.trial_division(state["cand"], SMALL_PRIMES)
    return rns.miller_rabin(state["cand"], state["bases"])


# ---- what a pass cannot do without ----------------------------------------

def _product_flops(bits):
    """The two base extensions of one product: k (k + 1) products of 32-bit
    residues each, 16 byte products and sums per residue product."""
    k = next(k for top, k in _CHANNELS if bits <= top)
    return 2 * 16 * 2 * k * (k + 1)


def _modexp_flops(bits, exp_bits, batch):
    # the squarings, and a multiplication for every sixth bit of a long exponent
    return batch * _product_flops(bits) * (exp_bits + (exp_bits / 6 if exp_bits > 32 else 1) + 1)


def work(case):
    kind = case["kind"]
    if kind == "mixed":
        flops = bytes_ = 0.0
        for j in range(case["keys"]):
            bits, ops = (1024, 2048, 3072, 4096)[j % 4], case["median"] * math.exp(0.125) / 2
            flops += _modexp_flops(bits, 17, ops) + 2 * _modexp_flops(bits // 2, bits // 2, ops)
            bytes_ += 2 * ops * 2 * bits / 8
        return {"bytes": bytes_, "flops": flops}
    bits, batch = case["bits"], case["batch"]
    row = 4 * _words(bits)
    if kind == "encrypt":
        return {"bytes": 2 * batch * row, "flops": _modexp_flops(bits, 17, batch)}
    if kind == "decrypt":
        return {"bytes": 2 * batch * row, "flops": 2 * _modexp_flops(bits // 2, bits // 2, batch)}
    if kind == "modexp":
        exps = (batch if case["per_element"] else 1) * 4 * _words(case["exp_bits"])
        return {"bytes": 2 * batch * row + exps, "flops": _modexp_flops(bits, case["exp_bits"], batch)}
    if kind == "montmul":
        k = next(k for top, k in _CHANNELS if bits <= top)
        return {"bytes": 3 * 4 * (2 * k + 1) * batch, "flops": batch * _product_flops(bits)}
    if kind == "trial":
        # one multiplication and addition per candidate limb and small prime
        return {"bytes": batch * (row + 1), "flops": 2 * batch * _words(bits) * SMALL_PRIMES}
    return {"bytes": batch * (row + case["rounds"] * row + 1),
            "flops": _modexp_flops(bits, bits, batch * case["rounds"])}


# ---- the definition, on the host ------------------------------------------

def _pow_seconds(bits, exp_bits):
    """About what one pow() takes on the host."""
    return exp_bits * 1.2 * (0.3e-6 + (bits / 2048) ** 2 * 7e-6)


def _crt(c, d, p, q):
    mp, mq = pow(c, d % (p - 1), p), pow(c, d % (q - 1), q)
    return mq + q * ((mp - mq) * pow(q, -1, p) % p)


def _strong(n, a):
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    x = pow(a, d, n)
    if x in (1, n - 1):
        return True
    for _ in range(s - 1):
        x = x * x % n
        if x == n - 1:
            return True
    return False


@lru_cache(maxsize=None)
def _first_primes():
    bound = 104730
    sieve = bytearray([1]) * bound
    sieve[:2] = b"\0\0"
    for i in range(2, int(bound ** 0.5) + 1):
        if sieve[i]:
            sieve[i * i::i] = bytearray(len(sieve[i * i::i]))
    return [i for i in range(bound) if sieve[i]][:SMALL_PRIMES]


def exact(case, seed):
    kind = case["kind"]
    limit = 20.0
    if kind == "montmul":
        return None   # the residues of the result depend on the bases the context drew
    if kind == "encrypt" and case["batch"] * _pow_seconds(case["bits"], 17) > limit:
        return None
    if kind == "decrypt" and case["batch"] * 2 * _pow_seconds(case["bits"] // 2, case["bits"] // 2) > limit:
        return None
    if kind == "modexp" and case["batch"] * _pow_seconds(case["bits"], case["exp_bits"]) > limit:
        return None
    if kind == "rabin" and case["batch"] * (1 + case["rounds"] / 8) * _pow_seconds(case["bits"], case["bits"]) > limit:
        return None
    if kind == "mixed" and case["keys"] * case["median"] > 1000:
        return None
    if kind == "trial" and case["batch"] > 40000:
        return None
    v = _draws(case, seed)
    if kind == "encrypt":
        return _rows([pow(m, E, v["n"]) for m in _ints(v["x"])], v["x"].shape[1])
    if kind == "decrypt":
        return _rows([_crt(c, v["d"], v["p"], v["q"]) for c in _ints(v["x"])], v["x"].shape[1])
    if kind == "modexp":
        exps = _ints(v["e"])
        rows = [pow(b, exps[i if case["per_element"] else 0], v["n"]) for i, b in enumerate(_ints(v["x"]))]
        return _rows(rows, v["x"].shape[1])
    if kind == "mixed":
        outs = []
        for bits, (n, d, p, q), parts in v["ops"]:
            for what, rows in parts:
                vals = [pow(x, E, n) if what == "encrypt" else _crt(x, d, p, q) for x in _ints(rows)]
                outs.append(_rows(vals, bits // 32))
        return outs
    if kind == "trial":
        product = math.prod(_first_primes())
        return np.array([math.gcd(product % n, n) == 1 for n in _ints(v["cand"])], dtype=np.uint8)
    flags = []
    for n, row in zip(_ints(v["cand"]), v["bases"]):
        flags.append(all(_strong(n, a) for a in _ints(row)))
    return np.array(flags, dtype=np.uint8)
