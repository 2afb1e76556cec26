"""Performance cases of the library: the calls a program makes, over the sizes it makes them at.

listed() names the cases, draw(rng) makes another one of the same ranges, prepare() sets up
what a program holds before the call, run() is one pass through the public entry points,
work() is what a pass cannot do without, and exact() is the same result in plain torch and
numpy (float64 FFTs of 11-bit pieces, whole numbers throughout).

A case is {"op", "n", "channels", "batch", "modulus"}; plans give their groups as text.
"""
import numpy as np
import torch

import paper_2307_06554_amd as pm

GOLDILOCKS = (1 << 64) - (1 << 32) + 1


def listed():
    return [
        # the lattice-signature size in one call: latency and launch count (small modulus, two limbs)
        {"name": "n256_q3329_b1024", "op": "negacyclic", "n": 256, "channels": 1, "batch": 1024, "modulus": "3329"},
        # one ciphertext times one ciphertext: the smallest useful RNS call
        {"name": "n4096_rns8_b1", "op": "rns", "n": 4096, "channels": 8, "batch": 1, "modulus": "ntt30"},
        # many small products under one prime, a ragged batch
        {"name": "n1024_q30_b4095", "op": "negacyclic", "n": 1024, "channels": 1, "batch": 4095, "modulus": "ntt30"},
        # the benchmark's batch: 256 pairs of 8-channel ciphertexts
        {"name": "n4096_rns8_b256", "op": "rns", "n": 4096, "channels": 8, "batch": 256, "modulus": "ntt30"},
        # the largest degree of the homomorphic-encryption range, a few pairs
        {"name": "n16384_rns6_b8", "op": "rns", "n": 16384, "channels": 6, "batch": 8, "modulus": "ntt30"},
        # one plaintext or key times a batch of ciphertexts
        {"name": "n4096_rns8_b128_shared", "op": "rns_shared", "n": 4096, "channels": 8, "batch": 128,
         "modulus": "ntt30"},
        # the other ring, x^n - 1
        {"name": "n2048_cyclic_b1000", "op": "cyclic", "n": 2048, "channels": 1, "batch": 1000, "modulus": "ntt30"},
        # the Karatsuba route at the library's own choice of depth
        {"name": "n8192_rns8_b64_kara", "op": "rns_karatsuba", "n": 8192, "channels": 8, "batch": 64,
         "modulus": "ntt30"},
        # the paper's small-modulus residues and CRT
        {"name": "n4096_rns8_b64_crt", "op": "rns_crt", "n": 4096, "channels": 8, "batch": 64, "modulus": "ntt30"},
        # uneven degrees in one planned launch
        {"name": "uneven_plan", "op": "plan", "groups": "2048x256 512x1024 128x2048 64x4096 16x8192",
         "modulus": "ntt30"},
        # 64-bit coefficients at the largest degree, direct and through Karatsuba
        {"name": "n65536_goldilocks_b16", "op": "u64", "n": 65536, "channels": 1, "batch": 16,
         "modulus": "goldilocks"},
        {"name": "n65536_goldilocks_b16_kara", "op": "u64_karatsuba", "n": 65536, "channels": 1, "batch": 16,
         "modulus": "goldilocks"},
    ]


# op -> (weight, smallest and largest log2 n, channels, most words per operand, most products * n^2)
_RANGES = {
    "negacyclic": (4, 8, 15, (1, 1), 1 << 23, 1 << 34),
    "rns": (4, 10, 15, (2, 12), 1 << 23, 1 << 34),
    "shared": (1, 8, 13, (1, 1), 1 << 22, 1 << 34),
    "rns_shared": (1, 10, 13, (2, 12), 1 << 22, 1 << 34),
    "cyclic": (1, 8, 14, (1, 1), 1 << 22, 1 << 34),
    "rns_karatsuba": (1, 10, 14, (2, 12), 1 << 22, 1 << 34),
    "rns_crt": (1, 10, 12, (2, 8), 1 << 21, 1 << 32),
    "u64": (2, 10, 16, (1, 1), 1 << 20, 1 << 35),
    "u64_karatsuba": (1, 11, 16, (1, 1), 1 << 20, 1 << 35),
    "plan": (1, 0, 0, (1, 1), 0, 0),
}
# NTT primes most of all, then the moduli that other users bring
_MOD32 = ["ntt30"] * 6 + ["ntt28", "3329", "12289", "2147483647", "4294967291", "1048576"]
_MOD64 = ["goldilocks"] * 2 + ["ntt54", "ntt60", "ntt36"]


def _log_between(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    ops = sorted(_RANGES)
    op = rng.choices(ops, [_RANGES[o][0] for o in ops])[0]
    if op == "plan":
        groups = []
        for _ in range(rng.randint(2, 6)):
            n = 1 << rng.randint(8, 13)
            groups.append("%dx%d" % (_log_between(rng, 1, (1 << 19) // n), n))
        return {"op": op, "groups": " ".join(groups), "modulus": rng.choice(["ntt30", "ntt30", "ntt28"])}
    _, lo, hi, (c0, c1), words, macs = _RANGES[op]
    n = 1 << rng.randint(lo, hi)
    channels = rng.randint(c0, c1)
    most = max(1, min(words // (n * channels), macs // (n * n * channels)))
    return {"op": op, "n": n, "channels": channels, "batch": _log_between(rng, 1, most),
            "modulus": rng.choice(_MOD64 if op.startswith("u64") else _MOD32 if channels == 1 else _MOD32[:7])}


# ------------------------------------------------------------------------------ inputs
def _is_prime(p):
    if p % 2 == 0 or p < 3:
        return p == 2
    d, s = p - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for b in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if p % b == 0:
            return p == b
        x = pow(b, d, p)
        if x in (1, p - 1):
            continue
        for _ in range(s - 1):
            x = x * x % p
            if x == p - 1:
                break
        else:
            return False
    return True


def _moduli(kind, n, count, seed):
    """`count` moduli: fixed ones as they are, "nttB" as distinct B-bit primes = 1 mod 2n from the seed."""
    if kind == "goldilocks":
        return [GOLDILOCKS] * count
    if not kind.startswith("ntt"):
        return [int(kind)] * count
    bits = int(kind[3:])
    rng = np.random.default_rng([seed, n, bits])
    lo, hi = (1 << (bits - 1)) // (2 * n) + 1, ((1 << bits) - 2) // (2 * n)
    got = []
    while len(got) < count:
        q = int(rng.integers(lo, hi + 1)) * 2 * n + 1
        if q not in got and _is_prime(q):
            got.append(q)
    return got


def _uniform(gen, shape, q, wide):
    """Words uniform in [0, q) on the GPU (int32 or int64 bit patterns)."""
    if q < (1 << 63):
        x = torch.randint(0, q, shape, generator=gen, device="cuda", dtype=torch.int64)
        return x if wide else x.to(torch.int32) if q <= (1 << 31) else (x & 0xFFFFFFFF).to(torch.int32)
    hi = torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, device="cuda", dtype=torch.int64)
    lo = torch.randint(0, 1 << 32, shape, generator=gen, device="cuda", dtype=torch.int64)
    x = (hi << 32) | lo
    top = q - (1 << 64)  # q as a signed word: words at or above it (as unsigned) are taken down by q
    return torch.where((x < 0) & (x >= top), x - top, x)


def _groups(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["groups"].split()]


def _inputs(case, seed):
    """The operands and moduli of a case: a list of (a, b, moduli, n), one per group."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "plan":
        out = []
        for i, (count, n) in enumerate(_groups(case)):
            q = _moduli(case["modulus"], n, 1, seed + 7919 * i)[0]
            out.append((_uniform(gen, (count, n), q, False), _uniform(gen, (count, n), q, False), [q], n))
        return out
    n, L, batch, op = case["n"], case["channels"], case["batch"], case["op"]
    qs = _moduli(case["modulus"], n, L, seed)
    wide, rns = op.startswith("u64"), op.startswith("rns")
    if rns:
        a = torch.stack([_uniform(gen, (batch, n), q, wide) for q in qs], dim=1)
        b = (torch.stack([_uniform(gen, (n,), q, wide) for q in qs]) if op.endswith("shared") else
             torch.stack([_uniform(gen, (batch, n), q, wide) for q in qs], dim=1))
    else:
        a = _uniform(gen, (batch, n), qs[0], wide)
        b = _uniform(gen, (n,) if op == "shared" else (batch, n), qs[0], wide)
    return [(a, b, qs, n)]


def prepare(case, seed):
    """Operands and an output buffer on the GPU; the plan or the workspace where the route keeps one."""
    groups = _inputs(case, seed)
    op = case["op"]
    if op == "plan":
        held = [(a, b, torch.empty_like(a), n, qs[0]) for a, b, qs, n in groups]
        return {"op": op, "plan": pm.Plan(held), "c": [g[2] for g in held]}
    a, b, qs, n = groups[0]
    state = {"op": op, "a": a, "b": b, "qs": qs, "c": torch.empty_like(a)}
    if op == "rns_karatsuba":
        need = pm.polymul_karatsuba_workspace_size(n, len(qs), case["batch"], 0)
        state["ws"] = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
    if op == "u64_karatsuba":
        need = pm.polymul_karatsuba_u64_workspace_size(n, case["batch"], 0)
        state["ws"] = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    op = state["op"]
    if op == "plan":
        state["plan"].execute()
        return state["c"]
    a, b, c, qs = state["a"], state["b"], state["c"], state["qs"]
    if op == "negacyclic":
        return pm.polymul_negacyclic(a, b, qs[0], out=c)
    if op == "rns":
        return pm.polymul_negacyclic_rns(a, b, qs, out=c)
    if op == "shared":
        return pm.polymul_negacyclic_shared(a, b, qs[0], out=c)
    if op == "rns_shared":
        return pm.polymul_negacyclic_rns_shared(a, b, qs, out=c)
    if op == "cyclic":
        return pm.polymul_cyclic(a, b, qs[0], out=c)
    if op == "rns_karatsuba":
        return pm.polymul_negacyclic_rns_karatsuba(a, b, qs, 0, workspace=state["ws"], out=c)
    if op == "rns_crt":
        return pm.polymul_negacyclic_rns_crt(a, b, qs, out=c)
    if op == "u64":
        return pm.polymul_negacyclic_u64(a, b, qs[0], out=c)
    return pm.polymul_negacyclic_u64_karatsuba(a, b, qs[0], 0, workspace=state["ws"], out=c)


def work(case):
    """Operands read and products written once; the schoolbook product's n^2 multiply-adds of words."""
    if case["op"] == "plan":
        return {"bytes": sum(12 * k * n for k, n in _groups(case)),
                "flops": sum(2 * k * n * n for k, n in _groups(case))}
    n, products = case["n"], case["batch"] * case["channels"]
    word = 8 if case["op"].startswith("u64") else 4
    operands = products * n * 2 + (case["channels"] if case["op"].endswith("shared") else products) * n
    return {"bytes": operands * word, "flops": 2 * products * n * n}


# ------------------------------------------------------------------------------- exact
def _pieces(x, count):
    """11-bit pieces of non-negative words, lowest first (x: int64 words read as unsigned)."""
    return [((x >> (11 * i)) & 0x7FF if 11 * (i + 1) <= 63 else (x >> (11 * i)) & ((1 << (64 - 11 * i)) - 1))
            .to(torch.float64) for i in range(count)]


def _mod_add(x, y, q):
    """x + y mod q for uint64 words below q."""
    s = x + y
    return np.where((s < x) | (s >= q), s - q, s)


def _product(a, b, q, cyclic):
    """a * b in Z_q[x]/(x^n +- 1) for a [batch, n] and b [batch, n] or [n], any q < 2^64."""
    wide = a.dtype == torch.int64
    a64, b64 = (a, b) if wide else (a.to(torch.int64) & 0xFFFFFFFF, b.to(torch.int64) & 0xFFFFFFFF)
    n, count = a.shape[-1], 6 if wide else 3
    size = n if cyclic else 2 * n
    fb = [torch.fft.rfft(p, n=size) for p in _pieces(b64, count)]
    out = np.empty(a.shape, dtype=np.uint64 if wide else np.uint32)
    rows = max(1, (1 << 20) // n)
    for r0 in range(0, a.shape[0], rows):
        fa = [torch.fft.rfft(p, n=size) for p in _pieces(a64[r0:r0 + rows], count)]
        fbr = [f if b.dim() == 1 else f[r0:r0 + rows] for f in fb]
        acc = None
        for s in range(2 * count - 2, -1, -1):
            t = sum(fa[i] * fbr[s - i] for i in range(count) if 0 <= s - i < count)
            t = torch.round(torch.fft.irfft(t, n=size)).to(torch.int64)
            t = t if cyclic else t[..., :n] - t[..., n:]
            if not wide:  # below 2^32 * 2^11 + 2^41: 64-bit words hold it
                acc = torch.remainder(t if acc is None else acc * 2048 + t, q)
                continue
            t = t.cpu().numpy()
            t = np.where(t >= 0, t.astype(np.uint64), np.uint64(q) - (-t).astype(np.uint64)) if q > (1 << 45) else \
                np.mod(t, q).astype(np.uint64)
            if acc is not None:
                for _ in range(11):
                    acc = _mod_add(acc, acc, np.uint64(q))
                t = _mod_add(acc, t, np.uint64(q))
            acc = t
        out[r0:r0 + rows] = acc if wide else acc.cpu().numpy().astype(np.uint32)
    return torch.from_numpy(out.view(np.int64 if wide else np.int32))


def exact(case, seed):
    op = case["op"]
    got = []
    for a, b, qs, n in _inputs(case, seed):
        if op.startswith("rns"):
            got.append(torch.stack([_product(a[:, l], b[l] if b.dim() == 2 else b[:, l], q, False)
                                    for l, q in enumerate(qs)], dim=1))
        else:
            got.append(_product(a, b, qs[0], op == "cyclic"))
    return got if op == "plan" else got[0]
