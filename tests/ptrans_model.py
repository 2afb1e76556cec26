"""numpy model of the polynomial transform (csrc/pm_ptrans.h): products of degree bound k M as
2k negacyclic products of degree bound M, the split of x^n - 1, and the radix-R step of the outer
transform.  Arrays are int64 residues, q < 2^31; `product` multiplies in Z_q[y]/(y^M + 1)."""
import numpy as np


def bitrev(x, bits):
    return int(format(x, f"0{bits}b")[::-1], 2) if bits else 0


def rot(p, e, q):
    """y^e p mod y^M + 1."""
    m = len(p)
    e %= 2 * m
    r = np.roll(p, e % m)
    r[:e % m] = -r[:e % m]
    return (-r if e >= m else r) % q


def stages(v, first, direction, q):
    """Decimation in time over v (bit-reversed in, natural out): block sizes first .. len(v)."""
    size = first
    while size <= len(v):
        for j in range(size // 2):
            for b in range(0, len(v), size):
                m = len(v[b])
                t = rot(v[b + j + size // 2], direction * j * (2 * m // size), q)
                v[b + j], v[b + j + size // 2] = (v[b + j] + t) % q, (v[b + j] - t) % q
        size *= 2


def forward(a, k, q):
    """The 2k points of a (k columns' coefficients a[i + k j])."""
    cols, bits = a.reshape(-1, k).T, k.bit_length() - 1
    v = [cols[bitrev(p // 2, bits)].copy() for p in range(2 * k)]
    stages(v, 4, 1, q)
    return v


def inverse(c, k, q):
    """The product from its points' products, times 2k."""
    bits, m = k.bit_length() - 1, len(c[0])
    e, o = [None] * k, [None] * k
    for s in range(2 * k):
        y = rot(c[s], 1, q)
        (o if s & 1 else e)[bitrev(s >> 1, bits)] = (c[s] - y if s & 1 else c[s] + y) % q
    stages(e, 2, -1, q)
    stages(o, 2, -1, q)
    return np.stack([(e[i] + rot(o[i], -i * (m // k), q)) % q for i in range(k)]).T.reshape(-1)


def forward_radix(a, k, q):
    """The same points through k / 4 transforms of 4 columns and one step of radix R = k / 4."""
    r, m = k // 4, len(a) // k
    u = [forward(a.reshape(-1, k).T[i0::r].T.reshape(-1), 4, q) for i0 in range(r)]
    w = m // k
    return [sum(rot(rot(u[i0][s % 8], i0 * (s % 8) * w, q), 8 * i0 * (s // 8) * w, q) for i0 in range(r)) % q
            for s in range(2 * k)]


def inverse_radix(c, k, q):
    r, m = k // 4, len(c[0])
    w = m // k
    out = np.empty(k * m, dtype=np.int64)
    for i0 in range(r):
        v = [rot(sum(rot(c[s + 8 * t], -8 * i0 * t * w, q) for t in range(r)) % q, -i0 * s * w, q) for s in range(8)]
        out.reshape(-1, k).T[i0::r] = inverse(v, 4, q).reshape(-1, 4).T
    return out


def negacyclic(a, b, k, q, product, fwd=forward, inv=inverse):
    c = [product(x, y) for x, y in zip(fwd(a, k, q), fwd(b, k, q))]
    return inv(c, k, q) * pow(2 * k, -1, q) % q


def cyclic(a, b, k, q, product, cyclic_product):
    """x^n - 1 with n = k M: the factors x^(n/2) + 1 .. x^M + 1 and x^M - 1, one common scale 1/(2k)."""
    def levels(x):
        out = []
        while len(x) > len(a) // k:
            lo, hi = x[:len(x) // 2], x[len(x) // 2:]
            out.append((lo - hi) % q)
            x = (lo + hi) % q
        return out, x
    (la, ra), (lb, rb) = levels(a), levels(b)
    scale = pow(2 * k, -1, q)
    s = 2 * scale * cyclic_product(ra, rb) % q
    for x, y in zip(reversed(la), reversed(lb)):
        cols = len(x) * k // len(a)
        if cols == 1:
            d = 2 * scale * product(x, y) % q
        else:
            c = [scale * product(p, r) % q for p, r in zip(forward(x, cols, q), forward(y, cols, q))]
            d = inverse(c, cols, q)
        s = np.concatenate([s + d, s - d]) % q
    return s
