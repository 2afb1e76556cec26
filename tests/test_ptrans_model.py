"""The polynomial transform against the definition, on the CPU: every transform size, the split of
x^n - 1, the outer radix step, over odd moduli from 3 to the largest the route takes."""
import numpy as np
import pytest

import oracle
import ptrans_model as pt

QS = [3, 257, 3329, 1068236801, 0x7F7F7F7F]


def operands(n, q):
    rng = np.random.default_rng([n, q])
    a, b = rng.integers(0, q, n), rng.integers(0, q, n)
    a[: n // 2], b[1::3] = q - 1, q - 1
    return a, b


def by_oracle(fn, q):
    return lambda a, b: fn(a.astype(np.uint32)[None], b.astype(np.uint32)[None], q)[0].astype(np.int64)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("k", [2, 4, 8, 16])
def test_transform_is_the_product(k, q):
    product = by_oracle(oracle.negacyclic, q)
    a, b = operands(32 * k, q)
    want = product(a, b)
    assert np.array_equal(pt.negacyclic(a, b, k, q, product), want)
    if k >= 8:  # the outer kernels' two steps
        assert all(np.array_equal(x, y) for x, y in zip(pt.forward(a, k, q), pt.forward_radix(a, k, q)))
        assert np.array_equal(pt.negacyclic(a, b, k, q, product, pt.forward_radix, pt.inverse_radix), want)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("k", [4, 8, 16])
def test_cyclic_split_is_the_product(k, q):
    a, b = operands(32 * k, q)
    got = pt.cyclic(a, b, k, q, by_oracle(oracle.negacyclic, q), by_oracle(oracle.cyclic, q))
    assert np.array_equal(got, by_oracle(oracle.cyclic, q)(a, b))


def test_a_wrong_root_fails():
    q, k = 1068236801, 8
    product = by_oracle(oracle.negacyclic, q)
    a, b = operands(32 * k, q)
    shifted = lambda c, k, q: pt.inverse([pt.rot(x, s == 3, q) for s, x in enumerate(c)], k, q)
    assert not np.array_equal(pt.negacyclic(a, b, k, q, product, inv=shifted), product(a, b))
