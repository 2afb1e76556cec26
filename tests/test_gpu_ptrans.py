"""The polynomial-transform route (32-bit words, odd moduli) word for word against
the oracle: every transform size with full and ragged workgroups, moduli at the ends of its
range and of each limb count's window, mixed moduli in one workgroup, words outside [0, q),
the operands whose sums are largest, and a modulus just outside the range beside one inside."""
import numpy as np
import pytest

import oracle
import paper_2307_06554_amd as pm
from gpu_util import to_dev, to_host, mismatch_report

pytestmark = pytest.mark.gpu

Q_TOP = 0x7F7F7F7F  # the largest modulus the route takes
Q30 = 1068236801


def draw(rng, shape, q):
    return rng.integers(0, q, size=shape, dtype=np.uint64).astype(np.uint32)


def edge_operands(rng, batch, n, q):
    """Random rows, with all q - 1, all zero and any-32-bit-word rows among them."""
    a, b = draw(rng, (batch, n), q), draw(rng, (batch, n), q)
    if batch > 3:
        a[0], b[0] = q - 1, q - 1
        a[1] = 0
        a[2], b[2] = draw(rng, n, 1 << 32), draw(rng, n, 1 << 32)
        a[3], b[3] = (q - 1) * (np.arange(n) % 2), q // 2
    return a, b


def check(got, want, what):
    assert np.array_equal(got, want), what + ": " + mismatch_report(got, want)


@pytest.mark.parametrize("n", [1024, 2048, 4096])
@pytest.mark.parametrize("q", [3, 257, 3329, 32639, 32641, 65537, 8355711, 8355713, 16777213, Q30, Q_TOP, Q_TOP + 2,
                               Q30 - 1])
def test_moduli(n, q):
    rng = np.random.default_rng([n, q])
    for batch in (1, 7):  # 7: a ragged last workgroup at 1024 and 2048
        a, b = edge_operands(rng, batch, n, q)
        got = to_host(pm.polymul_negacyclic(to_dev(a), to_dev(b), q), np.uint32)
        check(got, oracle.negacyclic(a, b, q), f"n={n}, q={q}, batch {batch}")


@pytest.mark.parametrize("n", [1024, 2048, 4096])
def test_channels_and_shared_operand(n):
    rng = np.random.default_rng(n)
    qs = [Q30, 12289, Q_TOP] + [Q30 + 2 * i for i in range(1, 16)]  # 18: two launches
    a = np.stack([edge_operands(rng, 5, n, q)[0] for q in qs], axis=1)
    b = np.stack([edge_operands(rng, 5, n, q)[1] for q in qs], axis=1)
    check(to_host(pm.polymul_negacyclic_rns(to_dev(a), to_dev(b), qs), np.uint32), oracle.negacyclic_rns(a, b, qs),
          f"rns n={n}")
    bs = np.ascontiguousarray(b[2])
    want = oracle.negacyclic_rns(a, np.ascontiguousarray(np.broadcast_to(bs, a.shape)), qs)
    check(to_host(pm.polymul_negacyclic_rns_shared(to_dev(a), to_dev(bs), qs), np.uint32), want, f"shared n={n}")


def test_a_tile_side_turns_the_route_off_with_the_same_result():
    rng = np.random.default_rng(5)
    a, b = edge_operands(rng, 5, 2048, Q30)
    da, db = to_dev(a), to_dev(b)
    want = to_host(pm.polymul_negacyclic(da, db, Q30), np.uint32)
    try:
        for t in (32, 64, 128):
            pm.polymul_tune_set(2048, 4, t)
            check(to_host(pm.polymul_negacyclic(da, db, Q30), np.uint32), want, f"t={t}")
    finally:
        pm.polymul_tune_set(2048, 4, 0)
    check(want, oracle.negacyclic(a, b, Q30), "transform")
