"""Routes that the library's own choice leaves to special sizes, pinned to the kernels they are about by
entry point, modulus or batch, word for word against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2307_06554_amd as pm
from paper_2307_06554_amd import binding, inputs
from gpu_util import to_dev, to_host, mismatch_report

pytestmark = pytest.mark.gpu

GOLD = inputs.GOLDILOCKS
Q30 = 1068236801


def draw(rng, shape, q):
    return rng.integers(0, q, size=shape, dtype=np.uint64).astype(np.uint32)


def check(got, want, what):
    got = to_host(got, want.dtype)
    assert np.array_equal(got, want), what + ": " + mismatch_report(got, want)


@pytest.mark.parametrize("shapes", [
    [(3, 8192)], [(12, 8192)], [(14, 4096)], [(6, 8192), (6, 4096)], [(7, 8192), (30, 256)], [(5, 1024)], [(769, 1024)],
], ids=lambda s: "+".join(f"{c}x{n}" for c, n in s))
def test_light_plans(shapes):
    """Plans at the edges of the rule between tiles and transform: K-split runs of whole products, n = 1024
    on either side."""
    rng = np.random.default_rng(len(shapes) * 7919 + shapes[0][0])
    held, want = [], []
    for count, n in shapes:
        a, b = draw(rng, (count, n), Q30), draw(rng, (count, n), Q30)
        a[0], b[0] = Q30 - 1, Q30 - 1
        held.append((to_dev(a), to_dev(b), to_dev(np.full_like(a, 7)), n, Q30))
        want.append(oracle.negacyclic(a, b, Q30))
    for flags in (0, 1):
        plan = pm.Plan(held, flags)
        for _ in range(2):
            for g in held:
                g[2].fill_(-1)
            plan.execute()
            for g, w in zip(held, want):
                check(g[2], w, f"n={g[3]}, flags {flags}")
        plan.close()


@pytest.mark.parametrize("n,L,batch", [(8192, 1, 3), (8192, 2, 28), (8192, 3, 19), (1024, 2, 96), (1024, 1, 193)])
def test_depth_0_on_either_side_of_the_few(n, L, batch):
    rng = np.random.default_rng([n, batch])
    qs = [Q30, 12289, 0x7F7F7F7F][:L]
    a, b = (np.stack([draw(rng, (batch, n), q) for q in qs], axis=1) for _ in range(2))
    a[0], b[0] = np.array(qs, dtype=np.uint32)[:, None] - 1, draw(rng, (L, n), 1 << 32)
    want = oracle.negacyclic_rns(a, b, qs)
    da, db = to_dev(a), to_dev(b)
    check(pm.polymul_negacyclic_rns_karatsuba(da, db, qs, 0), want, "caller's workspace")
    check(pm.polymul_negacyclic_rns_karatsuba_noalloc(da, db, qs, 0), want, "the library's scratch")
