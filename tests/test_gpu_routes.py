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


def direct64(name, a, b, q):
    """A 64-bit entry point of the C ABI, which takes no workspace: the streaming kernel above n = 4096."""
    da, db = to_dev(a), to_dev(b)
    c = torch.full_like(da, -1)
    st = getattr(pm.load_library(), name)(da.data_ptr(), db.data_ptr(), c.data_ptr(), a.shape[-1], q, a.shape[0],
                                          torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return c


def product64(name, a, b, q):
    return (oracle.cyclic if name == "polymul_cyclic_u64" else oracle.negacyclic)(
        a, np.ascontiguousarray(np.broadcast_to(b, a.shape)), q)


STREAM64 = ["polymul_negacyclic_u64", "polymul_cyclic_u64", "polymul_negacyclic_u64_shared"]


@pytest.mark.parametrize("n", [8192, 16384, 32768])
@pytest.mark.parametrize("name", STREAM64)
def test_streaming_kernel_64(name, n):
    """Several K-chunks of 1024; from n = 16384 on an int32 flush between them."""
    rng = np.random.default_rng(n)
    a = rng.integers(0, GOLD, size=(2, n), dtype=np.uint64)
    b = rng.integers(0, GOLD, size=(n,) if name.endswith("shared") else (2, n), dtype=np.uint64)
    check(direct64(name, a, b, GOLD), product64(name, a, b, GOLD), name)


@pytest.mark.parametrize("words", [(0x8080808080808080 % GOLD,) * 2, (0x7F7F7F7F7F7F7F7F,) * 2,
                                   (0x7F7F7F7F7F7F7F7F, 0x7F7F7F7F7F7F7F80)], ids=["low", "top", "top and below"])
@pytest.mark.parametrize("name", STREAM64)
def test_streaming_kernel_64_largest_class_sums(name, words):
    """Every digit at an end of its window over 16 K-chunks: the largest int32 class sums between flushes."""
    n = 16384
    a, b = (np.full((1, n), w, dtype=np.uint64) for w in words)
    if name.endswith("shared"):
        b = b[0]
    check(direct64(name, a, b, GOLD), product64(name, a, b, GOLD), name)


@pytest.mark.parametrize("even", [False, True])
def test_streaming_kernel_32_more_channels_than_a_launch(even):
    rng = np.random.default_rng(44)
    n, batch = 16384, 2
    qs = [Q30 + 2 * i - even for i in range(10)]
    a, b = (np.stack([draw(rng, (batch, n), q) for q in qs], axis=1) for _ in range(2))
    da, db = to_dev(a), to_dev(b)
    c = torch.full_like(da, -1)
    st = pm.load_library().polymul_negacyclic_rns(da.data_ptr(), db.data_ptr(), c.data_ptr(), n, np.array(qs, np.uint32).ctypes.data,
                                                  len(qs), batch, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    got = to_host(c, np.uint32)
    for l, q in enumerate(qs):
        pidx, jidx = np.arange(64, dtype=np.uint64) % batch, rng.integers(0, n, size=64, dtype=np.uint64)
        jidx[:4] = [0, 1, n - 2, n - 1]
        want = oracle.negacyclic_sample(a[:, l], b[:, l], q, pidx, jidx)
        assert np.array_equal(got[pidx.astype(np.int64), l, jidx.astype(np.int64)], want), f"channel {l}"


# even moduli and one above the transform's range, with two, three and four limbs
TILES = [3330, 1 << 20, Q30 - 1, (1 << 32) - 5]


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
@pytest.mark.parametrize("q", TILES)
def test_tiles_beside_the_transform(n, q):
    rng = np.random.default_rng([n, q])
    for batch in (1, 5, 37) if n < 8192 else (1, 5):
        a, b = draw(rng, (batch, n), 1 << 32), draw(rng, (batch, n), q)
        a[0], b[0] = q - 1, q - 1
        da, db = to_dev(a), to_dev(b)
        shared = np.ascontiguousarray(np.broadcast_to(b[-1], a.shape))
        check(pm.polymul_negacyclic_shared(da, db[-1].clone(), q), oracle.negacyclic(a, shared, q), f"shared, batch {batch}")
        if batch < 37:
            check(pm.polymul_negacyclic(da, db, q), oracle.negacyclic(a, b, q), f"batch {batch}")
            check(pm.polymul_cyclic(da, db, q), oracle.cyclic(a, b, q), f"cyclic, batch {batch}")


def test_shared_rows_in_chunks_on_tiles():
    """More products than a round of workgroups takes one by one: chunks that reuse the staged rows."""
    rng = np.random.default_rng(70)
    qs = [Q30 - 1, (1 << 32) - 5, 1 << 20]
    for n, batch in ((1024, 700), (4096, 200)):
        a = np.stack([draw(rng, (batch, n), q) for q in qs], axis=1)
        b = np.stack([draw(rng, n, q) for q in qs])
        want = oracle.negacyclic_rns(a, np.ascontiguousarray(np.broadcast_to(b, a.shape)), qs)
        check(pm.polymul_negacyclic_rns_shared(to_dev(a), to_dev(b), qs), want, f"n={n}")


@pytest.mark.parametrize("n,depth", [(2048, 1), (4096, 1), (8192, 1), (4096, 2), (8192, 3)])
def test_karatsuba_sub_products_on_tiles(n, depth):
    rng = np.random.default_rng([n, depth])
    qs = [Q30 - 1, (1 << 32) - 5, 3329]
    a, b = (np.stack([draw(rng, (3, n), q) for q in qs], axis=1) for _ in range(2))
    check(pm.polymul_negacyclic_rns_karatsuba(to_dev(a), to_dev(b), qs, depth), oracle.negacyclic_rns(a, b, qs), "mixed moduli")


@pytest.mark.parametrize("n,batch", [(4096, 5), (16384, 3)])
def test_depth_0_in_the_library_scratch(n, batch):
    rng = np.random.default_rng(n)
    qs = [Q30, 12289]
    a, b = (np.stack([draw(rng, (batch, n), q) for q in qs], axis=1) for _ in range(2))
    want = oracle.negacyclic_rns(a, b, qs)
    for _ in range(2):  # the second over what the first left
        check(pm.polymul_negacyclic_rns_karatsuba_noalloc(to_dev(a), to_dev(b), qs, 0), want, f"n={n}")


def edge_rows(rng, n, qs, word):
    """One row per modulus: all q - 1, zero against random, any words, q - 1 in every other place."""
    dtype = np.uint64 if word == 8 else np.uint32
    a, b = (np.stack([rng.integers(0, q, size=n, dtype=np.uint64).astype(dtype) for q in qs]) for _ in range(2))
    a[0], b[0] = qs[0] - 1, qs[0] - 1
    a[1] = 0
    a[2], b[2] = (rng.integers(0, 1 << 8 * word, size=n, dtype=np.uint64).astype(dtype) for _ in range(2))
    a[3] = dtype(qs[3] - 1) * (np.arange(n, dtype=dtype) % dtype(2))
    return a, b


@pytest.mark.parametrize("n", [32768, 65536])
@pytest.mark.parametrize("word", [4, 8])
def test_outer_transform_edges(n, word):
    """The radix-2 and radix-4 outer kernels with the largest sums, zeros and words outside [0, q)."""
    rng = np.random.default_rng([n, word])
    qs = [GOLD] * 4 if word == 8 else [0x7F7F7F7F, Q30, 3329, 0x7F7F7F7F]
    a, b = edge_rows(rng, n, qs, word)
    if word == 8:
        got = to_host(pm.polymul_negacyclic_u64(to_dev(a), to_dev(b), GOLD), np.uint64)
    else:
        got = to_host(pm.polymul_negacyclic_rns(to_dev(a[None]), to_dev(b[None]), qs), np.uint32)[0]
    assert not got[1].any()
    jidx = np.concatenate([np.arange(256), np.arange(n - 256, n), rng.integers(0, n, size=512)]).astype(np.uint64)
    for l, q in enumerate(qs):
        want = oracle.negacyclic_sample(a[l:l + 1], b[l:l + 1], q, np.zeros_like(jidx), jidx)
        assert np.array_equal(got[l, jidx.astype(np.int64)], want), f"row {l}"
