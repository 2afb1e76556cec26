"""The polynomial-transform route (32-bit words, odd moduli) word for word against
the oracle: every transform size with full and ragged workgroups, moduli at the ends of its
range and of each limb count's window, mixed moduli in one workgroup, words outside [0, q),
the operands whose sums are largest, a modulus just outside the range beside one inside, and
the ring x^n - 1."""
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


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
@pytest.mark.parametrize("q", [3, 257, 3329, 32639, 32641, 65537, 8355711, 8355713, 16777213, Q30, Q_TOP, Q_TOP + 2,
                               Q30 - 1])
def test_moduli(n, q):
    rng = np.random.default_rng([n, q])
    for batch in (1, 7):  # 7: a ragged last workgroup at 1024 and 2048
        a, b = edge_operands(rng, batch, n, q)
        got = to_host(pm.polymul_negacyclic(to_dev(a), to_dev(b), q), np.uint32)
        check(got, oracle.negacyclic(a, b, q), f"n={n}, q={q}, batch {batch}")


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
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


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
@pytest.mark.parametrize("q", [3, 257, 32639, 32641, 8355711, 8355713, Q30, Q_TOP, Q_TOP + 2, Q30 - 1])
def test_cyclic_ring(n, q):
    rng = np.random.default_rng([n, q, 1])
    for batch in (1, 4, 7):  # 4: the smallest call on the route at 1024; 7: a ragged last workgroup
        a, b = edge_operands(rng, batch, n, q)
        got = to_host(pm.polymul_cyclic(to_dev(a), to_dev(b), q), np.uint32)
        check(got, oracle.cyclic(a, b, q), f"n={n}, q={q}, batch {batch}")


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


GOLDILOCKS = (1 << 64) - (1 << 32) + 1


def edge_operands64(rng, batch, n, q):
    a = rng.integers(0, q, size=(batch, n), dtype=np.uint64)
    b = rng.integers(0, q, size=(batch, n), dtype=np.uint64)
    if batch > 3:
        a[0], b[0] = q - 1, q - 1
        a[1] = 0
        if q >= 1 << 32:  # the oracle reads operands of smaller moduli as 32-bit words
            a[2] = rng.integers(0, 1 << 64, size=n, dtype=np.uint64)
            b[2] = rng.integers(0, 1 << 64, size=n, dtype=np.uint64)
        a[3], b[3] = np.uint64(q - 1) * (np.arange(n, dtype=np.uint64) % 2), q // 2
    return a, b


@pytest.mark.parametrize("n", [1024, 2048, 4096])
@pytest.mark.parametrize("q", [3, 65537, (1 << 32) - 5, (1 << 36) - 5, (1 << 48) - 59, (1 << 48) + 21, (1 << 63) - 25,
                               (1 << 63) + 29, 0x7F7F7F7F7F7F7F7F, 0x7F7F7F7F7F7F7F81, GOLDILOCKS, (1 << 64) - 1,
                               (1 << 54) - 32])
def test_moduli64(n, q):
    rng = np.random.default_rng([n, q & 0xFFFFFFFF, q >> 32])
    a, b = edge_operands64(rng, 5, n, q)
    da, db = to_dev(a), to_dev(b)
    want = oracle.negacyclic(a, b, q)
    check(to_host(pm.polymul_negacyclic_u64(da, db, q), np.uint64), want, f"n={n}, q={q}")
    shared = oracle.negacyclic(a, np.ascontiguousarray(np.broadcast_to(b[4], b.shape)), q)
    check(to_host(pm.polymul_negacyclic_u64_shared(da, db[4].clone(), q), np.uint64), shared, f"shared n={n}, q={q}")
    check(to_host(pm.polymul_negacyclic_u64_karatsuba(da, db, q, 0), np.uint64), want, f"depth 0 n={n}, q={q}")


@pytest.mark.parametrize("n,batch", [(8192, 5), (16384, 4), (32768, 1), (65536, 1)])
def test_outer_transform(n, batch):
    """Degrees above 4096: the route with a workspace, and the direct calls that take one from torch."""
    rng = np.random.default_rng(n)
    for q in (GOLDILOCKS, (1 << 36) - 5):
        a, b = edge_operands64(rng, batch, n, q)
        want = oracle.negacyclic(a, b, q)
        check(to_host(pm.polymul_negacyclic_u64_karatsuba(to_dev(a), to_dev(b), q, 0), np.uint64), want, f"{n}, {q}")
        check(to_host(pm.polymul_negacyclic_u64(to_dev(a), to_dev(b), q), np.uint64), want, f"direct {n}, {q}")
    qs = [Q30, Q_TOP, 3329]
    pairs = [edge_operands(rng, batch, n, q) for q in qs]
    a, b = (np.ascontiguousarray(np.stack([p[i] for p in pairs], axis=1)) for i in (0, 1))
    want = oracle.negacyclic_rns(a, b, qs)
    check(to_host(pm.polymul_negacyclic_rns_karatsuba(to_dev(a), to_dev(b), qs, 0), np.uint32), want, f"rns {n}")
    check(to_host(pm.polymul_negacyclic_rns(to_dev(a), to_dev(b), qs), np.uint32), want, f"rns direct {n}")
    check(to_host(pm.polymul_negacyclic(to_dev(a[:, 0].copy()), to_dev(b[:, 0].copy()), Q30), np.uint32),
          np.ascontiguousarray(want[:, 0]), f"direct {n}")


def test_direct_call_in_chunks_and_on_another_stream(monkeypatch):
    rng = np.random.default_rng(8)
    a, b = edge_operands64(rng, 5, 8192, GOLDILOCKS)
    want = oracle.negacyclic(a, b, GOLDILOCKS)
    da, db = to_dev(a), to_dev(b)
    import torch
    from paper_2307_06554_amd import binding
    per_row = pm.polymul_karatsuba_u64_workspace_size(8192, 1, 0)
    monkeypatch.setattr(binding, "_WS_BYTES", 2 * per_row)  # chunks of 2, 2 and 1 products
    check(to_host(pm.polymul_negacyclic_u64(da, db, GOLDILOCKS), np.uint64), want, "chunks")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    c = torch.full_like(da, -1)
    pm.polymul_negacyclic_u64(da, db, GOLDILOCKS, out=c, stream=s)  # not torch's current stream: no workspace
    check(to_host(c, np.uint64), want, "stream argument")
    with torch.cuda.stream(s):
        got = pm.polymul_negacyclic_u64(da, db, GOLDILOCKS)
    s.synchronize()
    check(to_host(got, np.uint64), want, "current stream")


def test_overlapping_output_is_refused_whatever_the_chunks(monkeypatch):
    import torch
    from paper_2307_06554_amd import binding
    buf = torch.zeros((8, 8192), dtype=torch.int64, device="cuda")
    b = torch.zeros((5, 8192), dtype=torch.int64, device="cuda")
    monkeypatch.setattr(binding, "_WS_BYTES", pm.polymul_karatsuba_u64_workspace_size(8192, 1, 0))  # rows one by one
    for x, y in ((buf[:5], b), (b, buf[:5])):
        with pytest.raises(pm.PolymulError):
            pm.polymul_negacyclic_u64(x, y, GOLDILOCKS, out=buf[3:])


def test_captured_call_takes_no_workspace(monkeypatch):
    import torch
    from paper_2307_06554_amd import binding
    rng = np.random.default_rng(10)
    a, b = edge_operands64(rng, 2, 8192, GOLDILOCKS)
    want = oracle.negacyclic(a, b, GOLDILOCKS)
    da, db = to_dev(a), to_dev(b)
    c = torch.empty_like(da)
    pm.polymul_negacyclic_u64(da, db, GOLDILOCKS, out=c)
    sizes = []
    size = binding.polymul_karatsuba_u64_workspace_size
    monkeypatch.setattr(binding, "polymul_karatsuba_u64_workspace_size", lambda *v: sizes.append(v) or size(*v))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pm.polymul_negacyclic_u64(da, db, GOLDILOCKS, out=c)
    assert not sizes
    for _ in range(3):
        c.fill_(-1)
        graph.replay()
        check(to_host(c, np.uint64), want, "replay")
        check(to_host(pm.polymul_negacyclic_u64(da, db, GOLDILOCKS), np.uint64), want, "eager between replays")


def test_plan_groups():
    """Plan items on the transform: full and ragged items of every degree, two groups of n = 8192 (their
    sub-products share the plan's buffer), moduli that stay on the tiles beside them, replays."""
    rng = np.random.default_rng(9)
    shapes = [(1024, 5, Q30), (1024, 4, Q_TOP), (2048, 3, Q30 + 2), (4096, 2, Q30), (8192, 2, Q30), (8192, 1, Q_TOP),
              (8192, 1, Q30 - 1), (4096, 1, 12289), (2048, 1, Q_TOP + 2), (256, 9, Q30)]
    operands = [edge_operands(rng, count, n, q) for n, count, q in shapes]
    operands[4][0][1] = draw(rng, 8192, 1 << 32)  # words outside [0, q) through the Karatsuba level
    held = [(to_dev(a), to_dev(b), to_dev(np.full_like(a, 7)), n, q) for (a, b), (n, _, q) in zip(operands, shapes)]
    want = [oracle.negacyclic(a, b, q) for (a, b), (_, _, q) in zip(operands, shapes)]
    for flags in (0, 1):
        plan = pm.Plan(held, flags)
        for _ in range(2):
            for g in held:
                g[2].fill_(-1)
            plan.execute()
            for g, w in zip(held, want):
                check(to_host(g[2], np.uint32), w, f"n={g[3]}, q={g[4]}, flags {flags}")
        plan.close()
