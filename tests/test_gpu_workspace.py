"""The workspace that direct products of large degree take from torch's allocator: how much, in
which chunks, whatever the Karatsuba table says, and what happens where there is none to have."""
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


def operands(n, batch, q, word, seed=0):
    rng = np.random.default_rng([n, batch, seed])
    dtype = np.uint64 if word == 8 else np.uint32
    a, b = (rng.integers(0, q, size=(batch, n), dtype=np.uint64).astype(dtype) for _ in range(2))
    return a, b, oracle.negacyclic(a, b, q)


def direct(word):
    return pm.polymul_negacyclic_u64 if word == 8 else pm.polymul_negacyclic


def check(got, want, what):
    got = to_host(got, want.dtype)
    assert np.array_equal(got, want), what + ": " + mismatch_report(got, want)


@pytest.fixture
def asked(monkeypatch):
    """Sizes of the byte tensors asked of torch.empty; those above `asked.limit` find no room."""
    class Sizes(list):
        limit = None
    sizes, empty = Sizes(), torch.empty

    def spy(*shape, **kw):
        if kw.get("dtype") is torch.uint8:
            sizes.append(shape[0])
            if sizes.limit is not None and shape[0] > sizes.limit:
                raise torch.cuda.OutOfMemoryError("no room")
        return empty(*shape, **kw)

    monkeypatch.setattr(torch, "empty", spy)
    return sizes


@pytest.mark.parametrize("n,word,q", [(16384, 4, Q30), (65536, 4, 3329), (8192, 8, GOLD), (65536, 8, GOLD)])
def test_size_and_chunks(asked, monkeypatch, n, word, q):
    a, b, want = operands(n, 3, q, word)
    da, db = to_dev(a), to_dev(b)
    check(direct(word)(da, db, q), want, "one chunk")
    monkeypatch.setattr(binding, "_WS_BYTES", 2 * 4 * n * word + 5)  # chunks of 2 and 1
    check(direct(word)(da, db, q), want, "two chunks")
    assert asked == [3 * 4 * n * word, 2 * 4 * n * word]


@pytest.mark.parametrize("depth", [0, 1])
def test_karatsuba_table_does_not_touch_direct_calls(asked, depth):
    for n, word, q in ((16384, 4, Q30), (16384, 8, GOLD)):
        a, b, want = operands(n, 2, q, word)
        pm.polymul_tune_set_karatsuba(n, 2, word, depth)
        try:
            check(direct(word)(to_dev(a), to_dev(b), q), want, f"{word} bytes a word")
        finally:
            pm.polymul_tune_set_karatsuba(n, 2, word, binding.KARATSUBA_BUILTIN)
        assert asked.pop() == 2 * 4 * n * word


def test_captured_call_asks_for_none(asked):
    a, b, want = operands(8192, 2, GOLD, 8)
    da, db = to_dev(a), to_dev(b)
    c = torch.empty_like(da)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pm.polymul_negacyclic_u64(da, db, GOLD, out=c)
    assert not asked
    for _ in range(3):
        c.fill_(-1)
        graph.replay()
        check(c, want, "replay")


@pytest.mark.parametrize("in_thread", [False, True], ids=["same thread", "other thread"])
def test_call_beside_a_capture(in_thread):
    """A direct call on one stream while another one is captured in the default, global mode: torch has
    to call hipMalloc for the workspace, and neither the call nor the capture minds."""
    import threading
    n, batch = 65536, 16
    rng = np.random.default_rng(3)
    da, db = (to_dev(rng.integers(0, GOLD, size=(batch, n), dtype=np.uint64)) for _ in range(2))
    want = pm.polymul_negacyclic_u64(da, db, GOLD)
    c, x, side, errors = torch.empty_like(da), torch.zeros(64, device="cuda"), torch.cuda.Stream(), []

    def call():
        try:
            with torch.cuda.stream(side):
                pm.polymul_negacyclic_u64(da, db, GOLD, out=c)
        except Exception as e:
            errors.append(e)

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):  # empties torch's cache first
        x.add_(1)
        if in_thread:
            thread = threading.Thread(target=call)
            thread.start()
            thread.join()
        else:
            call()
    assert not errors
    side.synchronize()
    assert torch.equal(c, want)
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert x.eq(3).all()


def test_little_room(asked):
    """Where there is no room for a chunk, smaller ones before the call goes without a workspace."""
    n, row = 8192, 4 * 8192 * 8
    a, b, want = operands(n, 11, GOLD, 8)
    da, db = to_dev(a), to_dev(b)
    asked.limit = row
    check(pm.polymul_negacyclic_u64(da, db, GOLD), want, "rows one by one")
    assert asked == [11 * row, 3 * row, row]
    asked.clear()
    asked.limit = 0
    check(pm.polymul_negacyclic_u64(da, db, GOLD), want, "no workspace")
    assert asked == [11 * row, 3 * row, row]
